// One precision and one leg of the fused multigrid cycle (EH_T: float or
// double, EH_UP: 0 down, 1 up): kernels and their launch.
#include "eh_launch.h"
#include "eh_fused_kernels.h"

namespace eh {

#if EH_UP == 0

template <class T>
void launch_fdown(hipStream_t stream, const GArgs<T>& a, int l, int cfg, int nrhs, const CplArgs<T>* cpl) {
    const FCfg k = kFDown[cfg];
    int gx = 1, gy = 1;
    for (int s = 0; s < a.ns; ++s) {
        gx = std::max(gx, (a.dc[s].g[0] + k.x - 1) / k.x);
        gy = std::max(gy, (a.dc[s].g[1] + k.y - 1) / k.y);
    }
    const int rch = rhs_chunk(gx * gy, a.ns, nrhs);
    const int nch = (std::max(nrhs, 1) + rch - 1) / rch;
    const dim3 g((unsigned)gx, (unsigned)gy, (unsigned)(a.ns * nch)), blk((unsigned)k.threads);
    const bool pb = a.kind[0] == 2;
    const NoCpl no{};
#define EH_LFD(CF)                                                                                        \
    if (cpl) {                                                                                            \
        hipLaunchKernelGGL((k_fdown<T, true, CF, false, CplArgs<T>>), g, blk, 0, stream, a, nrhs, rch, *cpl); \
    } else if (l == 0) {                                                                                  \
        if (pb) hipLaunchKernelGGL((k_fdown<T, true, CF, true>), g, blk, 0, stream, a, nrhs, rch, no);    \
        else hipLaunchKernelGGL((k_fdown<T, true, CF, false>), g, blk, 0, stream, a, nrhs, rch, no);      \
    } else {                                                                                              \
        if (pb) hipLaunchKernelGGL((k_fdown<T, false, CF, true>), g, blk, 0, stream, a, nrhs, rch, no);   \
        else hipLaunchKernelGGL((k_fdown<T, false, CF, false>), g, blk, 0, stream, a, nrhs, rch, no);     \
    }
    switch (cfg) {
        case 0: EH_LFD(0) break;
        case 1: EH_LFD(1) break;
        case 2: EH_LFD(2) break;
        default: EH_LFD(3) break;
    }
#undef EH_LFD
}

template void launch_fdown<EH_T>(hipStream_t, const GArgs<EH_T>&, int, int, int, const CplArgs<EH_T>*);

#else

template <class T>
void launch_fup(hipStream_t stream, int nu_post, const GArgs<T>& a, int l, int cfg, int nrhs) {
    const FCfg k = kFUp[cfg];
    int gx = 1, gy = 1;
    for (int s = 0; s < a.ns; ++s) {
        gx = std::max(gx, (a.d[s].g[0] + k.x - 1) / k.x);
        gy = std::max(gy, (a.d[s].g[1] + k.y - 1) / k.y);
    }
    const int rch = rhs_chunk(gx * gy, a.ns, nrhs);
    const int nch = (std::max(nrhs, 1) + rch - 1) / rch;
    const dim3 g((unsigned)gx, (unsigned)gy, (unsigned)(a.ns * nch)), blk((unsigned)k.threads);
    const bool two = nu_post == 2;
    const bool pb = a.kind[0] == 2;
#define EH_LFU1(CF, FI, NU)                                                                            \
    if (pb) hipLaunchKernelGGL((k_fup<T, FI, NU, CF, true>), g, blk, 0, stream, a, nrhs, rch);         \
    else hipLaunchKernelGGL((k_fup<T, FI, NU, CF, false>), g, blk, 0, stream, a, nrhs, rch);
#define EH_LFU(CF)                                                                                     \
    if (l == 0) {                                                                                      \
        if (two) { EH_LFU1(CF, true, 2) } else { EH_LFU1(CF, true, 1) }                                \
    } else {                                                                                           \
        if (two) { EH_LFU1(CF, false, 2) } else { EH_LFU1(CF, false, 1) }                              \
    }
    switch (cfg) {
        case 0: EH_LFU(0) break;
        case 1: EH_LFU(1) break;
        case 2: EH_LFU(2) break;
        default: EH_LFU(3) break;
    }
#undef EH_LFU
#undef EH_LFU1
}

template void launch_fup<EH_T>(hipStream_t, int, const GArgs<EH_T>&, int, int, int);

#endif

}  // namespace eh
