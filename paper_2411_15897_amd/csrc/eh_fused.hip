// One precision and one leg of the fused multigrid cycle (EH_T: float or
// double, EH_UP: 0 down, 1 up): kernels and their launch.
#include "eh_launch.h"
#include "eh_fused_kernels.h"

namespace eh {

#if EH_UP == 0

template <class T>
void launch_fdown(hipStream_t stream, const GArgs<T>& a, int l, int cfg, int nrhs) {
    const FCfg k = kFDown[cfg];
    int gx = 1, gy = 1;
    for (int s = 0; s < a.ns; ++s) {
        gx = std::max(gx, (a.dc[s].g[0] + k.x - 1) / k.x);
        gy = std::max(gy, (a.dc[s].g[1] + k.y - 1) / k.y);
    }
    const int rch = rhs_chunk(gx * gy, a.ns, nrhs);
    const int nch = (std::max(nrhs, 1) + rch - 1) / rch;
    const dim3 g((unsigned)gx, (unsigned)gy, (unsigned)(a.ns * nch)), blk((unsigned)k.threads);
#define EH_LFD(CF)                                                                               \
    if (l == 0) hipLaunchKernelGGL((k_fdown<T, true, CF>), g, blk, 0, stream, a, nrhs, rch);     \
    else hipLaunchKernelGGL((k_fdown<T, false, CF>), g, blk, 0, stream, a, nrhs, rch);
    switch (cfg) {
        case 0: EH_LFD(0) break;
        case 1: EH_LFD(1) break;
        case 2: EH_LFD(2) break;
        default: EH_LFD(3) break;
    }
#undef EH_LFD
}

template void launch_fdown<EH_T>(hipStream_t, const GArgs<EH_T>&, int, int, int);

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
#define EH_LFU(CF)                                                                                    \
    if (l == 0) {                                                                                     \
        if (two) hipLaunchKernelGGL((k_fup<T, true, 2, CF>), g, blk, 0, stream, a, nrhs, rch);        \
        else hipLaunchKernelGGL((k_fup<T, true, 1, CF>), g, blk, 0, stream, a, nrhs, rch);            \
    } else {                                                                                          \
        if (two) hipLaunchKernelGGL((k_fup<T, false, 2, CF>), g, blk, 0, stream, a, nrhs, rch);       \
        else hipLaunchKernelGGL((k_fup<T, false, 1, CF>), g, blk, 0, stream, a, nrhs, rch);           \
    }
    switch (cfg) {
        case 0: EH_LFU(0) break;
        case 1: EH_LFU(1) break;
        case 2: EH_LFU(2) break;
        default: EH_LFU(3) break;
    }
#undef EH_LFU
}

template void launch_fup<EH_T>(hipStream_t, int, const GArgs<EH_T>&, int, int, int);

#endif

}  // namespace eh
