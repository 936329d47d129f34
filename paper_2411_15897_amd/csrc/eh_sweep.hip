// The per-sweep multigrid kernels and transfers of one precision (EH_T:
// float or double) and their launches.
#include "eh_launch.h"
#include "eh_fine3_kernels.h"
#include "eh_stencil3_kernels.h"
#include "eh_transfer3_kernels.h"

namespace eh {

template <class T>
void launch_sweep(hipStream_t stream, int dim, const GArgs<T>& a, int l, int mode, const dim3& blk, int nrhs) {
    const bool P = a.kind[0] == dim;
    if (l == 0 && dim == 3 && (mode == 1 || mode == 2 || mode == 5)) {
        // the plane-staged kernel: FTX x FTY tiles of two planes, 256 threads
        int gx = 1, gy = 1;
        for (int s = 0; s < a.ns; ++s) {
            gx = std::max(gx, (a.d[s].g[0] + FTX - 1) / FTX);
            gy = std::max(gy, (a.d[s].g[1] + FTY - 1) / FTY);
        }
        const int nzb = (a.maxg2 + 1) / 2;   // plane pairs
        const int rch = rhs_chunk(gx * gy * nzb, a.ns, nrhs);
        const int nch = (std::max(nrhs, 1) + rch - 1) / rch;
        const dim3 g((unsigned)gx, (unsigned)gy, (unsigned)(nzb * a.ns * nch));
#define EH_G3(KIND)                                                                                              \
    if (mode == 1) hipLaunchKernelGGL((k_gfine3_lds<T, KIND, 1>), g, dim3(256), 0, stream, a, nrhs, rch);          \
    else if (mode == 2) hipLaunchKernelGGL((k_gfine3_lds<T, KIND, 2>), g, dim3(256), 0, stream, a, nrhs, rch);     \
    else hipLaunchKernelGGL((k_gfine3_lds<T, KIND, 5>), g, dim3(256), 0, stream, a, nrhs, rch);
        if (P && a.tilde) { EH_G3(2) } else if (P) { EH_G3(1) } else { EH_G3(0) }
#undef EH_G3
        return;
    }
    if (l > 0 && dim == 3 && a.mixed && (mode == 1 || mode == 2 || mode == 5)) {
        // the plane-staged 27-point kernel: STX x STY tiles of 256 threads
        int rch = 1;
        const dim3 g = ggrid(a, dim3(STX, STY, 1), nrhs, rch);
        if (mode == 1) hipLaunchKernelGGL((k_gstencil3_lds<T, 1>), g, dim3(256), 0, stream, a, nrhs, rch);
        else if (mode == 2) hipLaunchKernelGGL((k_gstencil3_lds<T, 2>), g, dim3(256), 0, stream, a, nrhs, rch);
        else hipLaunchKernelGGL((k_gstencil3_lds<T, 5>), g, dim3(256), 0, stream, a, nrhs, rch);
        return;
    }
    int rch = 1;
    const dim3 g = ggrid(a, blk, nrhs, rch);
    if (l == 0) {
#define EH_GF(KIND, DIM, MODE) hipLaunchKernelGGL((k_gfine<T, KIND, DIM, MODE>), g, blk, 0, stream, a, nrhs, rch)
#define EH_GF_M(KIND, DIM)                      \
    switch (mode) {                             \
        case 0: EH_GF(KIND, DIM, 0); break;     \
        case 1: EH_GF(KIND, DIM, 1); break;     \
        case 2: EH_GF(KIND, DIM, 2); break;     \
        case 3: EH_GF(KIND, DIM, 3); break;     \
        case 4: EH_GF(KIND, DIM, 4); break;     \
        default: EH_GF(KIND, DIM, 5); break;    \
    }
        if (dim == 2) {
            if (P && a.tilde) { EH_GF_M(2, 2) } else if (P) { EH_GF_M(1, 2) } else { EH_GF_M(0, 2) }
        } else {
            if (P && a.tilde) { EH_GF_M(2, 3) } else if (P) { EH_GF_M(1, 3) } else { EH_GF_M(0, 3) }
        }
#undef EH_GF_M
#undef EH_GF
    } else {
#define EH_GS(DIM, MODE)                                                                   \
    if (a.mixed) hipLaunchKernelGGL((k_gstencil<T, DIM, MODE, true>), g, blk, 0, stream, a, nrhs, rch);  \
    else hipLaunchKernelGGL((k_gstencil<T, DIM, MODE, false>), g, blk, 0, stream, a, nrhs, rch)
#define EH_GS_M(DIM)                        \
    switch (mode) {                         \
        case 0: EH_GS(DIM, 0); break;       \
        case 1: EH_GS(DIM, 1); break;       \
        case 2: EH_GS(DIM, 2); break;       \
        case 3: EH_GS(DIM, 3); break;       \
        case 4: EH_GS(DIM, 4); break;       \
        default: EH_GS(DIM, 5); break;      \
    }
        if (dim == 2) { EH_GS_M(2) } else { EH_GS_M(3) }
#undef EH_GS_M
#undef EH_GS
    }
}

template <class T>
void launch_transfer(hipStream_t stream, int dim, const GArgs<T>& t, const dim3& blk, bool restrict_to_coarse, int nrhs) {
    int rch = 1;
    if (dim == 3) {
        // the staged 3D transfers: tiles of 256 threads
        if (restrict_to_coarse) {
            const dim3 g = ggrid(t, dim3(RTX, RTY, 1), nrhs, rch);
            if (t.mixed) hipLaunchKernelGGL((k_grestrict3_lds<T, true>), g, dim3(256), 0, stream, t, nrhs, rch);
            else hipLaunchKernelGGL((k_grestrict3_lds<T, false>), g, dim3(256), 0, stream, t, nrhs, rch);
        } else {
            const dim3 g = ggrid(t, dim3(PTX, PTY, 1), nrhs, rch);
            hipLaunchKernelGGL((k_gprolong3_lds<T>), g, dim3(256), 0, stream, t, nrhs, rch);
        }
        return;
    }
    const dim3 g = ggrid(t, blk, nrhs, rch);
    if (restrict_to_coarse) {
        if (dim == 2) hipLaunchKernelGGL((k_gtransfer<T, 2, true>), g, blk, 0, stream, t, nrhs, rch);
        else hipLaunchKernelGGL((k_gtransfer<T, 3, true>), g, blk, 0, stream, t, nrhs, rch);
    } else {
        if (dim == 2) hipLaunchKernelGGL((k_gtransfer<T, 2, false>), g, blk, 0, stream, t, nrhs, rch);
        else hipLaunchKernelGGL((k_gtransfer<T, 3, false>), g, blk, 0, stream, t, nrhs, rch);
    }
}

template void launch_sweep<EH_T>(hipStream_t, int, const GArgs<EH_T>&, int, int, const dim3&, int);
template void launch_transfer<EH_T>(hipStream_t, int, const GArgs<EH_T>&, const dim3&, bool, int);

}  // namespace eh
