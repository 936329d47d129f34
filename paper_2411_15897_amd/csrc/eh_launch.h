// Launches of the multigrid kernels: the fused legs (eh_fused.hip) and the
// per-sweep kernels and transfers (eh_sweep.hip).  Their many instantiations
// are most of the library's compile time, so these files are compiled once
// per precision (and leg), next to the host driver.  The caller checks
// hipGetLastError.
#pragma once

#include <algorithm>

#include "eh_common.h"
#include "eh_group_kernels.h"

namespace eh {

// Tile configurations (x extent, y extent, threads): the down leg's tile
// is in coarse points, the up leg's in fine points.  Large tiles amortise
// the halo on big levels; small ones give the few-thousand-point levels
// enough workgroups and keep every phase to about one round of loads per
// thread.  The autotuner picks one per level and block group.  The phase
// loops stay rolled: on small levels each compute unit runs a workgroup or
// two, so the kernel's instruction fetch from a cold cache is part of its
// latency, and unrolled code costs more there than it gains on big levels.
struct FCfg {
    int x, y, threads;
};
constexpr FCfg kFDown[] = {{32, 8, 256}, {32, 8, 512}, {16, 8, 256}, {7, 3, 128}};
constexpr FCfg kFUp[] = {{64, 16, 1024}, {64, 8, 512}, {32, 8, 256}, {16, 8, 128}};
constexpr int kFCfgs = 4;

// Right-hand sides per workgroup of a multigrid launch (fused leg or
// per-sweep kernel) with `tiles` workgroups per slot: the whole batch while the tiles alone give
// kSplitWgs workgroups or more (the operator in registers then serves every right-hand side);
// below that the batch is split into chunks, up to one right-hand side per
// workgroup, so that a small level runs its right-hand sides side by side
// instead of one after the other.
#ifndef EH_SPLIT_WGS
#define EH_SPLIT_WGS 4096
#endif
constexpr int kSplitWgs = EH_SPLIT_WGS;
inline int rhs_chunk(int tiles, int ns, int nrhs) {
    const int64_t wgs = (int64_t)tiles * ns;
    if (nrhs <= 1 || wgs >= kSplitWgs) return (nrhs > 1 ? nrhs : 1);
    const int nch = (int)std::min<int64_t>(nrhs, (kSplitWgs + wgs - 1) / wgs);
    return (nrhs + nch - 1) / nch;
}

// Grid of a per-sweep kernel over the slots of a and the chunks of the
// batch; rch receives the right-hand sides per workgroup.
template <class T>
dim3 ggrid(const GArgs<T>& a, const dim3& blk, int nrhs, int& rch) {
    int gx = 1, gy = 1;
    for (int s = 0; s < a.ns; ++s) {
        gx = std::max(gx, (int)((a.d[s].g[0] + blk.x - 1) / blk.x));
        gy = std::max(gy, (int)((a.d[s].g[1] + blk.y - 1) / blk.y));
    }
    rch = rhs_chunk(gx * gy * a.maxg2, a.ns, nrhs);
    const int nch = (std::max(nrhs, 1) + rch - 1) / rch;
    return dim3((unsigned)gx, (unsigned)gy, (unsigned)(a.maxg2 * a.ns * nch));
}

// Fused down leg on level l with tile configuration cfg: a.d / a.dc = levels
// l / l+1, a.f = f_l, a.out = f_{l+1}.  With cpl (l = 0, shear blocks) the
// launch forms and stores f_0 itself.
template <class T>
void launch_fdown(hipStream_t stream, const GArgs<T>& a, int l, int cfg, int nrhs, const CplArgs<T>* cpl = nullptr);

// Fused up leg on level l with nu_post (1 or 2) sweeps: a.f = f_l, a.u =
// e_{l+1}, a.out = e_l.
template <class T>
void launch_fup(hipStream_t stream, int nu_post, const GArgs<T>& a, int l, int cfg, int nrhs);

// One sweep-type launch (modes of k_gfine / k_gstencil) on level l with
// workgroups of shape blk where the kernel leaves the choice.
template <class T>
void launch_sweep(hipStream_t stream, int dim, const GArgs<T>& a, int l, int mode, const dim3& blk, int nrhs);

// Restriction (grid = coarse level) or prolongation with correction (grid
// = fine level) for the slots of t.
template <class T>
void launch_transfer(hipStream_t stream, int dim, const GArgs<T>& t, const dim3& blk, bool restrict_to_coarse, int nrhs);

}  // namespace eh
