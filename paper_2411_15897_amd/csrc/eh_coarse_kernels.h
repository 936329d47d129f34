// Direct solve of the coarsest multigrid level by block elimination (FP64).
//
// The paper solves the coarsest grid of every block directly (Section
// 4.4.1, "Multigrid setup").  A coarse stencil of half width w_a along axis
// a couples only points whose index along a differs by at most w_a, so
// cutting the grid into groups of w_a consecutive planes (lines in 2D)
// normal to a makes the operator block tridiagonal:
//     L_I x_{I-1} + D_I x_I + U_I x_{I+1} = f_I.
// Groups are eliminated in levels.  A level removes a set of groups no two
// of which are neighbours in the current chain; the groups left form a
// block-tridiagonal chain again, with
//     G_l = -L_K S_e1^-1, G_r = -U_K S_e2^-1         (K kept, e1 / e2 removed beside it)
//     D_K += G_l U_e1 + G_r L_e2,  L_K <- G_l L_e1,  U_K <- G_r U_e2
//     f_K += G_l f_e1 + G_r f_e2
// and, going back,
//     x_e = S_e^-1 f_e - S_e^-1 L_e x_l - S_e^-1 U_e x_r.
// Removing every other group (cyclic reduction) halves the chain per level;
// the last few groups are inverted as one dense matrix.  Stored per removed
// group: [S_e^-1 | -S_e^-1 L_e | -S_e^-1 U_e], per kept group beside one:
// [G_l | G_r], row-major; five matrices per group in all.  A solve is one
// launch per level down, one for the dense rest and one per level back up.
//
// On the first level L_e, U_e, L_K and U_K are still the stencil's few entries
// per row, so where its matrices are large the products with them run from
// lists of these entries and only S_e^-1 is stored:
//     v_e = S_e^-1 f_e,  f_K -= L_K v_e1 + U_K v_e2;
//     x_e = S_e^-1 (f_e - L_e x_l - U_e x_r),
// two matrices read per removed group instead of five for two more launches.
//
// Why levels: a sweep over the groups one after the other needs two launches
// per group, each a few microseconds of dependent latency however small its
// matrix; here the launches number 2 log2(groups), and a level's groups run
// side by side.  The price is 5 b^2 matrix entries per group instead of 3.
// Inverses by blocked Gauss-Jordan (32 x 32 pivot blocks, partial pivoting
// inside each pivot block).
#pragma once

#include "eh_common.h"

namespace eh {

// Partition of one block's coarsest grid into groups of planes normal to
// axis `ax`.  Local index m of group I: plane t = I*gsz + m / P, in-plane
// index q = m % P = c[a1] + g[a1] * c[a2].
struct BTPart {
    Dims d;
    Widths w;
    int ax, a1, a2;
    int gsz;        // planes per group (= w[ax])
    int nb;         // groups
    int P;          // points per plane
    __host__ __device__ int planes(int I) const { return min(gsz, d.g[ax] - I * gsz); }
    __host__ __device__ int bsize(int I) const { return (I < 0 || I >= nb) ? 0 : planes(I) * P; }
    __host__ __device__ void coords(int I, int m, int c[3]) const {
        const int t = I * gsz + m / P, q = m % P;
        c[ax] = t;
        c[a1] = q % d.g[a1];
        c[a2] = q / d.g[a1];
    }
    __host__ __device__ int64_t point(const int c[3]) const {
        return ((int64_t)c[2] * d.g[1] + c[1]) * d.g[0] + c[0];
    }
    __host__ __device__ int group(const int c[3]) const { return c[ax] / gsz; }
    __host__ __device__ int local(const int c[3]) const {
        return (c[ax] - (c[ax] / gsz) * gsz) * P + c[a1] + d.g[a1] * c[a2];
    }
    __host__ __device__ bool inside(const int c[3]) const {
        return c[0] >= 0 && c[0] < d.g[0] && c[1] >= 0 && c[1] < d.g[1] && c[2] >= 0 && c[2] < d.g[2];
    }
    __host__ __device__ int offset_index(int ox, int oy, int oz) const {
        return ((oz + w.w[2]) * (2 * w.w[1] + 1) + (oy + w.w[1])) * (2 * w.w[0] + 1) + (ox + w.w[0]);
    }
};

// ---------------------------------------------------------------------------
// setup

// Dense block (I, I + dir) of the operator, padded to bp x bp (the diagonal
// block with the identity, the couplings with 0).  One matrix per blockIdx.z.
struct BTBlock {
    c128* M;
    int I, dir;
};
__global__ void __launch_bounds__(256)
k_bt_couple_dense(BTPart pt, const c128* __restrict__ st, const BTBlock* __restrict__ blocks, int bp) {
    const BTBlock bl = blocks[blockIdx.z];
    const int col = blockIdx.x * blockDim.x + threadIdx.x;
    const int row = blockIdx.y;
    if (col >= bp) return;
    c128* out = bl.M + (int64_t)row * bp + col;
    c128 v = mk(bl.dir == 0 && row == col ? 1.0 : 0.0, 0.0);
    if (row < pt.bsize(bl.I) && col < pt.bsize(bl.I + bl.dir)) {
        int cr[3], cc[3];
        pt.coords(bl.I, row, cr);
        pt.coords(bl.I + bl.dir, col, cc);
        const int ox = cc[0] - cr[0], oy = cc[1] - cr[1], oz = cc[2] - cr[2];
        v = mk(0.0, 0.0);
        if (abs(ox) <= pt.w.w[0] && abs(oy) <= pt.w.w[1] && abs(oz) <= pt.w.w[2])
            v = st[(int64_t)pt.offset_index(ox, oy, oz) * pt.d.np() + pt.point(cr)];
    }
    *out = v;
}

// The couplings of every row to its neighbouring groups as entry-major lists
// in elimination order (perm: elimination order -> point, inv the other
// way): coefficient and the neighbour's place, rows with fewer entries
// filled with zero coefficients at a place on the other side of the coupling
// (removed entries are 0 .. n0 - 1, kept ones follow), which k_bt_sparse finds
// written: its own side still holds what an earlier solve left, or nothing.
__global__ void __launch_bounds__(256)
k_bt_couple_list(BTPart pt, const c128* __restrict__ st, const int* __restrict__ perm, const int* __restrict__ inv,
                 int ne, int n0, c128* __restrict__ k, int* __restrict__ at) {
    const int N = (int)pt.d.np();
    const int q = blockIdx.x * 256 + threadIdx.x;
    if (q >= N) return;
    const int p = perm[q];
    const int c[3] = {p % pt.d.g[0], (p / pt.d.g[0]) % pt.d.g[1], p / (pt.d.g[0] * pt.d.g[1])};
    const int g = pt.group(c);
    int e = 0;
    for (int oz = -pt.w.w[2]; oz <= pt.w.w[2]; ++oz)
    for (int oy = -pt.w.w[1]; oy <= pt.w.w[1]; ++oy)
    for (int ox = -pt.w.w[0]; ox <= pt.w.w[0]; ++ox) {
        const int n[3] = {c[0] + ox, c[1] + oy, c[2] + oz};
        if (!pt.inside(n) || pt.group(n) == g) continue;
        k[(int64_t)e * N + q] = st[(int64_t)pt.offset_index(ox, oy, oz) * N + p];
        at[(int64_t)e * N + q] = inv[pt.point(n)];
        ++e;
    }
    for (; e < ne; ++e) {
        k[(int64_t)e * N + q] = mk(0.0, 0.0);
        at[(int64_t)e * N + q] = q < n0 ? n0 : 0;
    }
}

constexpr int GJB = 32;   // pivot block of the blocked Gauss-Jordan inversion

// Matrices inverted side by side, one per blockIdx.z: bp x bp, bp a multiple
// of GJB (padded with the identity).  Matrices of a launch may differ in
// bp; those with fewer pivot blocks drop out.
struct GJMat {
    c128* M;
    int bp;
};

// Pivot block K of M (bp x bp, in place): A_KK <- A_KK^-1 by Gauss-Jordan
// with partial pivoting on [A_KK | I].  A zero pivot sets *bad.
//
// The 32 steps are a serial chain of one workgroup, so each keeps its
// matrix in registers: thread t owns column t % 64 and the rows t / 64 + 4 q
// and only the pivot column and two rows pass through LDS, in two buffers,
// two barriers per step.  Every wavefront finds the pivot by itself.
__global__ void __launch_bounds__(256)
k_gj_diag(const GJMat* __restrict__ mats, int K, int* __restrict__ bad) {
    __shared__ c128 col[2][GJB], rowk[2][2 * GJB], rowp[2][2 * GJB];
    const GJMat gm = mats[blockIdx.z];
    if (K * GJB >= gm.bp) return;
    c128* M = gm.M + (int64_t)K * GJB * gm.bp + K * GJB;
    const int j = threadIdx.x & 63, r0 = threadIdx.x >> 6, lane = j;
    c128 A[8];
#pragma unroll
    for (int q = 0; q < 8; ++q) {
        const int i = r0 + 4 * q;
        A[q] = j < GJB ? M[(int64_t)i * gm.bp + j] : mk(j - GJB == i ? 1.0 : 0.0, 0.0);
    }
    for (int k = 0; k < GJB; ++k) {
        const int s = k & 1;
        if (j == k) {
#pragma unroll
            for (int q = 0; q < 8; ++q) col[s][r0 + 4 * q] = A[q];
        }
        __syncthreads();
        // pivot row: the largest |column entry| from row k on, the lowest on ties
        double best = -1.0;
        int p = k;
        if (lane < GJB && lane >= k) { best = cabs2(col[s][lane]); p = lane; }
        for (int off = 16; off > 0; off >>= 1) {
            const double ob = __shfl_xor(best, off, 64);
            const int op = __shfl_xor(p, off, 64);
            if (ob > best || (ob == best && op < p)) { best = ob; p = op; }
        }
        best = __shfl(best, 0, 64);
        p = __shfl(p, 0, 64);
        if (!(best > 0.0)) {             // uniform: every wavefront found the same pivot
            *bad = 1;
            return;
        }
        if ((p & 3) == r0 || (k & 3) == r0) {
#pragma unroll
            for (int q = 0; q < 8; ++q) {
                if (r0 + 4 * q == p) rowp[s][j] = A[q];
                if (r0 + 4 * q == k) rowk[s][j] = A[q];
            }
        }
        __syncthreads();
        const c128 pr = cdiv(mk(1.0, 0.0), col[s][p]) * rowp[s][j];   // the new row k
        const c128 rk = rowk[s][j], ck = col[s][k];
#pragma unroll
        for (int q = 0; q < 8; ++q) {
            const int i = r0 + 4 * q;
            if (i == k) A[q] = pr;
            else if (i == p) A[q] = rk - ck * pr;
            else A[q] = A[q] - col[s][i] * pr;
        }
    }
    if (j >= GJB) {
#pragma unroll
        for (int q = 0; q < 8; ++q) M[(int64_t)(r0 + 4 * q) * gm.bp + j - GJB] = A[q];
    }
}

// Row panel of pivot block K: A_Kj <- A_KK^-1 A_Kj for every column j
// outside the block (64 columns per workgroup).
__global__ void __launch_bounds__(256)
k_gj_rowpanel(const GJMat* __restrict__ mats, int K) {
    c128* __restrict__ M = mats[blockIdx.z].M;
    const int bp = mats[blockIdx.z].bp;
    if (K * GJB >= bp || (int)blockIdx.x * 64 >= bp) return;
    __shared__ c128 Dv[GJB][GJB];
    __shared__ c128 Pn[GJB][64];
    const int tid = threadIdx.x;
    const int k0 = K * GJB, j0 = blockIdx.x * 64;
    for (int e = tid; e < GJB * GJB; e += 256) Dv[e / GJB][e % GJB] = M[(int64_t)(k0 + e / GJB) * bp + k0 + e % GJB];
    for (int e = tid; e < GJB * 64; e += 256) {
        const int i = e / 64, j = j0 + e % 64;
        Pn[i][e % 64] = j < bp ? M[(int64_t)(k0 + i) * bp + j] : mk(0.0, 0.0);
    }
    __syncthreads();
    for (int e = tid; e < GJB * 64; e += 256) {
        const int i = e / 64, jl = e % 64, j = j0 + jl;
        if (j >= bp || (j >= k0 && j < k0 + GJB)) continue;
        c128 acc = mk(0.0, 0.0);
#pragma unroll 8
        for (int m = 0; m < GJB; ++m) acc = acc + Dv[i][m] * Pn[m][jl];
        M[(int64_t)(k0 + i) * bp + j] = acc;
    }
}

// Rank-32 update: A_ij <- A_ij - A_iK A_Kj for i, j outside block K (A_Kj
// already multiplied by A_KK^-1).  64 x 64 output tile per workgroup, each
// thread 4 x 4 entries 16 apart.
__global__ void __launch_bounds__(256)
k_gj_update(const GJMat* __restrict__ mats, int K) {
    c128* __restrict__ M = mats[blockIdx.z].M;
    const int bp = mats[blockIdx.z].bp;
    if (K * GJB >= bp || (int)blockIdx.x * 64 >= bp || (int)blockIdx.y * 64 >= bp) return;
    __shared__ c128 Ac[64][GJB + 1];
    __shared__ c128 Br[GJB][64];
    const int tid = threadIdx.x;
    const int k0 = K * GJB, i0 = blockIdx.y * 64, j0 = blockIdx.x * 64;
    for (int e = tid; e < 64 * GJB; e += 256) {
        const int i = e / GJB, m = e % GJB;
        Ac[i][m] = i0 + i < bp ? M[(int64_t)(i0 + i) * bp + k0 + m] : mk(0.0, 0.0);
    }
    for (int e = tid; e < GJB * 64; e += 256) {
        const int m = e / 64, j = e % 64;
        Br[m][j] = j0 + j < bp ? M[(int64_t)(k0 + m) * bp + j0 + j] : mk(0.0, 0.0);
    }
    __syncthreads();
    const int tx = tid % 16, ty = tid / 16;
    double ar[4][4], ai[4][4];
#pragma unroll
    for (int a = 0; a < 4; ++a)
#pragma unroll
        for (int b = 0; b < 4; ++b) { ar[a][b] = 0.0; ai[a][b] = 0.0; }
    for (int m = 0; m < GJB; ++m) {
        c128 x[4], y[4];
#pragma unroll
        for (int a = 0; a < 4; ++a) x[a] = Ac[ty + 16 * a][m];
#pragma unroll
        for (int b = 0; b < 4; ++b) y[b] = Br[m][tx + 16 * b];
#pragma unroll
        for (int a = 0; a < 4; ++a)
#pragma unroll
            for (int b = 0; b < 4; ++b) {
                ar[a][b] += x[a].re * y[b].re - x[a].im * y[b].im;
                ai[a][b] += x[a].re * y[b].im + x[a].im * y[b].re;
            }
    }
#pragma unroll
    for (int a = 0; a < 4; ++a) {
        const int i = i0 + ty + 16 * a;
        if (i >= bp || (i >= k0 && i < k0 + GJB)) continue;
#pragma unroll
        for (int b = 0; b < 4; ++b) {
            const int j = j0 + tx + 16 * b;
            if (j >= bp || (j >= k0 && j < k0 + GJB)) continue;
            c128* p = M + (int64_t)i * bp + j;
            *p = *p - mk(ar[a][b], ai[a][b]);
        }
    }
}

// Column panel of pivot block K: A_iK <- -A_iK A_KK^-1 for every row i
// outside the block (64 rows per workgroup).
__global__ void __launch_bounds__(256)
k_gj_colpanel(const GJMat* __restrict__ mats, int K) {
    c128* __restrict__ M = mats[blockIdx.z].M;
    const int bp = mats[blockIdx.z].bp;
    if (K * GJB >= bp || (int)blockIdx.x * 64 >= bp) return;
    __shared__ c128 Dv[GJB][GJB];
    __shared__ c128 Pn[64][GJB + 1];
    const int tid = threadIdx.x;
    const int k0 = K * GJB, i0 = blockIdx.x * 64;
    for (int e = tid; e < GJB * GJB; e += 256) Dv[e / GJB][e % GJB] = M[(int64_t)(k0 + e / GJB) * bp + k0 + e % GJB];
    for (int e = tid; e < 64 * GJB; e += 256) {
        const int i = e / GJB, m = e % GJB;
        Pn[i][m] = i0 + i < bp ? M[(int64_t)(i0 + i) * bp + k0 + m] : mk(0.0, 0.0);
    }
    __syncthreads();
    for (int e = tid; e < 64 * GJB; e += 256) {
        const int il = e / GJB, k = e % GJB, i = i0 + il;
        if (i >= bp || (i >= k0 && i < k0 + GJB)) continue;
        c128 acc = mk(0.0, 0.0);
#pragma unroll 8
        for (int m = 0; m < GJB; ++m) acc = acc + Pn[il][m] * Dv[m][k];
        M[(int64_t)i * bp + k0 + k] = mk(-acc.re, -acc.im);
    }
}

// C = sgn * A B (+ C with acc), bp x bp matrices, one product per
// blockIdx.z: the dense products of a level of the elimination.  A 64 x 64
// tile per workgroup, 16 columns of A and rows of B staged in LDS per step,
// on the FP64 matrix unit (v_mfma_f64_16x16x4: lane l holds A[l % 16][l / 16]
// and B[l / 16][l % 16], result register i holds D[l / 16 + 4 i][l % 16]); a
// complex product is four real ones on split re / im planes.  The planes'
// pitch keeps a wavefront's four rows (or its 16 rows) on different banks.
struct GJProd {
    const c128* A;
    const c128* B;
    c128* C;
    double sgn;
    int acc;
};
typedef double gj_f64x4 __attribute__((ext_vector_type(4)));
constexpr int GJP_KC = 16;
__global__ void __launch_bounds__(256)
k_gj_product(const GJProd* __restrict__ prods, int bp) {
    __shared__ double Ar[64][GJP_KC + 1], Ai[64][GJP_KC + 1];
    __shared__ double Br[GJP_KC][64 + 4], Bi[GJP_KC][64 + 4];
    const GJProd pd = prods[blockIdx.z];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int i0 = blockIdx.y * 64, j0 = blockIdx.x * 64;
    const int wi = (wave >> 1) * 32, wj = (wave & 1) * 32;
    const int lr = lane & 15, lk = lane >> 4;
    gj_f64x4 cr[2][2], ci[2][2];
#pragma unroll
    for (int a = 0; a < 2; ++a)
#pragma unroll
        for (int b = 0; b < 2; ++b) {
            cr[a][b] = gj_f64x4{0.0, 0.0, 0.0, 0.0};
            ci[a][b] = gj_f64x4{0.0, 0.0, 0.0, 0.0};
        }
    for (int k0 = 0; k0 < bp; k0 += GJP_KC) {   // bp is a multiple of 32
        c128 va[4], vb[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const int e = tid + 256 * u;
            const int ia = i0 + e / GJP_KC, jb = j0 + e % 64;
            va[u] = ia < bp ? pd.A[(int64_t)ia * bp + k0 + e % GJP_KC] : mk(0.0, 0.0);
            vb[u] = jb < bp ? pd.B[(int64_t)(k0 + e / 64) * bp + jb] : mk(0.0, 0.0);
        }
        __syncthreads();
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const int e = tid + 256 * u;
            Ar[e / GJP_KC][e % GJP_KC] = va[u].re;
            Ai[e / GJP_KC][e % GJP_KC] = va[u].im;
            Br[e / 64][e % 64] = vb[u].re;
            Bi[e / 64][e % 64] = vb[u].im;
        }
        __syncthreads();
#pragma unroll
        for (int kk = 0; kk < GJP_KC; kk += 4) {
            double xr[2], xi[2], yr[2], yi[2];
#pragma unroll
            for (int a = 0; a < 2; ++a) {
                xr[a] = Ar[wi + 16 * a + lr][kk + lk];
                xi[a] = Ai[wi + 16 * a + lr][kk + lk];
                yr[a] = Br[kk + lk][wj + 16 * a + lr];
                yi[a] = Bi[kk + lk][wj + 16 * a + lr];
            }
#pragma unroll
            for (int a = 0; a < 2; ++a)
#pragma unroll
                for (int b = 0; b < 2; ++b) {
                    cr[a][b] = __builtin_amdgcn_mfma_f64_16x16x4f64(xr[a], yr[b], cr[a][b], 0, 0, 0);
                    ci[a][b] = __builtin_amdgcn_mfma_f64_16x16x4f64(xr[a], yi[b], ci[a][b], 0, 0, 0);
                    cr[a][b] = __builtin_amdgcn_mfma_f64_16x16x4f64(-xi[a], yi[b], cr[a][b], 0, 0, 0);
                    ci[a][b] = __builtin_amdgcn_mfma_f64_16x16x4f64(xi[a], yr[b], ci[a][b], 0, 0, 0);
                }
        }
    }
#pragma unroll
    for (int a = 0; a < 2; ++a)
#pragma unroll
        for (int b = 0; b < 2; ++b)
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const int i = i0 + wi + 16 * a + lk + 4 * q, j = j0 + wj + 16 * b + lr;
                if (i >= bp || j >= bp) continue;
                c128* p = pd.C + (int64_t)i * bp + j;
                const c128 v = mk(pd.sgn * cr[a][b][q], pd.sgn * ci[a][b][q]);
                *p = pd.acc ? *p + v : v;
            }
}

// Copy the leading rows x cols of src (row stride lds) to dst (row stride
// ldd); one copy per blockIdx.z.
struct BTCopy {
    const c128* src;
    c128* dst;
    int rows, cols, lds, ldd;
};
__global__ void __launch_bounds__(256)
k_bt_store_inv(const BTCopy* __restrict__ copies) {
    const BTCopy cp = copies[blockIdx.z];
    const int col = blockIdx.x * blockDim.x + threadIdx.x;
    const int row = blockIdx.y;
    if (col < cp.cols && row < cp.rows) cp.dst[(int64_t)row * cp.ldd + col] = cp.src[(int64_t)row * cp.lds + col];
}

// Identity, the start of a padded dense matrix.
__global__ void __launch_bounds__(256)
k_gj_identity(c128* __restrict__ M, int bp) {
    const int col = blockIdx.x * blockDim.x + threadIdx.x;
    const int row = blockIdx.y;
    if (col < bp) M[(int64_t)row * bp + col] = mk(row == col ? 1.0 : 0.0, 0.0);
}

// y = X x with an FP64 stencil (the setup's accuracy check).
__global__ void __launch_bounds__(256)
k_stencil_f64(Dims d, Widths w, const c128* __restrict__ st, const c128* __restrict__ x, c128* __restrict__ y) {
    const int64_t N = d.np();
    const int64_t q = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (q >= N) return;
    const int i = (int)(q % d.g[0]);
    const int j = (int)((q / d.g[0]) % d.g[1]);
    const int k = (int)(q / ((int64_t)d.g[0] * d.g[1]));
    const int NX = 2 * w.w[0] + 1, NY = 2 * w.w[1] + 1;
    c128 acc = mk(0.0, 0.0);
    for (int oz = -w.w[2]; oz <= w.w[2]; ++oz)
    for (int oy = -w.w[1]; oy <= w.w[1]; ++oy)
    for (int ox = -w.w[0]; ox <= w.w[0]; ++ox) {
        const int a = i + ox, b = j + oy, c = k + oz;
        if (a < 0 || a >= d.g[0] || b < 0 || b >= d.g[1] || c < 0 || c >= d.g[2]) continue;
        const int o = ((oz + w.w[2]) * NY + (oy + w.w[1])) * NX + (ox + w.w[0]);
        acc = acc + st[(int64_t)o * N + q] * x[((int64_t)c * d.g[1] + b) * d.g[0] + a];
    }
    y[q] = acc;
}

// ---------------------------------------------------------------------------
// solve

constexpr int BT_MAXS = 4;
constexpr int BT_RW = 4;                // rows per workgroup, one per wavefront

// The rows of one group in one launch: a rows x (n[0] + n[1] + n[2]) matrix,
// row-major at mats + mat, times entries of up to three vectors.  Vectors
// are in elimination order; off and out index them.
struct BTTask {
    int64_t mat;
    int rows;
    int n[3], off[3];
    int out;
    int add;        // down: the result is added to the right-hand side's entry
};

// One launch over up to BT_MAXS blocks.  Per slot: its tasks in this launch,
// the permutation from elimination order to the level's points, the right-
// hand side (the level's f on the first level of the elimination, y after),
// the eliminated right-hand side y and the solution x (FP64, elimination
// order, N entries per right-hand side), and the level's vector e.
template <class T>
struct BTRun {
    int ns;
    int nrhs;
    const BTTask* tasks[BT_MAXS];
    int ntasks[BT_MAXS];
    int first[BT_MAXS];
    const c128* mats[BT_MAXS];
    const int* perm[BT_MAXS];
    int N[BT_MAXS];
    c128* y[BT_MAXS];
    c128* x[BT_MAXS];
    const cplx<T>* f[BT_MAXS];
    int64_t vf[BT_MAXS];
    cplx<T>* e[BT_MAXS];
    int64_t ve[BT_MAXS];
};

// Down (BACK false): y_K = f_K + G_l f_e1 + G_r f_e2 (a kept group without
// removed neighbours has no columns: y_K = f_K; without add, y_e = S_e^-1
// f_e).  Up (BACK true): x_e =
// S_e^-1 f_e - S_e^-1 L_e x_l - S_e^-1 U_e x_r, written to x and, in the
// level's layout and precision, to e; also the dense rest (one vector).
//
// Bound by the matrix entries, each read once per chunk of right-hand sides:
// one row per wavefront, four per workgroup, whose vector chunk (every
// right-hand side, FP64) is staged in LDS while the row's loads are in
// flight.  Each lane sums its columns in a fixed order, a butterfly adds the
// lanes; a right-hand side's arithmetic does not depend on the others.
// Columns per lane and chunk: the staged chunk holds 40 KB at most.
// Grid (row blocks of the largest group, tasks x slots (slot fastest),
// chunks of RB right-hand sides).
template <int RB>
constexpr int bt_na() { return RB >= 8 ? 5 : 10; }

template <class T, int RB, bool BACK>
__global__ void __launch_bounds__(256)
k_bt_rows(BTRun<T> a) {
    constexpr int NA = bt_na<RB>(), CW = 64 * NA;
    __shared__ c128 xs[RB * CW];
    const int s = blockIdx.y % a.ns, t = blockIdx.y / a.ns;
    if (t >= a.ntasks[s]) return;
    const BTTask tk = a.tasks[s][t];
    const int row0 = blockIdx.x * BT_RW;
    if (row0 >= tk.rows) return;
    const int row = row0 + (threadIdx.x >> 6), lane = threadIdx.x & 63;
    const int r0 = blockIdx.z * RB;
    const int cnt = min(RB, a.nrhs - r0);
    const int N = a.N[s];
    const bool first = a.first[s] != 0;
    const int* __restrict__ perm = a.perm[s];
    const cplx<T>* f = a.f[s] + (int64_t)r0 * a.vf[s];
    c128* y = a.y[s] + (int64_t)r0 * N;
    c128* x = a.x[s] + (int64_t)r0 * N;
    const int64_t vf = a.vf[s];
    const int n0 = tk.n[0], n01 = n0 + tk.n[1], nc = n01 + tk.n[2];
    const c128* A = row < tk.rows ? a.mats[s] + tk.mat + (int64_t)row * nc : nullptr;
    // this lane's result: right-hand side r0 + lane of the wavefront's row
    const bool wr = row < tk.rows && lane < cnt;
    const int po = (wr && (BACK || first)) ? perm[tk.out + row] : 0;
    c128 add = mk(0.0, 0.0);
    if (!BACK && wr && tk.add) {
        if (first) add = ccast<double>(f[lane * vf + po]);
        else add = y[(int64_t)lane * N + tk.out + row];
    }
    double ar[RB], ai[RB];
#pragma unroll
    for (int r = 0; r < RB; ++r) { ar[r] = 0.0; ai[r] = 0.0; }
    for (int c0 = 0; c0 < nc; c0 += CW) {
        const int w = min(CW, nc - c0);
        c128 mv[NA];
#pragma unroll
        for (int u = 0; u < NA; ++u) {
            const int c = lane + 64 * u;
            mv[u] = (A && c < w) ? A[c0 + c] : mk(0.0, 0.0);
        }
        if (c0 > 0) __syncthreads();          // the previous chunk is consumed
        for (int cc = threadIdx.x; cc < w; cc += 256) {
            const int c = c0 + cc;
            const int q = c < n0 ? tk.off[0] + c : (c < n01 ? tk.off[1] + c - n0 : tk.off[2] + c - n01);
            // down: every vector is the right-hand side; up: the first one
            // is, the neighbours' entries come from the solution
            const bool rhs = !BACK || c < n0;
            if (rhs && first) {
                const int pq = perm[q];
#pragma unroll
                for (int r = 0; r < RB; ++r)
                    xs[r * CW + cc] = r < cnt ? ccast<double>(f[r * vf + pq]) : mk(0.0, 0.0);
            } else {
                const c128* v = rhs ? y : x;
#pragma unroll
                for (int r = 0; r < RB; ++r) xs[r * CW + cc] = r < cnt ? v[(int64_t)r * N + q] : mk(0.0, 0.0);
            }
        }
        __syncthreads();
#pragma unroll
        for (int u = 0; u < NA; ++u) {
            const int c = lane + 64 * u;
            if (c < w) {
#pragma unroll
                for (int r = 0; r < RB; ++r) {
                    const c128 v = xs[r * CW + c];
                    ar[r] = fmat(-mv[u].im, v.im, fmat(mv[u].re, v.re, ar[r]));
                    ai[r] = fmat(mv[u].im, v.re, fmat(mv[u].re, v.im, ai[r]));
                }
            }
        }
    }
#pragma unroll
    for (int r = 0; r < RB; ++r)
        for (int off = 32; off > 0; off >>= 1) {
            ar[r] += __shfl_xor(ar[r], off, 64);
            ai[r] += __shfl_xor(ai[r], off, 64);
        }
    if (!wr) return;
    double sr = 0.0, si = 0.0;
#pragma unroll
    for (int r = 0; r < RB; ++r)
        if (lane == r) { sr = ar[r]; si = ai[r]; }
    const c128 v = mk(add.re + sr, add.im + si);
    const int64_t o = (int64_t)lane * N + tk.out + row;
    if (BACK) {
        x[o] = v;
        a.e[s][(int64_t)(r0 + lane) * a.ve[s] + po] = mk<T>(T(v.re), T(v.im));
    } else {
        y[o] = v;
    }
}

// First level's couplings: for the entries lo .. hi - 1 (elimination order)
// of groups that are all removed, or all kept,
//     y = f - (the couplings to the two neighbouring groups) v,
// v the right-hand side y of the removed groups (v_e) or the solution x of
// the kept ones.  A few thousand rows of 12 to 100 entries, so latency is all
// there is to it: coefficients and vector positions lie in entry-major
// lists (k_bt_couple_list), a row's entries are dealt to the workgroup's four
// wavefronts, six in flight each.  (From the stencil itself, with the
// neighbours' places worked out here: 13 to 20 us for 4500 rows.)
// Grid (64 entries, slots, right-hand sides).
template <class T>
struct BTSparse {
    int N[BT_MAXS], ne[BT_MAXS];             // points, entries per row
    const c128* k[BT_MAXS];                  // [entry][N]
    const int* at[BT_MAXS];                  // [entry][N]
    const int* perm[BT_MAXS];
    int lo[BT_MAXS], hi[BT_MAXS];
    const cplx<T>* f[BT_MAXS];
    int64_t vf[BT_MAXS];
    const c128* v[BT_MAXS];
    c128* y[BT_MAXS];
};
template <class T>
__global__ void __launch_bounds__(256)
k_bt_sparse(BTSparse<T> a) {
    __shared__ c128 part[4][64];
    const int s = blockIdx.y;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int q0 = a.lo[s] + blockIdx.x * 64;
    if (q0 >= a.hi[s]) return;               // uniform per workgroup
    const bool mine = q0 + lane < a.hi[s];
    const int q = mine ? q0 + lane : q0;
    const int N = a.N[s], ne = a.ne[s];
    const int64_t r = blockIdx.z;
    const c128* __restrict__ v = a.v[s] + r * N;
    const c128* __restrict__ k = a.k[s] + q;
    const int* __restrict__ at = a.at[s] + q;
    c128 fp = mk(0.0, 0.0);
    if (wave == 0) fp = ccast<double>(a.f[s][r * a.vf[s] + a.perm[s][q]]);
    c128 acc = mk(0.0, 0.0);
    constexpr int U = 6;
    for (int i0 = wave; i0 < ne; i0 += 4 * U) {
        c128 kk[U], u[U];
#pragma unroll
        for (int t = 0; t < U; ++t) {
            const int i = i0 + 4 * t < ne ? i0 + 4 * t : i0;
            kk[t] = k[(int64_t)i * N];
            u[t] = v[at[(int64_t)i * N]];
        }
#pragma unroll
        for (int t = 0; t < U; ++t) {
            if (i0 + 4 * t < ne) {
                acc.re = fmat(-kk[t].im, u[t].im, fmat(kk[t].re, u[t].re, acc.re));
                acc.im = fmat(kk[t].im, u[t].re, fmat(kk[t].re, u[t].im, acc.im));
            }
        }
    }
    part[wave][lane] = acc;
    __syncthreads();
    if (wave != 0 || !mine) return;
    const c128 s0 = part[0][lane] + part[1][lane], s1 = part[2][lane] + part[3][lane];
    a.y[s][r * N + q] = fp - (s0 + s1);
}

}  // namespace eh
