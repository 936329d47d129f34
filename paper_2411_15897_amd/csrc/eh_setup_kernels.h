// Setup kernels (FP64, run once per context):
//  k_galerkin_medium / _shear / _pressure: the medium's cell arrays and the
//                   fine-level operators, what the Galerkin products start
//                   from, one cell or face per thread;
//  k_galerkin       coarse stencil of X_H = R X_h P (eq. galerkin) in stencil
//                   form, one thread per coarse point;
//  k_dense_from_stencil / Gauss-Jordan kernels: explicit inverse of the
//                   coarsest operator with partial pivoting, applied later
//                   as a dense matrix (the paper's direct coarsest solve).
#pragma once

#include "eh_common.h"
#include "eh_mg_kernels.h"

namespace eh {

// Grid, frequency and absorbing layer of a context.
struct MediumArgs {
    int dim;
    int n[3];
    double h[3];
    double omega;
    double gamma0;
    int abc_width;
    unsigned abc_sides;
    __device__ int64_t cell(int i, int j, int k) const { return ((int64_t)k * n[1] + j) * n[0] + i; }
};

// mu = rho vs^2, lm = lambda + mu = rho (vp^2 - vs^2), C = 1 / lm, the
// attenuation gamma and the mass rho (1 - i gamma/w) per cell.
// gamma = gamma0 + w * sum_a l_a^2, l_a = max(0, W - d_a)/W, d_a the distance
// (cells, centre to side) to the nearest absorbing side along axis a
// (Section 4: a layer of gradually increasing attenuation).
__global__ void __launch_bounds__(256)
k_galerkin_medium(MediumArgs a, const double* __restrict__ vp, const double* __restrict__ vs,
                  const double* __restrict__ rho, double* __restrict__ mu, double* __restrict__ lm,
                  double* __restrict__ C, double* __restrict__ gamma, c128* __restrict__ mass) {
    const int64_t q = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (q >= (int64_t)a.n[0] * a.n[1] * a.n[2]) return;
    const int idx[3] = {(int)(q % a.n[0]), (int)((q / a.n[0]) % a.n[1]), (int)(q / ((int64_t)a.n[0] * a.n[1]))};
    double g = a.gamma0;
    if (a.abc_width > 0) {
        const double W = a.abc_width;
        for (int x = 0; x < a.dim; ++x) {
            double d = 1e300;
            if (a.abc_sides & (1u << (2 * x))) d = fmin(d, idx[x] + 0.5);
            if (a.abc_sides & (1u << (2 * x + 1))) d = fmin(d, a.n[x] - idx[x] - 0.5);
            const double l = fmax(0.0, W - d) / W;
            g += a.omega * l * l;
        }
    }
    const double r = rho[q], v = vp[q], w = vs[q];
    mu[q] = r * w * w;
    lm[q] = r * (v * v - w * w);
    C[q] = 1.0 / lm[q];
    gamma[q] = g;
    mass[q] = mk(r, -r * (g / a.omega));
}

// Mean of mu over the existing cells around the location whose nodal axes
// are `nodal` (bit mask) at location index L.
__device__ __forceinline__ double mu_mean(const MediumArgs& a, const double* mu, int nodal, const int L[3]) {
    double s = 0.0;
    int cnt = 0;
    for (int z = L[2] - ((nodal >> 2) & 1); z <= L[2]; ++z)
        for (int y = L[1] - ((nodal >> 1) & 1); y <= L[1]; ++y)
            for (int x = L[0] - (nodal & 1); x <= L[0]; ++x) {
                if (x < 0 || y < 0 || z < 0 || x >= a.n[0] || y >= a.n[1] || z >= a.n[2]) continue;
                s += mu[a.cell(x, y, z)];
                ++cnt;
            }
    return s / cnt;
}

// Fine-level operator as an FP64 stencil of half width 1 per axis, point p:
// centre D, couplings -wp[a] / -wm[a] to the neighbours along axis a.
__device__ __forceinline__ void put_stencil(int dim, int64_t np, int64_t p, c128 D, const double wp[3],
                                            const double wm[3], c128* st) {
    const int nst = dim == 3 ? 27 : 9, ctr = nst / 2;
    const int step[3] = {1, 3, 9};
    for (int o = 0; o < nst; ++o) st[(int64_t)o * np + p] = o == ctr ? D : mk(0.0, 0.0);
    for (int a = 0; a < dim; ++a) {
        st[(int64_t)(ctr + step[a]) * np + p] = mk(-wp[a], 0.0);
        st[(int64_t)(ctr - step[a]) * np + p] = mk(-wm[a], 0.0);
    }
}

template <class T>
struct FineOut {
    double* w[3];        // FP64 couplings of H (shear blocks)
    c128* D;             // FP64 diagonal of H, unshifted (shear blocks)
    T* fw[3];            // couplings in the multigrid precision
    cplx<T>* fD;         // shifted diagonal in the multigrid precision
    c128* st;            // shifted operator as a stencil, for the Galerkin products
};

// Fine-level acoustic block A_k on the k-faces: couplings w_a (between a
// face and its +e_a neighbour) and the diagonal, from grad_h^T A_e(mu) grad_h
// - w^2 A_f(m) (eq. mixed-discretized); alpha shifts the mass (eq. shift).
template <class T>
__global__ void __launch_bounds__(256)
k_galerkin_shear(MediumArgs a, int kb, double alpha, Dims d, const double* __restrict__ mu,
                 const double* __restrict__ rho, const double* __restrict__ gamma, FineOut<T> out) {
    const int64_t p = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (p >= d.np()) return;
    const int P[3] = {(int)(p % d.g[0]), (int)((p / d.g[0]) % d.g[1]), (int)(p / ((int64_t)d.g[0] * d.g[1]))};
    double wp[3] = {0.0, 0.0, 0.0}, wm[3] = {0.0, 0.0, 0.0};
    double stiff = 0.0;
    for (int x = 0; x < a.dim; ++x) {
        const double ih2 = 1.0 / (a.h[x] * a.h[x]);
        int q[3] = {P[0], P[1], P[2]};
        if (x == kb) {
            // derivative along the nodal axis lands on cells P[x]-1 and P[x]
            if (P[x] < a.n[x]) wp[x] = mu[a.cell(q[0], q[1], q[2])] * ih2;
            q[x] = P[x] - 1;
            if (P[x] >= 1) wm[x] = mu[a.cell(q[0], q[1], q[2])] * ih2;
            stiff += wp[x];
            stiff += wm[x];
        } else {
            // derivative along a cell-centred axis lands on edges at node
            // indices P[x] and P[x]+1 (zero ghost outside)
            const int nm = (1 << kb) | (1 << x);
            const double m0 = mu_mean(a, mu, nm, q) * ih2;
            q[x] = P[x] + 1;
            const double m1 = mu_mean(a, mu, nm, q) * ih2;
            stiff += m0 + m1;
            if (P[x] + 1 < d.g[x]) wp[x] = m1;
            if (P[x] >= 1) wm[x] = m0;
        }
    }
    // face mass: mean of the existing cells on both sides along kb
    double mr = 0.0, mi = 0.0, ms = 0.0;
    int cnt = 0;
    for (int off = -1; off <= 0; ++off) {
        int q[3] = {P[0], P[1], P[2]};
        q[kb] += off;
        if (q[kb] < 0 || q[kb] >= a.n[kb]) continue;
        const int64_t c = a.cell(q[0], q[1], q[2]);
        mr += rho[c];
        mi -= rho[c] * (gamma[c] / a.omega);
        ms -= rho[c] * (gamma[c] / a.omega + alpha);
        ++cnt;
    }
    const double om2 = a.omega * a.omega;
    const double re = stiff - om2 * (mr / cnt);
    const c128 D0 = mk(re, -om2 * (mi / cnt)), Ds = mk(re, -om2 * (ms / cnt));
    for (int x = 0; x < a.dim; ++x) {
        out.w[x][p] = wp[x];
        out.fw[x][p] = T(wp[x]);
    }
    out.D[p] = D0;
    out.fD[p] = ccast<T>(Ds);
    put_stencil(a.dim, d.np(), p, Ds, wp, wm, out.st);
}

// Fine-level H_p on the cells: H_p = B B^T diag(w) - w^2 diag(m/(lambda+mu)),
// w = (lambda + 2 mu)/(lambda + mu) (eqs. Ap, Hp); alpha shifts m.
//
// TILDE: with the Remark's A~_p = B A_f(mu) B^T - w^2 M_p in place of A_p,
// H~_p = B B^T + A~_p C.  Across the face between cell c and its neighbour
// nb along axis a the coupling is (1 + mu_f / (lambda+mu)_nb) / h_a^2, mu_f
// the mean of the face's existing cells (a boundary face has one); the
// diagonal collects (1 + mu_f / (lambda+mu)_c) / h_a^2 over the cell's
// faces and the shifted mass / (lambda+mu)_c.  fw[a] holds the pair
// (coupling to c + e_a, to c - e_a) per cell.
template <class T, bool TILDE>
__global__ void __launch_bounds__(256)
k_galerkin_pressure(MediumArgs a, double alpha, const double* __restrict__ mu, const double* __restrict__ lm,
                    const double* __restrict__ rho, const double* __restrict__ gamma, FineOut<T> out) {
    const int64_t np = (int64_t)a.n[0] * a.n[1] * a.n[2];
    const int64_t p = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (p >= np) return;
    const int64_t st[3] = {1, a.n[0], (int64_t)a.n[0] * a.n[1]};
    const int P[3] = {(int)(p % a.n[0]), (int)((p / a.n[0]) % a.n[1]), (int)(p / st[2])};
    double wp[3] = {0.0, 0.0, 0.0}, wm[3] = {0.0, 0.0, 0.0};
    double diag = 0.0;
    const double wc = 1.0 + mu[p] / lm[p];
    double sum_ih2 = 0.0;
    for (int x = 0; x < a.dim; ++x) {
        const double ih2 = 1.0 / (a.h[x] * a.h[x]);
        const bool hi = P[x] + 1 < a.n[x], lo = P[x] > 0;
        if (TILDE) {
            const double mhi = hi ? 0.5 * (mu[p] + mu[p + st[x]]) : mu[p];
            const double mlo = lo ? 0.5 * (mu[p] + mu[p - st[x]]) : mu[p];
            if (hi) wp[x] = (1.0 + mhi / lm[p + st[x]]) * ih2;
            if (lo) wm[x] = (1.0 + mlo / lm[p - st[x]]) * ih2;
            diag += (2.0 + (mlo + mhi) / lm[p]) * ih2;
            out.fw[x][2 * p] = T(wp[x]);
            out.fw[x][2 * p + 1] = T(wm[x]);
        } else {
            sum_ih2 += 2.0 / (a.h[x] * a.h[x]);
            if (hi) wp[x] = (1.0 + mu[p + st[x]] / lm[p + st[x]]) * ih2;
            if (lo) wm[x] = (1.0 + mu[p - st[x]] / lm[p - st[x]]) * ih2;
        }
    }
    if (!TILDE) {
        diag = wc * sum_ih2;
        out.fw[0][p] = T(wc);
    }
    const double om2 = a.omega * a.omega;
    const c128 D = mk(diag - om2 * rho[p] / lm[p], om2 * (rho[p] * (gamma[p] / a.omega + alpha)) / lm[p]);
    out.fD[p] = ccast<T>(D);
    put_stencil(a.dim, np, p, D, wp, wm, out.st);
}

constexpr int GAL_MAXW = 2;                                  // coarse half width
constexpr int GAL_MAXN = (2 * GAL_MAXW + 1) * (2 * GAL_MAXW + 1) * (2 * GAL_MAXW + 1);

// Fine stencil (widths wf, fine grid df) -> coarse stencil (widths wc,
// coarse grid dc).  For coarse point I: sum over fine k in the support of
// row I of R, over fine offsets o, over coarse parents J of l = k + o.
__global__ void __launch_bounds__(64)
k_galerkin(Dims df, Widths wf, const c128* __restrict__ cf, Dims dc, Widths wc, int nodal_mask, int mixed,
           c128* __restrict__ cc, int* __restrict__ overflow) {
    const int64_t npc = dc.np();
    const int64_t q = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (q >= npc) return;
    const int I = (int)(q % dc.g[0]);
    const int J = (int)((q / dc.g[0]) % dc.g[1]);
    const int K = (int)(q / ((int64_t)dc.g[0] * dc.g[1]));
    c128 acc[GAL_MAXN];
    const int ncs = wc.nst();
    for (int t = 0; t < ncs; ++t) acc[t] = mk(0.0, 0.0);
    const bool nz = (nodal_mask & 4) != 0;
    const bool three = (df.g[2] > 1) || nz;
    Transfer1D rx, ry, rz;
    rx.restrict_support(I, nodal_mask & 1, df.g[0], mixed);
    ry.restrict_support(J, nodal_mask & 2, df.g[1], mixed);
    if (three) rz.restrict_support(K, nz, df.g[2], mixed);
    else { rz.n = 1; rz.idx[0] = 0; rz.wt[0] = 1.0f; }
    const int64_t npf = df.np();
    const int NXf = 2 * wf.w[0] + 1, NYf = 2 * wf.w[1] + 1;
    const int NXc = 2 * wc.w[0] + 1, NYc = 2 * wc.w[1] + 1;
    for (int a = 0; a < rz.n; ++a)
    for (int b = 0; b < ry.n; ++b)
    for (int c = 0; c < rx.n; ++c) {
        const int kx = rx.idx[c], ky = ry.idx[b], kz = rz.idx[a];
        const double rw = double(rx.wt[c]) * double(ry.wt[b]) * double(rz.wt[a]);
        const int64_t kp = ((int64_t)kz * df.g[1] + ky) * df.g[0] + kx;
        for (int oz = -wf.w[2]; oz <= wf.w[2]; ++oz)
        for (int oy = -wf.w[1]; oy <= wf.w[1]; ++oy)
        for (int ox = -wf.w[0]; ox <= wf.w[0]; ++ox) {
            const int o = ((oz + wf.w[2]) * NYf + (oy + wf.w[1])) * NXf + (ox + wf.w[0]);
            const c128 x = cf[o * npf + kp];
            if (x.re == 0.0 && x.im == 0.0) continue;
            const int lx = kx + ox, ly = ky + oy, lz = kz + oz;
            if (lx < 0 || lx >= df.g[0] || ly < 0 || ly >= df.g[1] || lz < 0 || lz >= df.g[2]) {
                overflow[0] = 1;                  // nonzero coupling outside the grid
                continue;
            }
            Transfer1D px, py, pz;
            px.prolong_parents(lx, nodal_mask & 1, dc.g[0]);
            py.prolong_parents(ly, nodal_mask & 2, dc.g[1]);
            if (three) pz.prolong_parents(lz, nz, dc.g[2]);
            else { pz.n = 1; pz.idx[0] = 0; pz.wt[0] = 1.0f; }
            for (int e = 0; e < pz.n; ++e)
            for (int f = 0; f < py.n; ++f)
            for (int g = 0; g < px.n; ++g) {
                // prolongation weights are 2x the restriction weights per axis
                const int dx = px.idx[g] - I, dy = py.idx[f] - J, dz = pz.idx[e] - K;
                if (dx < -wc.w[0] || dx > wc.w[0] || dy < -wc.w[1] || dy > wc.w[1] ||
                    dz < -wc.w[2] || dz > wc.w[2]) {
                    overflow[0] = 1;
                    continue;
                }
                double pw = double(px.wt[g]) * double(py.wt[f]) * double(pz.wt[e]);
                const int t = ((dz + wc.w[2]) * NYc + (dy + wc.w[1])) * NXc + (dx + wc.w[0]);
                const double s = rw * pw;
                acc[t] = acc[t] + mk(s * x.re, s * x.im);
            }
        }
    }
    for (int t = 0; t < ncs; ++t) cc[t * npc + q] = acc[t];
}

// Dense matrix of a stencil, row-major with row stride ld: with augment
// [A | I] (N x 2N, cleared here), else A into a matrix that holds the
// identity (its own diagonal is overwritten, the padding stays).
__global__ void k_dense_from_stencil(Dims d, Widths w, const c128* __restrict__ st, c128* __restrict__ M, int64_t ld,
                                     int augment) {
    const int64_t N = d.np();
    const int64_t q = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (q >= N) return;
    const int i = (int)(q % d.g[0]);
    const int j = (int)((q / d.g[0]) % d.g[1]);
    const int k = (int)(q / ((int64_t)d.g[0] * d.g[1]));
    c128* row = M + q * ld;
    if (augment) {
        for (int64_t c = 0; c < 2 * N; ++c) row[c] = mk(0.0, 0.0);
        row[N + q] = mk(1.0, 0.0);
    }
    const int NX = 2 * w.w[0] + 1, NY = 2 * w.w[1] + 1;
    for (int oz = -w.w[2]; oz <= w.w[2]; ++oz)
    for (int oy = -w.w[1]; oy <= w.w[1]; ++oy)
    for (int ox = -w.w[0]; ox <= w.w[0]; ++ox) {
        const int x = i + ox, y = j + oy, z = k + oz;
        if (x < 0 || x >= d.g[0] || y < 0 || y >= d.g[1] || z < 0 || z >= d.g[2]) continue;
        const int o = ((oz + w.w[2]) * NY + (oy + w.w[1])) * NX + (ox + w.w[0]);
        row[((int64_t)z * d.g[1] + y) * d.g[0] + x] = st[o * N + q];
    }
}

// Gauss-Jordan step kk, part 1: pivot = argmax_{i >= kk} |M[i][kk]| (one block).
__global__ void __launch_bounds__(256)
k_gj_pivot(int64_t N, int64_t kk, const c128* __restrict__ M, int64_t* __restrict__ piv,
           c128* __restrict__ pval) {
    __shared__ double bv[256];
    __shared__ int64_t bi[256];
    double best = -1.0;
    int64_t besti = kk;
    for (int64_t i = kk + threadIdx.x; i < N; i += blockDim.x) {
        const double a = cabs2(M[i * 2 * N + kk]);
        if (a > best) { best = a; besti = i; }
    }
    bv[threadIdx.x] = best; bi[threadIdx.x] = besti;
    __syncthreads();
    for (int s = 128; s > 0; s >>= 1) {
        if (threadIdx.x < s) {
            const double o = bv[threadIdx.x + s];
            const int64_t oi = bi[threadIdx.x + s];
            if (o > bv[threadIdx.x] || (o == bv[threadIdx.x] && oi < bi[threadIdx.x])) {
                bv[threadIdx.x] = o; bi[threadIdx.x] = oi;
            }
        }
        __syncthreads();
    }
    if (threadIdx.x == 0) {
        *piv = bi[0];
        *pval = M[bi[0] * 2 * N + kk];
    }
}

// part 2: swap rows kk and pivot and scale row kk by 1 / pivot value (the
// value was saved by k_gj_pivot, so no thread reads a row being rewritten).
__global__ void __launch_bounds__(256)
k_gj_swap_scale(int64_t N, int64_t kk, c128* __restrict__ M, const int64_t* __restrict__ piv,
                const c128* __restrict__ pval) {
    const int64_t pr = *piv;
    const c128 pv = *pval;
    const c128 inv = cdiv(mk(1.0, 0.0), pv);
    for (int64_t c = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; c < 2 * N;
         c += (int64_t)gridDim.x * blockDim.x) {
        const c128 a = M[kk * 2 * N + c];
        const c128 b = M[pr * 2 * N + c];
        if (pr != kk) M[pr * 2 * N + c] = a;
        M[kk * 2 * N + c] = inv * b;
    }
}

__global__ void __launch_bounds__(256)
k_gj_column(int64_t N, int64_t kk, const c128* __restrict__ M, c128* __restrict__ mult) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < N) mult[i] = (i == kk) ? mk(0.0, 0.0) : M[i * 2 * N + kk];
}

// part 3: M[i][c] -= mult[i] * M[kk][c] for i != kk
__global__ void __launch_bounds__(256)
k_gj_eliminate(int64_t N, int64_t kk, c128* __restrict__ M, const c128* __restrict__ mult) {
    const int64_t c = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    const int64_t i = blockIdx.y;
    if (c >= 2 * N || i == kk) return;
    const c128 m = mult[i];
    if (m.re == 0.0 && m.im == 0.0) return;
    M[i * 2 * N + c] = M[i * 2 * N + c] - m * M[kk * 2 * N + c];
}

__global__ void k_gj_extract(int64_t N, const c128* __restrict__ M, c128* __restrict__ inv) {
    const int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (t >= N * N) return;
    const int64_t i = t / N, c = t % N;
    inv[t] = M[i * 2 * N + N + c];
}

}  // namespace eh
