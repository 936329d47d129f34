"""GPU parity of the block-tridiagonal coarsest solve (needs an MI355X).

The coarsest level of every block is solved directly (Section 4.4.1).  The
oracle solves it by sparse LU (scipy's splu); the GPU factors it block-
tridiagonally over groups of planes.  Both are exact up to rounding, so the
results agree to 1e-10 relative (FP64), on the fine operators themselves
(one level: the cycle is the direct solve) and under Galerkin coarsening
with either intergrid, in 2D (coarsest 64 x 64) and 3D (coarsest 12^3).
"""
import sys

import numpy as np
import pytest
import scipy.sparse.linalg as spla

import workloads as W
from oracle.elastic import ElasticSystem, face_nodal
from oracle.multigrid import Hierarchy

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


def say(*a):
    print(*a, file=sys.stderr, flush=True)


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2411_15897_amd import _native
    _native.lib()          # fails loudly when the library is missing


def hetero_medium(n, seed):
    rng = np.random.default_rng(seed)
    shape = tuple(reversed(n))
    vp = rng.uniform(2.0, 3.5, shape)
    vs = vp * rng.uniform(0.35, 0.55, shape)
    rho = rng.uniform(1.0, 2.0, shape)
    return vp, vs, rho


def make(n, seed=0, omega=0.7, abc=4, **kw):
    from paper_2411_15897_amd import ElasticHelmholtz
    dim = len(n)
    h = tuple(1.0 + 0.1 * a for a in range(dim))
    vp, vs, rho = hetero_medium(n, seed)
    sides = W.ABC_ALL[dim]
    gpu = ElasticHelmholtz(n, h, vp, vs, rho, omega, abc_width=abc, abc_sides=sides, **kw)
    sys_ = ElasticSystem(n, h, vp, vs, rho, omega, abc, sides)
    return gpu, sys_


def crand(shape, seed):
    rng = np.random.default_rng(seed)
    return rng.standard_normal(shape) + 1j * rng.standard_normal(shape)


def to_dev(a):
    return torch.from_numpy(np.ascontiguousarray(a)).to("cuda")


def rel(a, b):
    return np.linalg.norm(a - b) / max(np.linalg.norm(b), 1e-300)


def block_op(s, b, alpha):
    return s.H_p(alpha) if b == s.dim else s.A_block(b, alpha)


@pytest.mark.parametrize("n", [(64, 64), (40, 24), (12, 12, 12), (10, 6, 8)])
def test_direct_solve_of_fine_blocks(n):
    """One level: the cycle is the coarsest solve of the shifted fine block.
    Block-tridiagonal against splu (1e-10), and against the dense inverse
    where that fits (1e-10); two right-hand sides at once equal one at a
    time bitwise."""
    say("block-tridiagonal direct solve, one level", n)
    alpha = 0.3
    gpu, s = make(n, seed=1, levels=1, alpha=alpha, mg_precision=64, coarse_solver="bt")
    dense = None
    if max(int(np.prod(gpu.block_dims(b, 0))) for b in range(s.dim + 1)) <= 6000:
        dense, _ = make(n, seed=1, levels=1, alpha=alpha, mg_precision=64, coarse_solver="dense")
    for b in range(s.dim + 1):
        X = block_op(s, b, alpha).tocsc()
        f = crand((2, X.shape[0]), 5 + b)
        e = gpu.block_cycle(b, to_dev(f)).cpu().numpy()
        lu = spla.splu(X)
        for k in range(2):
            ref = lu.solve(f[k])
            assert rel(e[k], ref) <= 1e-10, (b, k, rel(e[k], ref))
            e1 = gpu.block_cycle(b, to_dev(f[k])).cpu().numpy()
            assert np.array_equal(e1, e[k])
        if dense is not None:
            ed = dense.block_cycle(b, to_dev(f)).cpu().numpy()
            assert rel(e, ed) <= 1e-10
    gpu.close()
    if dense is not None:
        dense.close()


@pytest.mark.parametrize("n,intergrid,levels", [
    ((128, 128), "full", 2),     # coarsest 64 x 64: line pairs along the cell-centred axes
    ((128, 128), "mixed", 2),
    ((128, 64), "full", 3),
    ((24, 24, 24), "mixed", 2),  # coarsest 12^3: plane groups of one
    ((24, 24, 24), "full", 2),   # plane pairs along cell-centred axes
])
def test_cycle_with_block_tridiagonal_coarsest(n, intergrid, levels):
    """A full cycle (V(1,2) in 2D, V(2,2) in 3D) whose coarsest Galerkin
    level is solved block-tridiagonally, against the oracle's cycle with
    splu on the coarsest level (FP64, 1e-10); complex64 multigrid within
    1e-5."""
    say("cycle with block-tridiagonal coarsest", n, intergrid, levels)
    alpha = 0.3
    dim = len(n)
    nu = (1, 2) if dim == 2 else (2, 2)
    damping = (0.8, 0.8, 0.3) if dim == 2 else (0.8, 0.8, 0.2)
    kw = dict(levels=levels, alpha=alpha, nu=nu, damping=damping, intergrid=intergrid, coarse_solver="bt")
    gpu, s = make(n, seed=2, mg_precision=64, **kw)
    g32, _ = make(n, seed=2, mg_precision=32, **kw)
    for b in range(dim + 1):
        X = block_op(s, b, alpha)
        nodal = tuple(False for _ in range(dim)) if b == dim else face_nodal(dim, b)
        mg = Hierarchy(X, s.n, nodal, levels, damping=damping, nu=nu, intergrid=intergrid)
        f = crand(X.shape[0], 30 + b)
        ref = mg(f)
        e = gpu.block_cycle(b, to_dev(f)).cpu().numpy()
        assert rel(e, ref) <= 1e-10, (b, rel(e, ref))
        e32 = g32.block_cycle(b, to_dev(f)).cpu().numpy()
        say(f"  block {b}: FP64 {rel(e, ref):.2e}, complex64 multigrid {rel(e32, ref):.2e}")
        assert rel(e32, ref) <= 1e-5
    gpu.close()
    g32.close()


@pytest.mark.parametrize("intergrid", ["mixed", "full"])
def test_wide_groups_batched(intergrid):
    """Coarsest 20^3: groups of one plane (400-420 unknowns) with the mixed
    intergrid, plane pairs (800-840) with full weighting, so the forward
    and back steps and the S_I^-1 f_I launch take their columns in several
    chunks (320 columns per chunk with 5-8 right-hand sides, 640 with
    fewer).  Each right-hand side of a batch of 7, and one alone, against
    the oracle's cycle with splu on the coarsest level (FP64, 1e-10)."""
    say("block-tridiagonal wide groups, batched", intergrid)
    n, alpha = (40, 40, 40), 0.3
    nu, damping = (2, 2), (0.8, 0.8, 0.2)
    kw = dict(levels=2, alpha=alpha, nu=nu, damping=damping, intergrid=intergrid, coarse_solver="bt")
    gpu, s = make(n, seed=5, mg_precision=64, **kw)
    for b in range(4):
        X = block_op(s, b, alpha)
        nodal = (False,) * 3 if b == 3 else face_nodal(3, b)
        mg = Hierarchy(X, s.n, nodal, 2, damping=damping, nu=nu, intergrid=intergrid)
        f = crand((7, X.shape[0]), 50 + b)
        e = gpu.block_cycle(b, to_dev(f)).cpu().numpy()
        e1 = gpu.block_cycle(b, to_dev(f[:1])).cpu().numpy()[0]
        errs = [rel(e[k], mg(f[k])) for k in range(7)]
        say(f"  block {b}: max rel err {max(errs):.1e}")
        assert max(errs) <= 1e-10, (b, errs)
        assert rel(e1, e[0]) <= 1e-13
    gpu.close()


@pytest.mark.parametrize("nrhs", [3, 7, 9])
def test_batch_equals_single(nrhs):
    """Chunks of 4 or 8 right-hand sides per workgroup (and a ragged last
    chunk) give each right-hand side bitwise what it gets alone, through
    the whole preconditioner."""
    say("block-tridiagonal batch", nrhs)
    n = (48, 32)
    gpu, s = make(n, seed=3, levels=2, alpha=0.4, mg_precision=32, coarse_solver="bt")
    r = crand((nrhs, s.ndof), 4)
    zb = gpu.apply_preconditioner(to_dev(r)).cpu().numpy()
    for k in range(nrhs):
        zk = gpu.apply_preconditioner(to_dev(r[k:k + 1])).cpu().numpy()[0]
        assert np.array_equal(zb[k], zk), k
    gpu.close()


@pytest.mark.parametrize("n", [
    (50, 41),        # 50 groups of 41: one level of the elimination, then 25 groups dense
    (33, 97),        # odd group counts on two levels
    (130, 17),       # long chain of narrow groups, the last one kept or removed
    (200, 9),
    (61, 64),        # 61 or 62 groups: the chain ends on a removed group
    (13, 14, 15),    # 3D, groups of one plane of about 180
    (150, 151),      # groups of 150: the first level's couplings from lists, odd count
    (160, 150),      # the same along the other axis, even count for two of the blocks
    (18, 20, 23),    # and in 3D
])
@pytest.mark.parametrize("nrhs", [1, 2, 3, 6])
def test_elimination_levels(n, nrhs):
    """Chains of groups whose elimination in levels ends differently (odd
    and even counts, a last group without a right neighbour, a dense rest of
    several groups) and every chunk width of the solve, against splu on the
    fine blocks (one level, FP64, 1e-10 as above)."""
    say("elimination levels", n, nrhs)
    alpha = 0.3
    gpu, s = make(n, seed=11, levels=1, alpha=alpha, mg_precision=64, coarse_solver="bt")
    for b in range(s.dim + 1):
        X = block_op(s, b, alpha).tocsc()
        f = crand((nrhs, X.shape[0]), 70 + b)
        e = gpu.block_cycle(b, to_dev(f)).cpu().numpy()
        lu = spla.splu(X)
        for k in range(nrhs):
            assert rel(e[k], lu.solve(f[k])) <= 1e-10, (b, k)
    gpu.close()


def test_dense_inverse_with_small_pivot_blocks():
    """The dense inverse's pivot blocks pivot only inside themselves.  A
    medium whose constant velocities make the leading diagonal entries of
    the unshifted, unattenuated operator vanish (the stiffness of the
    pressure block's interior cells equals the mass term) is still inverted:
    against splu, FP64, with the accuracy the set-up's check asks for
    (1e-11) times the operator's conditioning taken from the oracle."""
    from paper_2411_15897_amd import ElasticHelmholtz
    n, h = (24, 20), (1.0, 1.0)
    shape = tuple(reversed(n))
    vp, vs, rho = np.full(shape, 2.0), np.full(shape, 1.0), np.ones(shape)
    # H_p: (1 + mu / (lambda + mu)) * 4 = omega^2 rho / (lambda + mu)
    omega = float(np.sqrt(4.0 * (1.0 + 1.0 / 3.0) * 3.0))
    gpu = ElasticHelmholtz(n, h, vp, vs, rho, omega, levels=1, alpha=0.05, abc_width=0, abc_sides=0xF, gamma0=0.0,
                           mg_precision=64, coarse_solver="dense")
    s = ElasticSystem(n, h, vp, vs, rho, omega, 0, 0xF, gamma0=0.0)
    for b in range(3):
        X = block_op(s, b, 0.05).tocsc()
        f = crand(X.shape[0], 90 + b)
        e = gpu.block_cycle(b, to_dev(f)).cpu().numpy()
        cond = np.linalg.cond(X.toarray())
        assert rel(e, spla.splu(X).solve(f)) <= max(1e-10, 1e-11 * cond), b
    gpu.close()


@pytest.mark.parametrize("n,solver", [
    ((150, 151), "bt"),      # the first level's couplings from lists
    ((18, 20, 23), "bt"),    # and in 3D
    ((50, 41), "bt"),
    ((24, 20), "dense"),
])
@pytest.mark.parametrize("nrhs", [1, 4])
def test_no_trace_of_an_earlier_solve(n, solver, nrhs):
    """What a solve leaves in the work vectors (here NaN everywhere, as fresh
    memory may hold) does not enter the next one: bitwise the same."""
    gpu, s = make(n, seed=12, levels=1, alpha=0.3, mg_precision=64, coarse_solver=solver)
    for b in range(s.dim + 1):
        f = to_dev(crand((nrhs, block_op(s, b, 0.3).shape[0]), 80 + b))
        e = gpu.block_cycle(b, f)
        assert torch.isnan(torch.view_as_real(gpu.block_cycle(b, torch.full_like(f, float("nan"))))).any()
        assert torch.equal(gpu.block_cycle(b, f), e), b
    gpu.close()


@pytest.mark.parametrize("n", [(24, 20), (11, 12)])
def test_dense_inverse_with_pivoting_over_all_rows(n):
    """The blocked inverse pivots inside its 32 x 32 blocks only.  Without
    shift and attenuation, at the frequency where the stiffness of the
    pressure block's diagonal equals the mass, its leading block is singular
    (asserted here) while the matrix is not, so the inverse has to come from
    the elimination that pivots over all rows: against splu within 1e-11,
    the residual the set-up asks of the blocked form, times the condition."""
    from paper_2411_15897_amd import ElasticHelmholtz
    say("dense inverse, pivoting over all rows", n)
    h, shape = (1.0, 1.0), tuple(reversed(n))
    vp, vs, rho = np.full(shape, 2.0), np.full(shape, 1.0), np.ones(shape)
    # (1 + mu / (lambda + mu)) * 4 = omega^2 rho / (lambda + mu), lambda + mu = 3
    omega = float(np.sqrt(4.0 * (1.0 + 1.0 / 3.0) * 3.0))
    s = ElasticSystem(n, h, vp, vs, rho, omega, 0, 0xF, gamma0=0.0)
    lead = np.linalg.svd(s.H_p(0.0).toarray()[:32, :32], compute_uv=False)
    assert lead[-1] <= 1e-14 * lead[0]
    gpu = ElasticHelmholtz(n, h, vp, vs, rho, omega, levels=1, alpha=0.0, abc_width=0, abc_sides=0xF, gamma0=0.0,
                           mg_precision=64, coarse_solver="dense")
    for b in range(3):
        X = block_op(s, b, 0.0).tocsc()
        cond = np.linalg.cond(X.toarray())
        assert cond < 1e3
        f = crand((3, X.shape[0]), 95 + b)
        e = gpu.block_cycle(b, to_dev(f)).cpu().numpy()
        for k in range(3):
            assert rel(e[k], spla.splu(X).solve(f[k])) <= 1e-11 * max(cond, 10.0), (b, k)
    gpu.close()


@pytest.mark.parametrize("n,k,delta,limit", [
    ((40, 50), 13, 0.0, 1e-11),      # 50 groups of 40
    ((150, 160), 20, 0.0, 5e-11),    # matrices large enough for the first level's lists, dropped with them
    ((40, 50), 13, 3e-4, 1e-11),     # near-singular: the nested order loses digits (1e-10) but not all
])
def test_groups_eliminated_one_after_the_other(n, k, delta, limit):
    """A line of cells whose own block of the pressure operator is singular
    to `delta` (asserted here), the third of the chain: removing every other
    group meets it as it is, removing the groups one after the other adds a
    Schur complement first.  The lines around it are stiff, no shift, no
    attenuation.  Limits: 30 times and more the residual of a NumPy replay
    of that order with these right-hand sides (2e-13, 1.5e-12, 6e-14)."""
    from paper_2411_15897_amd import ElasticHelmholtz
    say("groups one after the other", n)
    h, rng = (1.0, 1.0), np.random.default_rng(0)
    line = 3.0 + rng.random(n[1])
    line[2] = 1.0
    vs = np.repeat(line[:, None], n[0], 1)
    vp, rho = 2.0 * vs, np.ones_like(vs)
    # the k-th eigenvalue of line 2: lambda + mu = 3, mu = 1
    omega = float(np.sqrt(3.0 * (4.0 / 3.0 * (4.0 - 2.0 * np.cos(k * np.pi / (n[0] + 1))) - delta)))
    s = ElasticSystem(n, h, vp, vs, rho, omega, 0, 0xF, gamma0=0.0)
    X = s.H_p(0.0).tocsr()
    own = slice(2 * n[0], 3 * n[0])
    assert abs(np.linalg.svd(X[own, own].toarray(), compute_uv=False)[-1] - delta) <= 1e-12
    gpu = ElasticHelmholtz(n, h, vp, vs, rho, omega, levels=1, alpha=0.0, abc_width=0, abc_sides=0xF, gamma0=0.0,
                           mg_precision=64, coarse_solver="bt")
    f = crand((3, X.shape[0]), 99)
    e = gpu.block_cycle(2, to_dev(f)).cpu().numpy()
    e1 = gpu.block_cycle(2, to_dev(f[1])).cpu().numpy()
    gpu.close()
    for q in range(3):
        res = rel(X @ e[q], f[q])
        say(f"  residual {res:.1e}")
        assert res <= limit, q
    assert np.array_equal(e1, e[1])


def test_chain_beyond_one_launch():
    """24 000 groups of two points: the first level's 72 000 blocks and its
    inverses take several launches; FP64 against splu, 1e-10 as above."""
    n, alpha = (24000, 2), 0.3
    say("long chain", n)
    gpu, s = make(n, seed=13, levels=1, alpha=alpha, mg_precision=64, coarse_solver="bt")
    for b in range(3):
        X = block_op(s, b, alpha).tocsc()
        f = crand(X.shape[0], 60 + b)
        assert rel(gpu.block_cycle(b, to_dev(f)).cpu().numpy(), spla.splu(X).solve(f)) <= 1e-10, b
    gpu.close()
