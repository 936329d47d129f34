"""The Arnoldi step at the edges of its launch rules (needs an MI355X).

Short vectors take one entry per thread and their columns four at a time;
grids of few tiles deal the basis columns of the first Gram-Schmidt pass to
several workgroups; few workgroups leave their partial sums to the
coefficient and rotation kernels.  Each of these changes with the grid, the
restart length and the batch, so solves on grids to both sides of every
threshold are checked against the oracle's operator.
"""
import numpy as np
import pytest

import workloads as W
from oracle.elastic import apply_H_stencil, medium_arrays

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2411_15897_amd import _native
    _native.lib()


@pytest.mark.parametrize("n,levels", [
    ((16, 12), 1),          # one tile in x, four in y
    ((64, 64), 3),          # 34 tiles: sums folded, columns over 10 workgroups
    ((120, 168), 3),        # 86 tiles: folded, the norm's 238 sums too
    ((136, 256), 3),        # 195 tiles: the first pass reduced by its own launch
    ((288, 296), 4),        # the longest vectors still short, norm reduced by its own launch
    ((304, 296), 4),        # the shortest of the others
    ((12, 10, 8), 1),       # 3D: the pass is a launch of its own
])
@pytest.mark.parametrize("restart", [1, 2, 5, 32])
def test_restart_lengths(n, levels, restart):
    """Three sources, alone and batched: the true residual recomputed by the
    oracle is below the tolerance, the Arnoldi estimate of the last step
    equals it to 1e-10 (FP64 sums), and the batch gives each source bitwise
    what it gets alone."""
    from paper_2411_15897_amd import ElasticHelmholtz
    d, h = len(n), tuple(1.0 for _ in n)
    rng = np.random.default_rng(2)
    vp = rng.uniform(2.0, 2.6, tuple(reversed(n)))
    vs, rho = 0.5 * vp, np.ones_like(vp)
    omega = W.omega_for_ppw(vs, h, 12.0)
    sides = W.ABC_ALL[d]
    s = ElasticHelmholtz(n, h, vp, vs, rho, omega, levels=levels, alpha=0.4, mg_precision=64, restart=restart,
                         abc_width=4, abc_sides=sides)
    src = [(d - 1, tuple(n[a] // 2 + q - 1 if a < d - 1 else n[a] // 2 for a in range(d))) for q in range(3)]
    b = W.point_source_rhs(n, h, src)
    tol = 1e-6
    x, info = s.solve(torch.from_numpy(b).cuda(), tol=tol, maxit=600)
    mu, lm, mass = medium_arrays(n, h, vp, vs, rho, omega, 4, sides)
    for q in range(3):
        xq = x[q].cpu().numpy()
        rr = np.linalg.norm(b[q] - apply_H_stencil(n, h, mu, lm, mass, omega, xq)) / np.linalg.norm(b[q])
        assert info[q]["converged"] and rr < tol
        assert abs(info[q]["relres_est"] - rr) <= 1e-10
        x1, i1 = s.solve(torch.from_numpy(b[q:q + 1]).cuda(), tol=tol, maxit=600)
        assert i1[0]["iters"] == info[q]["iters"] and np.array_equal(x1[0].cpu().numpy(), xq)
    s.close()


@pytest.mark.parametrize("n,nsrc", [
    ((848, 840), 4),        # vectors of the batch just above 128 MiB: H z formed twice
    ((840, 832), 4),        # just below: H z written and read back
    ((624, 600), 8),        # above, the batch split over workgroups
])
@pytest.mark.parametrize("restart", [2, 5])
def test_second_pass_forms_the_vector_again(n, nsrc, restart):
    """The second Gram-Schmidt pass on a large batch forms H z again instead
    of reading it: true residuals recomputed by the oracle below the
    tolerance and equal to the Arnoldi estimate to 1e-10, as above; finished
    sources leave the batch on the way."""
    from paper_2411_15897_amd import ElasticHelmholtz
    h, levels = (1.0, 1.0), 4
    vp, vs, rho = W.layered_medium(n, seed=5)
    omega = W.omega_for_ppw(vs, h, 12.0)
    sides = W.abc_all_but_top(2)
    s = ElasticHelmholtz(n, h, vp, vs, rho, omega, levels=levels, alpha=0.5, restart=restart, abc_width=20,
                         abc_sides=sides)
    b = W.point_source_rhs(n, h, [(1, ((2 * q + 1) * n[0] // (2 * nsrc), 1)) for q in range(nsrc)])
    x, info = s.solve(torch.from_numpy(b).cuda(), tol=1e-6, maxit=600)
    mu, lm, mass = medium_arrays(n, h, vp, vs, rho, omega, 20, sides)
    for q in range(nsrc):
        rr = np.linalg.norm(b[q] - apply_H_stencil(n, h, mu, lm, mass, omega, x[q].cpu().numpy()))
        rr /= np.linalg.norm(b[q])
        assert info[q]["converged"] and rr < 1e-6
        assert abs(info[q]["relres_est"] - rr) <= 1e-10
    s.close()


@pytest.mark.parametrize("n,nsrc,precision,above", [
    ((848, 840), 4, 32, True),     # the batch forms H z twice, a source alone writes and reads it
    ((840, 824), 4, 32, False),    # the batch writes and reads it too
    ((624, 600), 8, 64, True),
    ((256, 256), 43, 32, True),    # the shortest vectors summed by tiles
    ((256, 248), 44, 32, True),    # just shorter
])
def test_batch_gives_each_source_what_it_gets_alone(n, nsrc, precision, above):
    """Batches on both sides of 128 MiB per basis vector, of which sources
    leave on the way: true residuals recomputed by the oracle are below the
    tolerance and equal to the Arnoldi estimate to 1e-10, x and the counts
    of every source are bitwise those it gets alone, in a pair, and with
    drop_converged off."""
    from paper_2411_15897_amd import ElasticHelmholtz
    ndof = (n[0] + 1) * n[1] + n[0] * (n[1] + 1) + n[0] * n[1]
    assert (nsrc * ndof * 16 >= 128 * 2**20) == above
    h = (1.0, 1.0)
    vp, vs, rho = W.layered_medium(n, seed=5)
    omega = W.omega_for_ppw(vs, h, 12.0)
    kw = dict(levels=4, alpha=0.5, restart=3, abc_width=20, abc_sides=W.abc_all_but_top(2),
              mg_precision=precision)
    # from the middle of the top to inside the absorbing layer at the bottom
    b = W.point_source_rhs(n, h, [(1, (n[0] // 2 + q, 1 + q * (n[1] - 3) // (nsrc - 1))) for q in range(nsrc)])
    bt = torch.from_numpy(b).cuda()
    s = ElasticHelmholtz(n, h, vp, vs, rho, omega, **kw)
    x, info = s.solve(bt, tol=1e-3, maxit=90)
    its = [i["iters"] for i in info]
    assert min(its) < max(its)
    mu, lm, mass = medium_arrays(n, h, vp, vs, rho, omega, 20, W.abc_all_but_top(2))
    for q in (0, nsrc - 1):
        rr = np.linalg.norm(b[q] - apply_H_stencil(n, h, mu, lm, mass, omega, x[q].cpu().numpy()))
        rr /= np.linalg.norm(b[q])
        assert info[q]["converged"] and rr < 1e-3 and abs(info[q]["relres_est"] - rr) <= 1e-10
    for q in (0, nsrc // 2, nsrc - 1):
        x1, i1 = s.solve(bt[q:q + 1], tol=1e-3, maxit=90)
        assert i1[0]["iters"] == its[q] and torch.equal(x1[0], x[q]), q
    x2, _ = s.solve(bt[:2], tol=1e-3, maxit=90)
    assert torch.equal(x2, x[:2])
    s.close()
    s = ElasticHelmholtz(n, h, vp, vs, rho, omega, drop_converged=False, **kw)
    xn, info = s.solve(bt, tol=1e-3, maxit=90)
    assert [i["iters"] for i in info] == its and torch.equal(xn, x)
    s.close()
