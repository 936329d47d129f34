"""The fine-level operators as the set-up kernels build them (needs an
MI355X), on grids where every point is next to a boundary, with absorbing
layers wider than the grid and on single sides, in both variants of A_p."""
import numpy as np
import pytest

from oracle.elastic import ElasticSystem
from oracle.precond import BlockAcoustic

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,abc,sides", [
    ((2, 2), 0, 0b1111),
    ((3, 5), 4, 0b1111),
    ((257, 2), 3, 0b0100),
    ((2, 130), 200, 0b0001),
    ((2, 2, 2), 1, 0b111111),
    ((3, 2, 5), 3, 0b010010),
    ((9, 17, 4), 2, 0b100000),
])
@pytest.mark.parametrize("variant", ["A_p", "tilde"])
@pytest.mark.parametrize("precision", [32, 64])
def test_fine_operators(n, abc, sides, variant, precision):
    """H and every shifted block against the oracle's assembled matrices,
    entry sums of at most 2d + 1 products: 1e-13 relative in FP64, 1e-6 for
    coefficients rounded to FP32."""
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2411_15897_amd import ElasticHelmholtz
    rng = np.random.default_rng(4)
    shape, h, alpha = tuple(reversed(n)), tuple(1.0 - 0.2 * a for a in range(len(n))), 0.35
    vp = rng.uniform(2.0, 3.5, shape)
    vs, rho = vp * rng.uniform(0.35, 0.55, shape), rng.uniform(1.0, 2.0, shape)
    s = ElasticHelmholtz(n, h, vp, vs, rho, 0.8, levels=1, alpha=alpha, abc_width=abc, abc_sides=sides,
                         ap_variant=variant, mg_precision=precision)
    o = ElasticSystem(n, h, vp, vs, rho, 0.8, abc, sides)

    def check(got, ref, tol):
        assert np.linalg.norm(got.cpu().numpy() - ref) <= tol * np.linalg.norm(ref)

    x = rng.standard_normal(s.ndof) + 1j * rng.standard_normal(s.ndof)
    check(s.apply_operator(torch.from_numpy(x).cuda()), o.H() @ x, 1e-13)
    ref = BlockAcoustic(o, alpha=alpha, solver="exact", tilde_Ap=variant == "tilde")
    for b in range(len(n) + 1):
        X = ref.Hp if b == len(n) else ref.blocks[b]
        v = rng.standard_normal(X.shape[0]) + 1j * rng.standard_normal(X.shape[0])
        check(s.block_apply(b, 0, torch.from_numpy(v).cuda()), X @ v, 1e-13 if precision == 64 else 1e-6)
    s.close()
