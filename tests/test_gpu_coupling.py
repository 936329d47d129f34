"""The coupling g = r_u - B^T e_p formed in the shear blocks' fine down leg
against its own launch (needs an MI355X): the number of cells times right-
hand sides decides, so a batch on one side of the rule is compared with its
right-hand sides alone on the other side."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,levels,nrhs", [
    ((264, 200), 3, 20),      # alone: in the leg, 20: its own launch; partial tiles
    ((2, 1024), 2, 513),      # a grid of one cell less than a tile in x
    ((512, 512), 5, 5),       # 4 would still be in the leg
    ((1056, 1024), 6, 16),    # alone: its own launch, 16: in the leg
])
@pytest.mark.parametrize("precision", [32, 64])
@pytest.mark.parametrize("intergrid", ["full", "mixed"])
def test_coupling_routes_bitwise(n, levels, nrhs, precision, intergrid):
    """Same arithmetic per point: bitwise equal."""
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2411_15897_amd import ElasticHelmholtz
    rng = np.random.default_rng(3)
    shape = tuple(reversed(n))
    vp = rng.uniform(2.0, 3.5, shape)
    s = ElasticHelmholtz(n, (1.0, 0.9), vp, 0.5 * vp, rng.uniform(1.0, 2.0, shape), 0.6, levels=levels, alpha=0.5,
                         mg_precision=precision, intergrid=intergrid, abc_width=4)
    r = torch.randn(nrhs, s.ndof, dtype=torch.complex128, device="cuda",
                    generator=torch.Generator("cuda").manual_seed(1))
    z = s.apply_preconditioner(r)
    assert bool(torch.isfinite(torch.view_as_real(z)).all())
    for q in (0, nrhs // 2, nrhs - 1):
        assert torch.equal(z[q], s.apply_preconditioner(r[q:q + 1])[0])
    s.close()
