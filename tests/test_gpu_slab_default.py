"""In-order slabs that a plan takes by itself (unpruned fields of more than twice
the last-level cache) compute what one slab computes, bit for bit: each plane's
chain is the same arithmetic whichever slab it falls in.  A cube, an ensemble, a
grid whose slabs are uneven, and a box below the line, which stays whole.
"""
import pytest
import torch

from gpu_util import DEV, say

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def B():
    from paper_1003_4322_amd import binding
    binding.lib()
    return binding


# fields of 736, 1189, 1359 and 368 MB: slabs of 230 MB at most, none below three
@pytest.mark.parametrize("dims,nf,slabs", [
    ((192, 192, 192), 6, 4),
    ([96] * 24, 3, 6),
    ((128, 96, 1024), 6, 6),
    ((192, 192, 192), 3, 1),
])
def test_default_slabs_bitwise(B, dims, nf, slabs):
    say("default slabs", dims, nf)
    grid = isinstance(dims, tuple)
    plan = lambda: B.Plan(nfields=nf, dtype="f64", grid=dims) if grid else B.Plan(dims, nf, "f64")  # noqa: E731
    model = B.PS_MHD if nf == 6 else B.PS_NS
    p, q = plan(), plan()
    q.set_variant("pipe", 0)
    g = torch.Generator(device=DEV).manual_seed(7)
    z = 1e-4 * torch.randn(p.n_complex(), generator=g, device=DEV, dtype=torch.complex128)
    a, b = z.clone(), z.clone()
    p.rk2_step(a, model, 1e-3, 5e-4, 1e-4, 2)
    q.rk2_step(b, model, 1e-3, 5e-4, 1e-4, 2)
    assert bool(torch.isfinite(torch.view_as_real(a)).all())
    assert torch.equal(torch.view_as_real(a).view(torch.int64), torch.view_as_real(b).view(torch.int64))
    for r, n in ((p, slabs), (q, 1)):
        r.set_timing(True)
        r.rk2_step(a, model, 1e-3, 5e-4, 1e-4, 1)
        assert r.timings()["x_prod"]["launches"] == 2 * n, r.timings()
        r.close()
