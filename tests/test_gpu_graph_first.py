"""ps_rk2_step launches the first step of a new state or coefficient kernel by
kernel and replays a graph once the step repeats: every mixture of the two gives,
bit for bit, what plain launches give, with the caller's own work between calls.
"""
import pytest
import torch

from gpu_util import DEV, say

pytestmark = pytest.mark.gpu

# (state, steps, dt): one-step calls that repeat, a change of state, of dt and
# back, several steps in a call
CALLS = [(0, 1, 1e-4), (0, 1, 1e-4), (0, 1, 1e-4), (1, 1, 1e-4), (0, 1, 1e-4), (1, 1, 1e-4), (1, 3, 1e-4),
         (1, 1, 2e-4), (0, 2, 2e-4), (0, 1, 1e-4), (1, 1, 1e-4), (1, 1, 1e-4)]


@pytest.mark.parametrize("pipe", [None, 0, 4, 8])
@pytest.mark.parametrize("dims,nf", [(24, 6), ((16, 96, 64), 3)])
def test_first_steps_bitwise(dims, nf, pipe):
    from paper_1003_4322_amd import binding as B

    say("graph first", dims, nf, pipe)
    plans = [B.Plan(nfields=nf, dtype="f64", grid=dims) if isinstance(dims, tuple) else B.Plan(dims, nf, "f64")
             for _ in range(2)]
    plans[1].set_graphs(False)
    if pipe is not None:
        for p in plans:
            p.set_variant("pipe", pipe)
    g = torch.Generator(device=DEV).manual_seed(3)
    z = [1e-3 * torch.randn(plans[0].n_complex(), generator=g, device=DEV, dtype=torch.complex128)
         for _ in range(2)]
    model = B.PS_MHD if nf == 6 else B.PS_NS
    runs = [[x.clone() for x in z] for _ in plans]
    for i, (k, n, dt) in enumerate(CALLS):
        for p, x in zip(plans, runs):
            p.rk2_step(x[k], model, 1e-3, 5e-4, dt, n)
            x[k].mul_(0.5)  # the caller's own work on the same stream
            if i % 3 == 2:
                torch.cuda.synchronize()
        a, b = (torch.view_as_real(x[k]).view(torch.int64) for x in runs)
        assert torch.equal(a, b), (i, k, n)
    assert all(bool(torch.isfinite(torch.view_as_real(x)).all()) for x in runs[0])
    for p in plans:
        p.close()
