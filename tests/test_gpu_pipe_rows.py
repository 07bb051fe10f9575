"""Every slab-pipeline setting computes the same step bit for bit on boxes whose
one-plane slabs hold 8 or 12 grid rows, fewer than a workgroup of the packed
product pass takes at 64 points (16).
"""
import numpy as np
import pytest
import torch

from gpu_util import say, to_dev
from paper_1003_4322_amd import synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dt", ["f64", "f32"])
@pytest.mark.parametrize("form,prune", [(0, 0), (0, 1), (1, 1)])
@pytest.mark.parametrize("mhd", [False, True], ids=["ns", "mhd"])
@pytest.mark.parametrize("n", [(64, 8, 16), (64, 12, 8), (128, 12, 16)], ids=lambda n: "x".join(map(str, n)))
def test_pipe_rows_bitwise(n, mhd, form, prune, dt):
    from paper_1003_4322_amd import binding as B
    say("pipe rows", n, mhd, form, prune, dt)
    u = synth.random_grid(*n, 41, 0.3 * n[0])
    z = u
    if mhd:
        b = synth.random_grid(*n, 42, 0.3 * n[0])
        z = np.concatenate([u + b, u - b])
    z = to_dev(z, dt)
    p = B.Plan(nfields=6 if mhd else 3, dtype=dt, grid=n)
    p.set_variant("form", form)
    p.set_variant("prune", prune)
    ref = None
    for v in range(p.variant_count("pipe")):
        p.set_variant("pipe", v)
        s = z.clone()
        p.rk2_step(s, B.PS_MHD if mhd else B.PS_NS, 1e-3, 5e-4, 1e-3, 2)
        bits = torch.view_as_real(s).view(torch.int64 if dt == "f64" else torch.int32)
        if ref is None:
            ref = bits.clone()
            assert bool(torch.isfinite(torch.view_as_real(s)).all())
        else:
            assert torch.equal(bits, ref), v
    p.close()
