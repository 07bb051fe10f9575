"""The packed product pass at the lengths where a wave holds several transforms
or a transform several waves, on grids with few rows: row counts that are not a
multiple of a workgroup's, and one-plane slabs of eight rows, fewer than a
workgroup takes at 64 points.  The nonlinear term against the oracle; the tolerance is
the parity tests' bar (FP64 1e-12, FP32 2e-5).
"""
import numpy as np
import pytest

from gpu_util import host, rel_l2, rounded, say, to_dev
from paper_1003_4322_amd import synth

pytestmark = pytest.mark.gpu

TOL = {"f64": 1e-12, "f32": 2e-5}

# (nx, ny, nz, pipe): 64 points: 8 threads a transform, 16 rows a workgroup
# (12 x 8 = 96 rows fill it, one-plane slabs of 8 do not); 96, 192 and 384: a
# transform's threads straddle waves; 512 and 1024: one and two waves each
CASES = [(64, 8, 8, 4), (64, 12, 8, 0), (96, 8, 12, 0), (128, 12, 8, 4), (192, 8, 12, 0), (256, 8, 8, 0),
         (384, 8, 8, 0), (512, 8, 8, 4), (1024, 8, 8, 0)]


@pytest.mark.parametrize("dt", ["f64", "f32"])
@pytest.mark.parametrize("form", [0, 1])
@pytest.mark.parametrize("prune", [0, 1])
@pytest.mark.parametrize("mhd", [False, True], ids=["ns", "mhd"])
@pytest.mark.parametrize("case", CASES, ids=lambda c: "%dx%dx%d-pipe%d" % c)
def test_xprod_rows(ref, case, mhd, prune, form, dt):
    from paper_1003_4322_amd import binding as B
    nx, ny, nz, pipe = case
    if mhd and dt == "f64" and nx > 512:
        pytest.skip("MHD in FP64 has rows of at most 512 points")
    say("xprod rows", case, mhd, prune, form, dt)
    n = (nx, ny, nz)
    u = synth.random_grid(*n, 31, 0.4 * nx)
    z = u
    if mhd:
        b = synth.random_grid(*n, 32, 0.4 * nx)
        z = np.concatenate([u + b, u - b])
    z = rounded(z, dt)
    p = B.Plan(nfields=6 if mhd else 3, dtype=dt, grid=n)
    for k, v in (("prune", prune), ("form", form), ("pipe", pipe)):
        p.set_variant(k, v)
    zd = to_dev(z, dt)
    got = host(p.nonlinear_mhd(zd) if mhd else p.nonlinear_ns(zd))
    want = ref.nonlinear_mhd(z) if mhd else ref.nonlinear_ns(z)
    assert rel_l2(got, want) < TOL[dt], rel_l2(got, want)
    p.close()
