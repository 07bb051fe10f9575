"""Plain transforms of rows of 8 points on grids whose planes are no squares: 256
row pairs a workgroup, copied through LDS, with pair counts below, at and beyond
whole workgroups and workgroups that span several fields.  Against the oracle at the
bars of the plain transforms (relative L2 1e-13 and 2e-6).
"""
import numpy as np
import pytest

from gpu_util import host, rel_l2, rounded, say, to_dev

pytestmark = pytest.mark.gpu

TOL = {"f64": 1e-13, "f32": 2e-6}


# 48, 256 and 288 pairs a field; 16 x 1024 pairs
@pytest.mark.parametrize("dt", ["f64", "f32"])
@pytest.mark.parametrize("nf", [3, 6])
@pytest.mark.parametrize("n", [(8, 12, 8), (8, 64, 8), (8, 48, 12), (8, 1024, 32)], ids=lambda n: "x".join(map(str, n)))
def test_rows_of_eight(ref, n, nf, dt):
    from paper_1003_4322_amd import binding as B
    say("rows of eight", n, nf, dt)
    nx, ny, nz = n
    rng = np.random.default_rng(ny + nz + nf)
    u = rounded(rng.standard_normal((nf, nz, ny, nx)), dt)
    s = (nf, nz, ny, nx // 2 + 1)
    X = rounded(rng.standard_normal(s) + 1j * rng.standard_normal(s), dt)
    p = B.Plan(nfields=nf, dtype=dt, grid=n)
    got, want = host(p.fft_r2c(to_dev(u, dt, "r"))), ref.fft_r2c(u)
    assert rel_l2(got, want) < TOL[dt], rel_l2(got, want)
    got, want = host(p.fft_c2r(to_dev(X, dt))), ref.fft_c2r(X)
    assert rel_l2(got, want) < TOL[dt], rel_l2(got, want)
    p.close()
