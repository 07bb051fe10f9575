"""The plain transforms against the oracle where the kernels change: planes that
live in LDS (nx = ny up to 96), the separate x pass at lengths whose transforms
share a wave, straddle waves or span several, odd numbers of planes per launch
and ensembles.  Tolerances as in the parity tests (relative L2 1e-13 and 2e-6).
The inverse is fed spectra that are not Hermitian on kx = 0 and N/2, whose
imaginary parts the pass-order convention drops.
"""
import numpy as np
import pytest
import torch

from gpu_util import CDT, DEV, RDT, host, rel_l2, rounded, say, to_dev

pytestmark = pytest.mark.gpu

TOL = {"f64": 1e-13, "f32": 2e-6}

GRIDS = [(8, 8, 12), (12, 12, 8), (16, 16, 24), (24, 24, 8), (32, 32, 16), (48, 48, 8), (64, 64, 12), (96, 96, 8),
         (128, 128, 8), (12, 8, 16), (96, 8, 8), (192, 12, 8), (256, 8, 8), (384, 8, 12), (768, 8, 8), (1024, 8, 8)]


@pytest.mark.parametrize("dt", ["f64", "f32"])
@pytest.mark.parametrize("nf", [3, 6])
@pytest.mark.parametrize("n", GRIDS, ids=lambda n: "x".join(map(str, n)))
def test_plain_fft(ref, n, nf, dt):
    from paper_1003_4322_amd import binding as B
    say("plain fft", n, nf, dt)
    nx, ny, nz = n
    rng = np.random.default_rng(nx + ny + nz + nf)
    u = rounded(rng.standard_normal((nf, nz, ny, nx)), dt)
    s = (nf, nz, ny, nx // 2 + 1)
    X = rounded(rng.standard_normal(s) + 1j * rng.standard_normal(s), dt)
    p = B.Plan(nfields=nf, dtype=dt, grid=n)
    got, want = host(p.fft_r2c(to_dev(u, dt, "r"))), ref.fft_r2c(u)
    assert rel_l2(got, want) < TOL[dt], rel_l2(got, want)
    xd = to_dev(X, dt)
    got, want = host(p.fft_c2r(xd)), ref.fft_c2r(X)
    assert rel_l2(got, want) < TOL[dt], rel_l2(got, want)
    assert np.array_equal(host(xd), X)  # the input is preserved
    p.close()


@pytest.mark.parametrize("dt", ["f64", "f32"])
def test_plain_fft_ensemble(ref, dt):
    from paper_1003_4322_amd import binding as B
    sizes = [32, 32, 96, 128]
    say("plain fft ensemble", sizes, dt)
    p = B.Plan(sizes, 3, dt)
    rng = np.random.default_rng(5)
    us = [rounded(rng.standard_normal((3, n, n, n)), dt) for n in sizes]
    flat = torch.cat([to_dev(u, dt, "r").reshape(-1) for u in us])
    X = p.fft_r2c(flat)
    back = host(p.fft_c2r(X))
    X = host(X)
    for b, u in enumerate(us):
        want = ref.fft_r2c(u)
        got = X[p.cplx_off[b]:p.cplx_off[b] + want.size].reshape(want.shape)
        assert rel_l2(got, want) < TOL[dt], (b, rel_l2(got, want))
        r = back[p.real_off[b]:p.real_off[b] + u.size].reshape(u.shape) / sizes[b] ** 3
        assert rel_l2(r, u) < 2 * TOL[dt], b
    p.close()
