"""Shell spectra at the edges of the kernel's enumeration: planes and rows that
are their own mirror image, rows longer and shorter than a 64-mode chunk,
shell counts next to a window's end, one and several workgroups in the final
sums, and every field count, on white fields against the oracle.

Tolerance: every term is positive and enters through at most six scan levels
and compensated sums, so a shell's relative error is a few ulp (1e-13 leaves a
factor of 100); a divergence is a sum of three products (1e-12 relative).
"""
import numpy as np
import pytest

from gpu_util import host, rounded, say, to_dev

pytestmark = pytest.mark.gpu

# 8 x 8 x 8: rows shorter than a wave; 128 x 8 x 12: 65 modes a row; 8 x 192 x 96:
# short rows, many orbits, two windows; 256 x 64 x 8: rows of several chunks;
# 64 x 64 x 96: 66 shells; 192 x 192 x 192: 167 shells, several final workgroups
GRIDS = [(8, 8, 8), (128, 8, 12), (8, 192, 96), (256, 64, 8), (64, 64, 96), (192, 192, 192)]


@pytest.mark.parametrize("dt", ["f64", "f32"])
@pytest.mark.parametrize("n", GRIDS, ids=lambda n: "x".join(map(str, n)))
def test_spectrum_edges(ref, n, dt):
    from paper_1003_4322_amd import binding as B
    say("spectrum edges", n, dt)
    nx, ny, nz = n
    rng = np.random.default_rng(nx + 7 * ny + 13 * nz)
    s = (6, nz, ny, nx // 2 + 1)
    F = rounded(rng.standard_normal(s) + 1j * rng.standard_normal(s), dt)
    p = B.Plan(nfields=6, dtype=dt, grid=n)
    for nf in (1, 2, 3, 4, 5, 6):
        f = np.ascontiguousarray(F[:nf])
        spec, tot = p.energy_spectrum(to_dev(f, dt), nf)
        stat = p.energy_spectrum_static(to_dev(f, dt), nf)
        ws, wt = ref.energy_spectrum(f)
        assert np.allclose(host(spec), ws, rtol=1e-13, atol=0), nf
        assert np.allclose(host(tot), wt, rtol=1e-12, atol=0), nf
        assert np.array_equal(host(stat[0]), host(spec)) and np.array_equal(host(stat[1]), host(tot)), nf
    spec, tot = p.mhd_spectrum(to_dev(F, dt))
    ws, wt = ref.mhd_spectrum(F)
    scale = ws[0] + ws[1]  # the cross-helicity's terms have both signs
    assert (np.abs(host(spec) - ws) <= 1e-13 * scale[None, :]).all()
    assert np.abs(host(tot) - wt).max() <= 1e-13 * (wt[0] + wt[1])
    p.close()
