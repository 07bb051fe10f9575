"""The spectra's sums stay compensated to the end: a total is the sum of its shells
and a shell the sum of its planes, to the last place, also where terms of both
signs cancel (the cross-helicity).

Tolerance of a total: a compensated sum of n terms is within u |S| + (n u)^2
sum |terms| of the exact sum S of the returned shells (u = 2^-53), and one more u
for the sum of value and compensation.
"""
import math

import numpy as np
import pytest

from gpu_util import host, say, to_dev
from paper_1003_4322_amd import synth

pytestmark = pytest.mark.gpu

U = 2.0 ** -53


def close_to_sum(total, terms):
    s = math.fsum(terms)
    return abs(total - s) <= 2 * U * abs(s) + (len(terms) * U) ** 2 * math.fsum(np.abs(terms))


# 29, 84, 167 and 361 shells: one workgroup in the final sums, and several
@pytest.mark.parametrize("dt", ["f64", "f32"])
@pytest.mark.parametrize("n", [(32, 32, 32), (96, 96, 96), (192, 192, 192), (16, 768, 96)],
                         ids=lambda n: "x".join(map(str, n)))
def test_totals_of_cancelling_shells(n, dt):
    from paper_1003_4322_amd import binding as B
    say("spectrum totals", n, dt)
    nx, ny, nz = n
    rng = np.random.default_rng(nx + ny + nz)
    wave = [np.where(np.arange(m) < m // 2, np.arange(m), np.arange(m) - m).astype(np.int64) for m in (nz, ny)]
    k2 = wave[0][:, None, None] ** 2 + wave[1][None, :, None] ** 2 + np.arange(nx // 2 + 1, dtype=np.int64) ** 2
    sh = synth.shell_index(k2)
    p = B.Plan(nfields=6, dtype=dt, grid=n)
    ns = p.nshells[0]
    u = rng.standard_normal((3, nz, ny, nx // 2 + 1)) + 1j * rng.standard_normal((3, nz, ny, nx // 2 + 1))
    u *= np.exp(-3.0 * sh / ns)
    # b = c_s u: Hc(s) = 2 c_s Eu(s), of both signs, cancelling to about 1e-6
    eu = host(p.energy_spectrum(to_dev(u, dt), 3)[0])
    c = rng.choice([-0.5, 0.5], ns) * rng.uniform(0.5, 1.0, ns)
    big = int(np.argmax(eu))
    c[big] -= float(np.dot(c, eu)) / eu[big]
    c[big] *= 1 + 1e-6
    b = c[sh] * u
    spec, tot = (host(x) for x in p.mhd_spectrum(to_dev(np.concatenate([u + b, u - b]), dt)))
    say("cancellation", abs(tot[2]) / np.abs(spec[2]).sum())
    for q in range(3):
        assert close_to_sum(tot[q], spec[q]), (q, tot[q] - math.fsum(spec[q]), np.abs(spec[q]).sum())
    spec, tot = (host(x) for x in p.energy_spectrum(to_dev(np.concatenate([u, b]), dt)))
    assert close_to_sum(tot[0], spec)
    p.close()


@pytest.mark.parametrize("dt", ["f64", "f32"])
def test_shell_sum_over_planes_is_compensated(dt):
    """Shell 40 of a 96 x 24 x 128 box: cross-helicity terms 2^60 on plane kz = 1,
    1 on kz = 33 (added by the same thread) and -2^60 on kz = 2 leave 1."""
    from paper_1003_4322_amd import binding as B
    say("spectrum planes", dt)
    z = np.zeros((6, 128, 24, 49), np.complex128)
    z[0, 1, 9, 39] = 2.0 ** 31   # u = b = 2^30
    z[0, 33, 5, 22] = 2.0        # u = b = 1
    z[3, 2, 9, 39] = 2.0 ** 31   # u = -b = 2^30
    p = B.Plan(nfields=6, dtype=dt, grid=(96, 24, 128))
    spec, tot = (host(x) for x in p.mhd_spectrum(to_dev(z, dt)))
    assert spec[2][40] == 1.0 and tot[2] == 1.0, (spec[2][40], tot[2])
    assert np.count_nonzero(spec[2]) == 1
    p.close()
