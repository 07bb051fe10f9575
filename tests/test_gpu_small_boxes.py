"""Small boxes against the oracle on flat inputs: planes that live in LDS (both
kernels), z passes with the fields side by side, and the rules that choose
them, on either side of each line.

* nx = ny at every length with a plane schedule, nz of another length, pruned
  and not, NS and MHD in both forms, FP32 and FP64: the nonlinear term (which
  writes zeros outside the sphere) and two RK2 steps, rotating.
* nx != ny: the three separate passes.
* Ensembles with fewer and with more planes than CUs, and enough columns for
  the z passes to take the fields one after another.

Tolerances are relative L2 errors over all fields: FP64 1e-12 (2e-12 after the two
steps); FP32 2e-5 for the nonlinear term, 4e-6 after the two steps and 2e-6 for an
ensemble's boxes.
"""
import numpy as np
import pytest
import torch

from gpu_util import CDT, DEV, host, rel_l2, rounded, say, to_dev
from oracle.psref import MHD, NS
from paper_1003_4322_amd import synth

pytestmark = pytest.mark.gpu

TOL_NL = {"f64": 1e-12, "f32": 2e-5}
TOL_STEP = {"f64": 1e-12, "f32": 2e-6}
OMEGA = (1.5, -2.0, 3.0)


@pytest.fixture(scope="module")
def B():
    from paper_1003_4322_amd import binding
    binding.lib()
    return binding


def fields(n, mhd, seed):
    """Solenoidal, truncated, every kept mode of order one."""
    k0 = 0.6 * max(n)
    u = synth.random_grid(*n, seed, k0)
    if not mhd:
        return u
    b = synth.random_grid(*n, seed + 50, k0)
    return np.concatenate([u + b, u - b])


def kept(n):
    """The 2/3 rule on [kz][ky][kx], in integers."""
    m = int(np.lcm.reduce(n))
    k = [np.fft.fftfreq(a, 1.0 / a).astype(np.int64) * (m // a) for a in n]
    kx = np.arange(n[0] // 2 + 1) * (m // n[0])
    return 9 * (kx[None, None, :] ** 2 + k[1][None, :, None] ** 2 + k[2][:, None, None] ** 2) < m * m


# every plane length, with another z length (12: fewer points than a wave holds
# columns; 96 and 128: the longest side-by-side z passes)
GRIDS = [(8, 8, 12), (12, 12, 8), (16, 16, 48), (24, 24, 96), (32, 32, 24), (48, 48, 64), (64, 64, 16), (24, 24, 128)]


@pytest.mark.parametrize("dt", ["f64", "f32"])
@pytest.mark.parametrize("form", [0, 1])
@pytest.mark.parametrize("prune", [0, 1])
@pytest.mark.parametrize("mhd", [False, True], ids=["ns", "mhd"])
@pytest.mark.parametrize("n", GRIDS + [(32, 48, 16)], ids=lambda n: "x".join(map(str, n)))
def test_small_grid(B, ref, n, mhd, prune, form, dt):
    say("small grid", n, mhd, prune, form, dt)
    z = rounded(fields(n, mhd, 11), dt)
    p = B.Plan(nfields=6 if mhd else 3, dtype=dt, grid=n)
    p.set_variant("prune", prune)
    p.set_variant("form", form)
    zd = to_dev(z, dt)
    got = host(p.nonlinear_mhd(zd) if mhd else p.nonlinear_ns(zd))
    want = ref.nonlinear_mhd(z) if mhd else ref.nonlinear_ns(z)
    assert rel_l2(got, want) < TOL_NL[dt], rel_l2(got, want)
    assert not got[:, ~kept(n)].any()  # exactly zero outside the sphere
    nu, eta, h = 5e-3, 3e-3, 1e-3
    p.set_rotation(*OMEGA)
    s = host(p.rk2_step(zd, B.PS_MHD if mhd else B.PS_NS, nu, eta, h, 2))
    want = ref.rk2_step(z, MHD if mhd else NS, nu, eta, h, 2, omega=OMEGA)
    assert rel_l2(s, want) < 2 * TOL_STEP[dt], rel_l2(s, want)


# (size, boxes, prune, form): 4 x 64 = 256 planes and 5 x 64 on either side of
# the line between the plane kernels; 8 boxes of 96^3 pruned are 12 856 columns,
# unpruned 37 632 (past the inverse z pass's line); 2 of 128^3 pruned 5 770 (past
# the epilogue's line)
ENSEMBLES = [(64, 4, 1, 1), (64, 5, 1, 1), (96, 8, 0, 0), (96, 2, 1, 1), (128, 2, 1, 1), (128, 1, 1, 1)]


@pytest.mark.parametrize("dt", ["f64", "f32"])
@pytest.mark.parametrize("case", ENSEMBLES, ids=lambda c: "%dx%d-p%d-f%d" % c)
def test_small_ensemble(B, ref, case, dt):
    N, count, prune, form = case
    say("small ensemble", case, dt)
    p = B.Plan([N] * count, 3, dt)
    p.set_variant("prune", prune)
    p.set_variant("form", form)
    zs = [rounded(fields((N, N, N), False, 20 + i), dt) for i in range(min(count, 2))]
    st = torch.empty(p.n_complex(), dtype=CDT[dt], device=DEV)
    for i in range(count):  # two distinct inputs, the last box the second one
        z = zs[i == count - 1] if len(zs) > 1 else zs[0]
        st[p.cplx_off[i]:p.cplx_off[i] + z.size] = torch.from_numpy(z.astype(np.complex64 if dt == "f32" else
                                                                             np.complex128).ravel()).to(DEV)
    p.rk2_step(st, B.PS_NS, 5e-3, 0.0, 1e-3, 1)
    s = host(st)
    wants = [ref.rk2_step(z, NS, 5e-3, 0.0, 1e-3, 1) for z in zs]
    for i in range(count):
        want = wants[i == count - 1] if len(wants) > 1 else wants[0]
        got = s[p.cplx_off[i]:p.cplx_off[i] + want.size].reshape(want.shape)
        assert rel_l2(got, want) < TOL_STEP[dt], (i, rel_l2(got, want))
