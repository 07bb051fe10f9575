"""The epilogue that combines a column's fields before the transform along z,
against the oracle: the variant of the long lengths on few columns (short nx and
ny: the kx = ky = 0 column, a ragged tile and single-row edges are all there) and
the default of 96, 128 and 192 points once the columns are many.  Each case
checks the nonlinear term (zeros outside the sphere, in pruned launches too) and
two rotating steps; tolerances are the parity tests' bars.
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
    u = synth.random_grid(*n, seed, 0.6 * min(n))
    if not mhd:
        return u
    b = synth.random_grid(*n, seed + 50, 0.6 * min(n))
    return np.concatenate([u + b, u - b])


@pytest.mark.parametrize("dt", ["f64", "f32"])
@pytest.mark.parametrize("form", [0, 1])
@pytest.mark.parametrize("prune", [0, 1])
@pytest.mark.parametrize("mhd", [False, True], ids=["ns", "mhd"])
@pytest.mark.parametrize("n", [(24, 8, 256), (16, 12, 384), (16, 8, 512), (12, 8, 768), (16, 8, 1024)],
                         ids=lambda n: "x".join(map(str, n)))
def test_epi_tile_variant(B, ref, n, mhd, prune, form, dt):
    say("epi tile", n, mhd, prune, form, dt)
    z = rounded(fields(n, mhd, 61), dt)
    p = B.Plan(nfields=6 if mhd else 3, dtype=dt, grid=n)
    p.set_variant("prune", prune)
    p.set_variant("form", form)
    p.set_variant("z_epi", p.variant_count("z_epi") - 1)
    zd = to_dev(z, dt)
    out = torch.full_like(zd, 7.0)
    got = host(p.nonlinear_mhd(zd, out) if mhd else p.nonlinear_ns(zd, out))
    want = ref.nonlinear_mhd(z) if mhd else ref.nonlinear_ns(z)
    assert rel_l2(got, want) < TOL_NL[dt], rel_l2(got, want)
    p.set_rotation(*OMEGA)
    s = host(p.rk2_step(zd, B.PS_MHD if mhd else B.PS_NS, 5e-3, 3e-3, 1e-3, 2))
    want = ref.rk2_step(z, MHD if mhd else NS, 5e-3, 3e-3, 1e-3, 2, omega=OMEGA)
    assert rel_l2(s, want) < 2 * TOL_STEP[dt], rel_l2(s, want)
    p.close()


# (size, boxes): pruned columns past 4096, the line to the epilogue by field
@pytest.mark.parametrize("dt", ["f64", "f32"])
@pytest.mark.parametrize("mhd", [False, True], ids=["ns", "mhd"])
@pytest.mark.parametrize("case", [(96, 3), (128, 2), (192, 1)], ids=lambda c: "%dx%d" % c)
def test_epi_tile_default(B, ref, case, mhd, dt):
    N, count = case
    say("epi tile default", case, mhd, dt)
    z = rounded(fields((N, N, N), mhd, 71), dt)
    p = B.Plan([N] * count, 6 if mhd else 3, dt)
    p.set_variant("prune", 1)
    p.set_variant("form", 1)
    st = to_dev(z, dt).reshape(-1).repeat(count)
    got = (p.nonlinear_mhd(st) if mhd else p.nonlinear_ns(st)).view(count, -1)
    assert all(torch.equal(got[0], g) for g in got[1:])
    want = ref.nonlinear_mhd(z) if mhd else ref.nonlinear_ns(z)
    g = host(got[0]).reshape(want.shape)
    assert rel_l2(g, want) < TOL_NL[dt], rel_l2(g, want)
    p.rk2_step(st, B.PS_MHD if mhd else B.PS_NS, 5e-3, 3e-3, 1e-3, 1)
    want = ref.rk2_step(z, MHD if mhd else NS, 5e-3, 3e-3, 1e-3, 1)
    s = host(st.view(count, -1)[count - 1]).reshape(want.shape)
    assert rel_l2(s, want) < TOL_STEP[dt], rel_l2(s, want)
    p.close()
