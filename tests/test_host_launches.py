"""The host code's choice of kernels and launches, over a HIP runtime that only
records (fake_hip.py): no GPU needed.
"""
import pytest

import fake_hip


@pytest.fixture(scope="module")
def fake(tmp_path_factory):
    from paper_1003_4322_amd import build
    import os
    if not os.path.exists(build.LIB):
        build.build()
    return fake_hip.library(tmp_path_factory.mktemp("fake"))


# grids whose one-plane slabs hold 8 or 12 rows: every slab of a box runs the
# kernels that the whole box runs (the results of every "pipe" setting agree bit
# for bit, so the kernel must not follow the launch's size)
@pytest.mark.parametrize("grid", [(64, 8, 16), (64, 12, 8), (96, 8, 12), (128, 12, 16), (192, 8, 8), (256, 8, 8)])
def test_slabs_run_the_same_kernels(fake, grid):
    fake_hip.run(fake, f"""
for nf in (3, 6):
    for f64 in (False, True):
        for prune in (0, 1):
            for form in (0, 1):
                h = plan({grid}, nf, f64, prune=prune, form=form)
                check(L.ps_plan_set_graphs(h, 0))
                kernels = []
                for v in range(L.ps_plan_variant_count(h, b"pipe")):
                    check(L.ps_plan_set_variant(h, b"pipe", v))
                    F.fake_reset()
                    check(step(h, nf))
                    kernels.append({{l[0] for l in launches()}})
                    assert len(kernels[-1]) == len(kernels[0]) and kernels[-1] == kernels[0], (nf, f64, prune, form, v)
                check(L.ps_plan_destroy(h))
""")


def test_tuner_may_choose_the_untuned_slabs(fake):
    """An unpruned plan takes in-order slabs by itself (NS 256^3 FP64: four); the
    tuner has that count among its candidates, and the choice can be set and read
    back.  Launches cost their threads, several times more where a launch exceeds
    a limit (the cache), and a fixed overhead."""
    fake_hip.run(fake, """
def shape(h):
    F.fake_reset()
    check(step(h, 3))
    return [(l[1], l[2]) for l in launches()]

def tuned(limit, slow, overhead, **v):
    h = plan(256, 3, True, **v)
    check(L.ps_plan_set_graphs(h, 0))
    untuned = shape(h)
    F.fake_cost(limit, slow, overhead)
    check(L.ps_plan_autotune(h, STATE, 0, 1))
    F.fake_cost(1e30, 1, 0)
    return h, untuned, shape(h), L.ps_plan_get_variant(h, b"pipe")

# slabs of a quarter fit, and every launch costs a little: the untuned count is best
h, untuned, got, pipe = tuned(3e6, 4.0, 0.1)
assert len(untuned) == 2 * (2 + 3 * 4), len(untuned)
assert pipe == 10 and len(got) == len(untuned), (pipe, len(got))
check(L.ps_plan_set_variant(h, b"pipe", 0))
assert len(shape(h)) == 10
check(L.ps_plan_set_variant(h, b"pipe", pipe))
assert len(shape(h)) == len(untuned)
# nothing to gain from slabs; only smaller ones fit
assert tuned(1e30, 1.0, 0.1)[3] == 0
assert tuned(2e5, 9.0, 0.0)[3] in (5, 6)
# pruned plans run one slab by themselves
h = plan(256, 3, True, prune=1, pipe=10)
check(L.ps_plan_set_graphs(h, 0))
assert len(shape(h)) == 10
""")


def test_failed_tuning_leaves_the_plan(fake):
    """A tuning run that fails at any launch leaves variants and slabs as they were."""
    fake_hip.run(fake, """
kinds = [b"y", b"z", b"z_curl", b"z_epi", b"x_prod", b"pipe"]
h = plan(256, 3, True)
check(L.ps_plan_set_graphs(h, 0))
def state():
    F.fake_reset()
    check(step(h, 3))
    return [L.ps_plan_get_variant(h, k) for k in kinds], [l[:3] for l in launches()]
before = state()
F.fake_reset()
g = plan(256, 3, True)
check(L.ps_plan_autotune(g, STATE, 0, 1))
total = len(launches())
assert total > 100
for n in sorted({0, 1, 10, 60, total - 200, total - 100, total - 1}):
    F.fake_reset()
    F.fake_fail_launch(n)
    assert L.ps_plan_autotune(h, STATE, 0, 1) != 0, n
    assert state() == before, n
F.fake_reset()
check(L.ps_plan_autotune(h, STATE, 0, 1))
""")


@pytest.mark.parametrize("where", ["begin", "end", "instantiate"])
def test_failed_capture_behind_a_step(fake, where):
    """The graph is captured behind a step that has run: where that fails, the call
    still takes its steps, kernel by kernel, and a later call captures.  A capture
    that comes first (slabs on helper streams) fails the call before any launch."""
    fake_hip.run(fake, f"""
where = {["begin", "end", "instantiate"].index(where)}
def fail_once():
    F.fake_reset()
    F.fake_fail(*[int(i == where) for i in range(3)])
def done():
    return sum(not l[4] for l in launches()), F.fake_replays()
h = plan(96, 3)
check(L.ps_plan_set_graphs(h, 0))
check(step(h, 3))
per = len(launches())
check(L.ps_plan_set_graphs(h, 1))
# several steps in a call; then the capture succeeds behind the next call's first
fail_once()
check(step(h, 3, 4))
assert done() == (4 * per, 0), done()
assert F.fake_last_error() == 0
F.fake_reset()
check(step(h, 3, 3))
assert done() == (per, 2), done()
# one-step calls: the second tries to capture
F.fake_reset()
check(step(h, 3, 1, state=2 * STATE))
fail_once()
check(step(h, 3, 1, state=2 * STATE))
assert done() == (per, 0), done()
F.fake_reset()
check(step(h, 3, 1, state=2 * STATE))
check(step(h, 3, 1, state=2 * STATE))
assert done() == (per, 1), done()
# slabs on helper streams: nothing has run when the call fails
check(L.ps_plan_set_variant(h, b"pipe", 8))
fail_once()
assert step(h, 3, 2) != 0
assert done() == (0, 0), done()
F.fake_reset()
check(step(h, 3, 2))
assert done() == (0, 2), done()
""")


def test_ensembles_past_one_launch(fake):
    """A launch holds fewer than 2^32 threads. Ensembles of small boxes whose plane
    kernels would need more (1.5 million boxes of 8^3, NS 94 GB of FP32 workspace)
    run them in several launches that take every plane once."""
    fake_hip.run(fake, """
for n, nb, nf in ((8, 1500000, 3), (8, 1500000, 6)):
    h, small = plan([n] * nb, nf), plan([n] * 1000, nf)
    check(L.ps_plan_set_graphs(h, 0))
    check(L.ps_plan_set_graphs(small, 0))
    def blocks(f, *a):
        F.fake_reset()
        check(f(*a))
        n = {}
        for l in launches():
            n[l[0]] = n.get(l[0], 0) + l[1]
        return n
    for f, a in ((L.ps_fft_r2c, (STATE, 2 * STATE)), (L.ps_fft_c2r, (STATE, 2 * STATE)),
                 (step, (nf,)), (L.ps_nonlinear_mhd if nf == 6 else L.ps_nonlinear_ns, (STATE, 2 * STATE))):
        big, ref = blocks(f, h, *a), blocks(f, small, *a)
        for k, m in big.items():
            if k in ref:  # (few boxes may run other kernels of a pass)
                assert m * 1000 == ref[k] * nb, (n, nf, f, m, ref[k])
    check(L.ps_plan_destroy(h))
""")


# FP64 rows of 128 and 192 points, whose product kernel is chosen by form and rows:
# workgroups and threads of the launch on one cube
@pytest.mark.parametrize("n,nf,form,launch", [(128, 6, 0, (8192, 192)), (128, 3, 0, (2048, 192)),
                                              (128, 3, 1, (4096, 160)), (192, 6, 0, (36864, 144))])
def test_product_kernel_fp64(fake, n, nf, form, launch):
    """Rotational MHD and the NS divergence form take the half-length form (one or
    two rows a workgroup), rotational NS at 128 the packed one in radix 16."""
    fake_hip.run(fake, f"""
h = plan({n}, {nf}, True, form={form}, pipe=0)
check(L.ps_plan_set_graphs(h, 0))
F.fake_reset()
check(step(h, {nf}))
assert launches()[2][1:3] == {launch}, launches()[2]
""")


# (boxes, fields, FP64, form, prune, pass, variant): each side of the lines of the
# default variants, where a variant measured at 512 points or on large boxes is
# the slower one
@pytest.mark.parametrize("dims,nf,f64,form,prune,kind,want", [
    ((48, 64, 768), 6, 0, 1, 1, "z_epi", 5), (768, 6, 0, 1, 1, "z_epi", 5), ((96, 384, 768), 6, 1, 1, 0, "z_epi", 5),
    ((48, 64, 1024), 6, 0, 1, 1, "z_epi", 5), ((16, 24, 1024), 3, 0, 0, 0, "z_epi", 0),
    ((48, 64, 512), 6, 0, 1, 0, "z_epi", 5), (512, 6, 0, 1, 1, "z_epi", 12),
    ((48, 64, 384), 6, 0, 0, 0, "z_epi", 5), ((16, 24, 384), 6, 0, 0, 0, "z_epi", 12), (384, 6, 0, 0, 0, "z_epi", 12),
    ((16, 24, 384), 6, 1, 0, 1, "z_epi", 5), (384, 6, 1, 0, 0, "z_epi", 0),
    (512, 3, 0, 1, 1, "z_epi", 2), ((16, 24, 512), 3, 0, 1, 1, "z_epi", 9), ((16, 24, 512), 3, 1, 0, 0, "z_epi", 2),
    ((256, 192, 768), 3, 1, 0, 0, "z_curl", 0), ((256, 192, 768), 6, 1, 1, 0, "z_curl", 0),
    ((16, 24, 768), 6, 1, 0, 0, "z_curl", 5), ((96, 384, 1024), 6, 0, 0, 0, "z_curl", 0),
    ((16, 24, 512), 3, 0, 0, 0, "z_curl", 0), (512, 3, 0, 0, 0, "z_curl", 6),
    ((48, 64, 256), 3, 1, 0, 1, "z_curl", 0), (256, 3, 1, 0, 1, "z_curl", 6),
])
def test_default_variants_by_size(fake, dims, nf, f64, form, prune, kind, want):
    fake_hip.run(fake, f"""
h = plan({dims}, {nf}, {f64}, form={form}, prune={prune})
assert L.ps_plan_get_variant(h, b"{kind}") == {want}, L.ps_plan_get_variant(h, b"{kind}")
""")


def test_inverse_z_pass_of_many_columns(fake):
    """Twelve boxes of MHD 64^3 FP32 have 25344 columns: one field after another (a
    workgroup for each tile of 8 columns), not one workgroup per field and tile; one
    box has 2112 and goes field by field."""
    fake_hip.run(fake, """
for nb, blocks in ((12, 12 * 64 * 5), (1, 12 * 64 * 5)):
    h = plan([64] * nb, 6)
    check(L.ps_plan_set_graphs(h, 0))
    F.fake_reset()
    check(step(h, 6))
    assert launches()[0][1] == blocks, (nb, launches()[0])
""")
