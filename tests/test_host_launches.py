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
