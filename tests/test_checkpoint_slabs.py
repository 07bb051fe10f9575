"""A plan that chooses its z-slabs by itself reads "pipe" 0; a run resumed from its
checkpoint goes on choosing them, and any other setting is restored.
"""
import pytest
import torch

from paper_1003_4322_amd import checkpoint as ck


class _Plan:
    """What apply_variants reads, and the settings it makes."""
    complex_dtype, nfields = torch.complex64, 3

    def __init__(self, pipe):
        self.v, self.set = {"pipe": pipe}, {}

    def n_complex(self):
        return 3 * 8 * 8 * 5

    def variant(self, kind):
        return self.v.get(kind, 0)

    def set_variant(self, kind, value):
        self.set[kind] = value


@pytest.mark.parametrize("saved,now,restored", [(0, 0, {}), (0, 5, {"pipe": 0}), (4, 0, {"pipe": 4}),
                                                (10, 0, {"pipe": 10}), (4, 4, {"pipe": 4})])
def test_resume_keeps_the_plans_own_slabs(saved, now, restored):
    header = {"dtype": "complex64", "nfields": 3, "shape": [3, 8, 8, 5], "variants": {"x_prod": 0, "pipe": saved}}
    p = _Plan(now)
    assert ck.apply_variants(p, header) == {"x_prod": 0, "pipe": saved}
    assert p.set == {"x_prod": 0, **restored}
