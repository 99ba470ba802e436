"""Default cache hints of a plan, by the size of its workspace and of its kx slabs."""

import pytest

import paper_1501_04438_amd as gs

# n, slab_planes (0: one slab), hint bits: none up to 20 MB of X2, P4 and P5 up to 160 MB, beyond and
# where a slab of such a plan is at most 20 MB, P1, P2, P4 and P5
CASES = [(32, 0, 0), (32, 8, 0), (80, 0, 0), (80, 20, 0), (96, 0, 24), (96, 24, 27), (96, 70, 27), (112, 60, 24), (112, 30, 27)]


@pytest.mark.parametrize("n,planes,bits", CASES)
def test_hints_of_slabs(n, planes, bits):
    p = gs.Plan("gaussian_sum", n=n, L=3.0, d=3, custom=([0.7], [1.3]), host_only=True, slab_planes=planes)
    assert p.info["hint_bits"] == bits


def test_chosen_hints_stay():
    kw = dict(n=96, L=3.0, d=3, custom=([0.7], [1.3]), host_only=True, slab_planes=24)
    assert gs.Plan("gaussian_sum", hint_bits=8, **kw).info["hint_bits"] == 8
    assert gs.Plan("gaussian_sum", n=(64, 96), L=3.0, d=2, custom=([0.7], [1.3]), host_only=True).info["hint_bits"] == 24
