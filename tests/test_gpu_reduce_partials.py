"""Sums of the copies of a gradient, below and above the 16 384 floats from which a workgroup takes twice as many: counts that do not fill the
last workgroup, few copies and many."""
import pytest

import workloads as W
from test_gpu_many_tiles import SMALL, check_tiled_gradient

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def M():
    import paper_2107_01460_amd as m
    return m


@pytest.fixture(scope="module")
def orc():
    import oracle
    return oracle


# W2 and b2 of 96 units: 9312 floats, of 160: 25 760, of 416: 173 472; W3, b3 and the statistics of 96 units and six outputs: 587.  128
# units and 27 inputs: one range of 20 877 floats
@pytest.mark.parametrize("ha,hc,view", [(96, 160, 7), (416, 128, 3)])
@pytest.mark.parametrize("copies", [1, 643])
def test_gradient(M, orc, ha, hc, view, copies):
    check_tiled_gradient(M, orc, W.scaled(W.CONFIGS[1], actor_hidden=ha, critic_hidden=hc, view=view, **SMALL), copies)
