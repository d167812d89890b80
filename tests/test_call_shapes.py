"""What the planner reports of a plan and of its calls, on the CPU."""
import pytest

import workloads as W
from paper_2608_13110_amd import Plan
from tests import helpers as H


@pytest.mark.parametrize("n,d,k", [(10, 20, 3), (9, 25, 0), (9, 33, 4), (20, 40, 6), (14, 48, 8), (12, 61, 5)])
@pytest.mark.parametrize("options", [None, dict(reg_bits=4, math=2)])
def test_info_counts_the_listed_passes(n, d, k, options):
    # n_passes and n_phases are those of the passes that tnc_plan_passes lists
    p = Plan.from_circuit(H.mixed_circuit(n, d, 3 * d + k, dense=0.3), options)
    info, passes = p.info(k), p.passes(k)
    assert info["n_passes"] == len(passes)
    assert info["n_phases"] == sum(x["phases"] for x in passes)


def test_info_does_not_depend_on_naming_the_default_tiles():
    c = W.brickwork_circuit(20, 40, 5, W.rng_for(471, 1))
    for k in (0, 6):
        assert Plan.from_circuit(c).info(k) == Plan.from_circuit(c, dict(max_tile_bits=13, low_bits=4, reg_bits=5)).info(k)
