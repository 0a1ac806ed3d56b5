"""Which origin-destination pairs a handle accepts."""
import numpy as np
import pytest

from paper_2603_25068_amd import workloads as W
from paper_2603_25068_amd.sim import SimError, footprint


@pytest.mark.parametrize("turn_back", [False, True])
def test_destinations_across_components(turn_back):
    """Two two-way roads joined by a one-way link: agents may cross it one way only, and the first agent (whose
    component is looked at first) may be in either part."""
    w = W.line(n_links=5, n_agents=4)
    net = w.net
    net.n_nodes = 4
    net.tail[:], net.head[:] = [0, 1, 1, 2, 3], [1, 0, 2, 3, 2]   # 0 <-> 1 -> 2 <-> 3
    net.origin_node = np.asarray([0, 3, 1], np.int32)
    for first in (0, 1):
        w.dem.agent_origin[:] = [first, 0, 2, 1]
        w.dem.agent_dest[:] = [1 if first == 0 else 2, 3, 2, 0 if turn_back else 2]
        if turn_back:
            with pytest.raises(SimError, match="rejected"):
                footprint(w)
        else:
            assert footprint(w) > 0
