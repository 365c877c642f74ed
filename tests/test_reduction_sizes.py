"""Reductions on both sides of the element count up to which a launch asks for all of its arguments at once, against the oracle."""
import numpy as np
import pytest

import oracle as orc
from paper_2406_02629_amd import SSNet
from util import P61, field_uniform, to_dev, to_np

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,t,edge", [(3, 1, 1 << 17), (5, 2, 1 << 17), (6, 2, 1 << 17), (7, 3, 1 << 18)])
@pytest.mark.parametrize("past", [0, 1])
def test_reduction_at_the_edge(n, t, edge, past):
    count = edge + past
    print("degree_reduce(+truncate)", n, t, count, flush=True)
    s = SSNet(n, t, f=13, seed=19)
    c = field_uniform((n, count), seed=count)
    red = orc.degree_reduce(c, n, t, P61, 19, 3)
    assert np.array_equal(to_np(s.degree_reduce(to_dev(c), stream_id=3)), red)
    assert np.array_equal(to_np(s.degree_reduce_truncate(to_dev(c), stream_id=3)), orc.truncate(red, n, t, 13, P61, 19, 3))
