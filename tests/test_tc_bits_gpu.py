"""The closure on packed rows: sizes on both sides of a band, a 128-column
quad and a 1024-column slab, row pitches of every alignment, and a few
workgroups for many rows, exactly against the oracle."""
import numpy as np
import pytest

import oracle
from paper_1908_06649_amd import tcu

from test_tc_gpu import graph, run_tc

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("extra", [0, 1, 6, 16])
@pytest.mark.parametrize("n", [3, 33, 129, 250, 257, 384, 385, 511, 640, 1025, 1153])
def test_tc_sizes_and_pitches(n, extra):
    d = graph(n, 1.3, n + extra)
    assert np.array_equal(run_tc(d, n + extra), oracle.transitive_closure(d))


@pytest.mark.parametrize("cus", [1, 3, 4, 40])
@pytest.mark.parametrize("n", [300, 1100, 2500])
def test_tc_few_workgroups(n, cus, knobs):
    """Row ranges of more than one step, one range per slab, and ragged ones."""
    knobs(tcu.TCU_KNOB_PP_GRID, cus)
    d = graph(n, 1.2, n + cus)
    assert np.array_equal(run_tc(d, n + 3), oracle.transitive_closure(d))


def test_tc_dense_and_long_cycle():
    """A band whose every row reaches every pivot, and reachability that has
    to pass through all of them in a scrambled order."""
    n = 1300
    d = graph(n, 600.0, 4)
    assert np.array_equal(run_tc(d), oracle.transitive_closure(d))
    perm = np.random.default_rng(3).permutation(n)
    cyc = np.zeros((n, n), np.uint8)
    cyc[perm, np.roll(perm, 1)] = 1
    assert np.all(run_tc(cyc, n + 7) == 1)
