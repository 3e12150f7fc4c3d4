"""The work that bench.py credits to a solve's phases: nothing is counted as packed or read from the node-offset
table where the library does not pack or does not take the table."""

import os
import sys

import numpy as np
import pytest

sys.path.insert(0, os.path.dirname(os.path.dirname(os.path.abspath(__file__))))

import bench  # noqa: E402
from workloads import generators as G  # noqa: E402

STATS = dict(nsources=1000, ntargets=300, ncells=80, n_m2l=500, n_p2p_lists=100, n_p2p_pairs=7000)


def _work(nsl, ntl, on, precision):
    w = dict(grid=G.GridSpec(64, 64, 1.0 / 64), p=12, tx=np.zeros(300), n_grid_targets=on)
    return bench.phase_work(dict(STATS, nsrc_leaves=nsl, ntgt_leaves=ntl), w, 5, precision)


@pytest.mark.parametrize("nsl,ntl,precision,packed", [
    (60, 20, "mixed", True), (80, 20, "mixed", True), (81, 20, "mixed", False), (60, 20, "fp64", False)])
def test_packing_counted_where_done(nsl, ntl, precision, packed):
    assert _work(nsl, ntl, 0, precision)["pack"][1] == 64 * 300 + (24 * 1000 if packed else 0)


@pytest.mark.parametrize("on,ops", [(0, 6.0), (150, 6.0), (225, 3.0), (300, 2.0)])
def test_pair_operations_follow_the_targets(on, ops):
    assert _work(60, 20, on, "mixed")["p2p"][1] == ops * 7000


def test_named_workloads_say_where_their_targets_lie():
    w = G.workload("gaussian64")
    assert bench.pair_ops(w) == 2
    assert bench.pair_ops(dict(w, n_grid_targets=0)) == 6  # as many targets as nodes, none of them on one
