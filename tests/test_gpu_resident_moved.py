"""Resident solves whose targets have moved off the grid's nodes, onto them, or back, inside their finest cells
since the tree was built: the near field that serves the targets where they are now does the work, whatever the kept
tree's were, and the results are bitwise those of fresh solves.  Sizes on both sides of the number of waves from
which both kinds are launched."""

import numpy as np
import pytest

from gpu_common import to_dev, to_host

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("first", ["nodes", "moved"])
@pytest.mark.parametrize("n,leaf_max", [(72, 64), (160, 64), (264, 64), (160, 16), (264, 300)])
@pytest.mark.parametrize("precision", ["mixed", "fp64"])
@pytest.mark.parametrize("method,graph", [("fmm", "0"), ("fmm", "1"), ("treecode", "0")])
def test_moved_targets(monkeypatch, first, n, leaf_max, precision, method, graph):
    import paper_1610_04398_amd as pp
    h = 1.0 / n
    rng = np.random.Generator(np.random.PCG64((n, leaf_max)))
    f = rng.standard_normal((n, n))
    f[rng.uniform(size=f.shape) < 0.02] = 0.0
    j, i = np.divmod(np.arange(n * n), n)
    at = {"nodes": ((i + 0.5) * h, (j + 0.5) * h)}
    at["moved"] = tuple((k + rng.uniform(0.1, 0.9, n * n)) * h for k in (i, j))
    some = rng.uniform(size=n * n) < 0.4
    at["some"] = tuple(np.where(some, a, b) for a, b in zip(at["moved"], at["nodes"]))
    fd, gd = to_dev(f, 0.5 * f)
    dev = {k: to_dev(*v) for k, v in at.items()}
    kw = dict(p=8, leaf_max=leaf_max, precision=precision, method=method)
    monkeypatch.setenv("PP_RESIDENT_GRAPH", graph)
    kept, fresh = pp.Solver(0), pp.Solver(0)
    try:
        want = {k: to_host(fresh.solve_grid(gd, h, *v, **kw)) for k, v in dev.items()}
        pairs = fresh.stats()["n_p2p_pairs"]
        kept.solve_grid(fd, h, *dev[first], **kw)
        for k in ("nodes", "moved", "some") * 3:
            assert np.array_equal(to_host(kept.solve_grid_resident(gd, *dev[k])), want[k]), k
            assert kept.stats()["n_p2p_pairs"] == pairs
    finally:
        kept.close()
        fresh.close()


@pytest.mark.parametrize("first", ["nodes", "moved"])
def test_moved_targets_in_little_memory(first):
    """The FP64 near field in two launches (of each kind)."""
    import paper_1610_04398_amd as pp
    n = 520
    h = 1.0 / n
    rng = np.random.Generator(np.random.PCG64(n))
    j, i = np.divmod(np.arange(n * n), n)
    at = {"nodes": ((i + 0.5) * h, (j + 0.5) * h)}
    at["moved"] = tuple((k + rng.uniform(0.1, 0.9, n * n)) * h for k in (i, j))
    f = to_dev(rng.standard_normal((n, n)))[0]
    dev = {k: to_dev(*v) for k, v in at.items()}
    free, tight = pp.Solver(0), pp.Solver(0, hbm_budget_bytes=82384932)
    try:
        want = {k: to_host(free.solve_grid(f, h, *v, precision="fp64")) for k, v in dev.items()}
        tight.solve_grid(f, h, *dev[first], precision="fp64")
        for k in ("moved", "nodes", "moved"):
            assert np.array_equal(to_host(tight.solve_grid_resident(f, *dev[k])), want[k]), k
    finally:
        free.close()
        tight.close()
