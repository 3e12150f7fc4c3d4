"""The target sort's buckets at the edges of what fits in them: node fields that fill them and a body's targets on
top (roots of more than 512 cells), the largest bucket one key below, at and above one run and its room on
either size of root, targets too many for the grid's share of the root, and crowded calls between even ones, of varying number
(the sort goes to radix passes for a while and back).  Keys and permutation equal the oracle's stable sort."""

import numpy as np
import pytest

from oracle import tree_ref
from gpu_common import to_dev

pytestmark = pytest.mark.gpu


def _nodes(nx, ny, h):
    return np.tile((np.arange(nx) + 0.5) * h, ny), np.repeat((np.arange(ny) + 0.5) * h, nx)


def _ellipse(m):
    a = 2 * np.pi * np.arange(m) / m
    return 0.5 + 0.2 * np.cos(a), 0.5 + 0.05 * np.sin(a)


def _filled(n, most, rng):
    """40,000 targets, `most` of them in the root's first bucket (one 512th of the Morton order: the lower left
    1/32 x 1/16 of the root)."""
    k = tree_ref.root_exponent(n, n)
    side = (1 << k) / n
    x, y = rng.uniform(0, 1, (2, 40000))
    inside = np.arange(40000) < most
    bx, by = side / 16, side / 32  # the first 2^(2k - 9) keys
    x = np.where(inside, rng.uniform(0, bx, 40000) * 0.999, bx + (1 - bx) * x)
    y = np.where(inside, rng.uniform(0, by, 40000) * 0.999, y)
    order = rng.permutation(40000)
    return x[order], y[order]


def _check(s, fd, n, h, x, y):
    xd, yd = to_dev(x, y)
    s.solve_grid(fd, h, xd, yd, p=2, leaf_max=4096)
    keys, perm = tree_ref.target_keys_sorted(x, y, 0.0, 0.0, h, tree_ref.root_exponent(n, n))
    np.testing.assert_array_equal(s.debug_array("TGT_KEY").astype(np.uint64), keys)
    np.testing.assert_array_equal(s.debug_array("TGT_PERM"), perm)
    return keys


def _sources(n, rng):
    f = np.zeros((n, n))
    f[rng.integers(0, n, 40), rng.integers(0, n, 40)] = 1.0
    return to_dev(f)[0]


@pytest.mark.parametrize("n,extra", [(513, 0), (513, 256), (600, 300), (700, 1000)])
def test_node_fields_on_larger_roots(n, extra):
    import paper_1610_04398_amd as pp
    rng = np.random.Generator(np.random.PCG64(n))
    x, y = (np.concatenate(c) for c in zip(_nodes(n, n, 1.0 / n), _ellipse(extra))) if extra else _nodes(n, n, 1.0 / n)
    fd = _sources(n, rng)
    s = pp.Solver(0)
    try:
        _check(s, fd, n, 1.0 / n, x, y)
    finally:
        s.close()


@pytest.mark.parametrize("n,room", [(400, 2048), (400, 4096), (900, 2048), (900, 4096)])
@pytest.mark.parametrize("over", [-1, 0, 1, 3000])
def test_bucket_room(n, room, over):
    import paper_1610_04398_amd as pp
    rng = np.random.Generator(np.random.PCG64((n, over + 1)))
    fd = _sources(n, rng)
    x, y = _filled(n, room + over, rng)
    s = pp.Solver(0)
    try:
        keys = _check(s, fd, n, 1.0 / n, x, y)
        k = tree_ref.root_exponent(n, n)
        assert np.bincount((keys >> np.uint64(2 * k - 9)).astype(int)).max() == room + over
    finally:
        s.close()


@pytest.mark.parametrize("n,m", [(257, 524288), (513, 400000), (513, 403000), (520, 524288)])
def test_grids_far_smaller_than_their_root(n, m):
    import paper_1610_04398_amd as pp
    rng = np.random.Generator(np.random.PCG64((n, m)))
    fd = _sources(n, rng)
    s = pp.Solver(0)
    try:
        _check(s, fd, n, 1.0 / n, *rng.uniform(0, 1, (2, m)))
    finally:
        s.close()


def test_crowded_calls_between_even_ones():
    import paper_1610_04398_amd as pp
    n = 300
    rng = np.random.Generator(np.random.PCG64(n))
    fd = _sources(n, rng)
    s = pp.Solver(0)
    try:
        for call in range(45):
            m = 33000 + 7 * call
            x, y = rng.uniform(0, 1, (2, m))
            if call % 3 != 1:
                x[: m // 2], y[: m // 2] = 0.3 + 1e-3 * x[: m // 2], 0.6 + 1e-3 * y[: m // 2]
            _check(s, fd, n, 1.0 / n, x, y)
    finally:
        s.close()
