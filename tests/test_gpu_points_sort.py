"""Sort of scattered sources and targets: both sorts together in runs and one merge (up to 131,072 of each, the
root square formed on the device), radix passes beyond.  Keys and permutations equal a stable sort on the CPU
exactly, at the edges of a run, of a merge stage and of the rule, with ties and zero-weight sources; a
non-finite input is refused on both paths, and the call after it is not."""

import numpy as np
import pytest

from gpu_common import to_dev

pytestmark = pytest.mark.gpu
DEPTH = 15


def _spread(v):
    v = v.astype(np.uint64)
    out = np.zeros_like(v)
    for b in range(DEPTH):
        out |= ((v >> np.uint64(b)) & np.uint64(1)) << np.uint64(2 * b)
    return out


def _keys(x, y, x0, y0, u):
    return _spread(np.floor((x - x0) / u)) | (_spread(np.floor((y - y0) / u)) << np.uint64(1))


@pytest.mark.parametrize("n,m", [(1, 1), (5, 1023), (1024, 1025), (1025, 300), (4097, 4096), (50001, 2),
                                 (131072, 131072), (131073, 40), (300, 131073)])
def test_sorted_as_on_the_cpu(n, m):
    rng = np.random.Generator(np.random.PCG64((n, m)))
    sx, sy = rng.uniform(-3, 5, n), rng.uniform(0, 1, n)
    tx, ty = rng.uniform(0, 1, m), rng.uniform(0, 2, m)
    if n > 1000:  # ties, and clusters below the dense levels
        sx[: n // 3], sy[: n // 3] = np.round(sx[: n // 3], 1), np.round(sy[: n // 3], 1)
        sx[n // 3: n // 2] = 0.4 + 1e-4 * sx[n // 3: n // 2]
    if m > 1000:
        tx[::7], ty[::7] = 0.25, 0.75
    w = rng.standard_normal(n)
    w[rng.uniform(size=n) < 0.2] = 0.0
    w[0] = 1.0
    live = w != 0.0
    xs, ys = np.concatenate([sx[live], tx]), np.concatenate([sy[live], ty])
    x0, y0 = xs.min(), ys.min()
    ext = max(xs.max() - x0, ys.max() - y0)
    u = 1.0
    if ext > 0:
        u = 2.0 ** (np.floor(np.log2(ext)) - DEPTH)
        while u * 2 ** DEPTH <= ext:
            u *= 2
    ks = np.where(live, _keys(np.where(live, sx, x0), np.where(live, sy, y0), x0, y0, u), np.uint64(0xFFFFFFFF))
    kt = _keys(tx, ty, x0, y0, u)
    so, to = np.argsort(ks, kind="stable")[: live.sum()], np.argsort(kt, kind="stable")
    dev = to_dev(sx, sy, w, tx, ty)
    bad = [d.clone() for d in dev]
    bad[n % 2][n - 1] = float("nan")
    badt = [d.clone() for d in dev]
    badt[3][m - 1] = float("inf")
    import paper_1610_04398_amd as pp
    s = pp.Solver(0)
    try:
        s.solve_points(*dev, p=4, theta=0.5, leaf_max=64)
        assert np.array_equal(s.debug_array("SRC_KEY"), ks[so].astype(np.uint32))
        assert np.array_equal(s.debug_array("SRC_INDEX"), so.astype(np.uint32))
        assert np.array_equal(s.debug_array("TGT_KEY"), kt[to].astype(np.uint32))
        assert np.array_equal(s.debug_array("TGT_PERM"), to)
        for b in (bad, badt):
            with pytest.raises(pp.PPError):
                s.solve_points(*b, p=4, theta=0.5, leaf_max=64)
        s.solve_points(*dev, p=4, theta=0.5, leaf_max=64)
        assert np.array_equal(s.debug_array("SRC_INDEX"), so.astype(np.uint32))
    finally:
        s.close()
