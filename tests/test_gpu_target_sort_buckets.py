"""The target sort by buckets (32,769 to 524,288 targets on roots of 256 and more cells a side): keys and
permutation equal the oracle's stable sort exactly, for targets spread over the domain, gathered along a line,
and crowded so that a bucket does not fit (the first segment is then repeated with radix passes).  Eager,
captured and replayed calls, and new targets in the buffers of a captured call."""

import numpy as np
import pytest

from oracle import tree_ref
from gpu_common import to_dev

pytestmark = pytest.mark.gpu


def _targets(kind, m, rng):
    if kind == "line":
        a = rng.uniform(0, 2 * np.pi, m)
        return 0.5 + 0.45 * np.cos(a), 0.5 + 0.4 * np.sin(a)
    tx, ty = rng.uniform(0, 1, (2, m))
    if kind == "crowded":
        tx[: m // 2], ty[: m // 2] = 0.7 + 1e-3 * tx[: m // 2], 0.2 + 1e-3 * ty[: m // 2]
    elif kind == "repeated":  # few distinct keys: equal keys keep their input order
        q = rng.integers(0, 3000, m)
        tx, ty = tx[q], ty[q]
    return tx, ty


@pytest.mark.parametrize("n,m", [(100, 40000), (129, 40000), (200, 32769), (300, 65536), (300, 65537),
                                 (1100, 100001), (513, 524288), (513, 524289)])
@pytest.mark.parametrize("kind", ["uniform", "line", "crowded", "repeated"])
def test_target_order(n, m, kind):
    h = 1.0 / n
    rng = np.random.Generator(np.random.PCG64((n, m)))
    f = np.zeros((n, n))
    f[rng.integers(0, n, 40), rng.integers(0, n, 40)] = 1.0
    first, other = _targets("uniform", m, rng), _targets(kind, m, rng)
    fd, txd, tyd, tx2, ty2 = to_dev(f, *first, *other)
    import paper_1610_04398_amd as pp
    s = pp.Solver(0)
    want = [tree_ref.target_keys_sorted(x, y, 0.0, 0.0, h, tree_ref.root_exponent(n, n)) for x, y in (first, other)]
    try:
        for call in range(7):
            if call == 3:  # new targets in the same buffers
                txd.copy_(tx2)
                tyd.copy_(ty2)
            s.solve_grid(fd, h, txd, tyd, p=4, theta=0.5, leaf_max=4096, precision="mixed")
            keys, perm = want[call >= 3]
            np.testing.assert_array_equal(s.debug_array("TGT_KEY").astype(np.uint64), keys)
            np.testing.assert_array_equal(s.debug_array("TGT_PERM"), perm)
    finally:
        s.close()
