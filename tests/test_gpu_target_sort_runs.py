"""The target sort carried by the ingest launches (runs of 1,024 keys sorted in LDS, merged in one step)
at the edges of its runs, of the merge's stages of four runs and of its range, against the oracle's stable
sort: keys and permutation are whole numbers and must be equal."""

import numpy as np
import pytest

from oracle import tree_ref
from gpu_common import to_dev

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,m", [(1, 1500), (2, 1), (48, 1023), (48, 1024), (48, 1025), (300, 4096), (300, 4097),
                                 (700, 5 * 1024 + 3), (2050, 32768), (2050, 32769)])
@pytest.mark.parametrize("spread", ["uniform", "repeated"])
def test_target_order(n, m, spread):
    import paper_1610_04398_amd as pp
    h = 1.0 / n
    rng = np.random.Generator(np.random.PCG64((n, m)))
    f = np.zeros((n, n))
    f[rng.integers(0, n, 40), rng.integers(0, n, 40)] = 1.0
    tx, ty = rng.uniform(0, 1, m), rng.uniform(0, 1, m)
    if spread == "repeated":  # few distinct keys, in one corner of the domain: equal keys keep their input order
        q = rng.integers(0, 7, m)
        tx, ty = 0.1 * tx[q % m], 0.1 * ty[q % m]
    fd, txd, tyd = to_dev(f, tx, ty)
    s = pp.Solver(0)
    try:
        for _ in range(3):  # eager, captured, replayed
            s.solve_grid(fd, h, txd, tyd, p=4, theta=0.5, leaf_max=4096, precision="fp64")
            keys, perm = tree_ref.target_keys_sorted(tx, ty, 0.0, 0.0, h, tree_ref.root_exponent(n, n))
            np.testing.assert_array_equal(s.debug_array("TGT_KEY").astype(np.uint64), keys)
            np.testing.assert_array_equal(s.debug_array("TGT_PERM"), perm)
    finally:
        s.close()
