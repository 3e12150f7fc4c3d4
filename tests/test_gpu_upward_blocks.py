"""The upward pass by 64 x 64-node cells on the matrix cores (P2M and three levels of M2M, then three levels
per launch) against the lane groups' P2M by leaves, cell by cell: trees whose leaves are narrower than the 8-node
blocks, wider than a workgroup's cell, or the root itself, and every number of 16-column tiles.

Tolerance: a coefficient of either path is a sum of at most 4,096 products of weights with numbers of modulus at
most 1, so their difference is at most 4,096 eps sum |w| = 9.1e-13 sum |w| over the cell's sources (the levels
above add at most their number times that); 1e-11 sum |w| bounds it for the depths used here."""

import numpy as np
import pytest

from gpu_common import to_dev

pytestmark = pytest.mark.gpu


def _case(kind, n, rng):
    f = np.zeros((n, n))
    if kind == "isolated":  # at most leaf_max sources: the root is a leaf
        f[rng.integers(0, n, 30), rng.integers(0, n, 30)] = rng.standard_normal(30)
    elif kind == "sparse":  # wide leaves beside a full corner
        f[rng.integers(0, n, 3 * n // 4), rng.integers(0, n, 3 * n // 4)] = 1.0
        f[:n // 3, :n // 5] = rng.standard_normal((n // 3, n // 5))
    else:
        f = rng.standard_normal((n, n))
    k = 400 if kind == "clustered" else 40
    tx, ty = rng.uniform(0, 1, 300), rng.uniform(0, 1, 300)
    if kind == "clustered":  # targets that split leaves far below the blocks
        tx, ty = np.concatenate([tx, 0.3 + rng.uniform(0, 4 / n, k)]), np.concatenate([ty, 0.6 + rng.uniform(0, 4 / n, k)])
    return f, tx, ty


@pytest.mark.parametrize("kind", ["isolated", "sparse", "full", "clustered"])
@pytest.mark.parametrize("n,p", [(64, 7), (33, 8), (96, 3), (200, 12), (300, 15), (520, 16), (520, 20)])
def test_multipoles_match_leaf_path(monkeypatch, kind, n, p):
    import paper_1610_04398_amd as pp
    rng = np.random.Generator(np.random.PCG64((n, p)))
    f, tx, ty = _case(kind, n, rng)
    h = 1.0 / n
    fd, txd, tyd = to_dev(f, tx, ty)
    blocks = pp.Solver(0)
    monkeypatch.setenv("PP_P2M_LATTICE", "0")
    leaves = pp.Solver(0)
    try:
        out = []
        for s in (blocks, leaves):
            s.solve_grid(fd, h, txd, tyd, p=p, theta=0.5, leaf_max=64, precision="fp64")
            out.append(s.debug_array("MULTIPOLE").reshape(-1, p + 1, 2))
        sb, se = blocks.debug_array("CELL_SB"), blocks.debug_array("CELL_SE")
        ij = blocks.debug_array("SRC_INDEX").astype(np.int64)
        w = np.abs(f[ij >> 16, ij & 0xFFFF]) * h * h
        total = np.concatenate([[0.0], np.cumsum(w)])
        scale = total[se] - total[sb]
        has = se > sb
        assert has.any()
        err = np.abs(out[0] - out[1]).max(axis=(1, 2))
        assert np.all(err[has] <= 1e-11 * scale[has]), float(np.max(err[has] / scale[has]))
    finally:
        blocks.close()
        leaves.close()
