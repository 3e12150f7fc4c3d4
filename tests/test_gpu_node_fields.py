"""Near field of node fields by the tables of log2(r^2) and ln(r^2) over node offsets, against the loops of the
one-stream schedule, which evaluate every pair: the same terms in the same order, so near sums and outputs are
equal bit for bit.  Full fields, culled nodes, grids that end inside a leaf, targets beside the nodes (leaves
split below 8 nodes), repeated targets, leaves of up to 16 nodes, and list radii up to and beyond the tables'
reach."""

import numpy as np
import pytest

from gpu_common import to_dev, to_host

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("nx,ny", [(40, 64), (96, 96), (101, 87), (200, 136)])
@pytest.mark.parametrize("kind", ["full", "culled", "extra", "subset"])
@pytest.mark.parametrize("theta,leaf_max", [(0.5, 64), (0.2, 64), (0.8, 64), (0.5, 300)])
@pytest.mark.parametrize("precision", ["mixed", "fp64"])
def test_node_field_equals_pairwise(monkeypatch, nx, ny, kind, theta, leaf_max, precision):
    rng = np.random.Generator(np.random.PCG64((nx, ny)))
    n = max(nx, ny)
    h = 1.0 / n
    f = rng.standard_normal((ny, nx))
    x, y = np.meshgrid((np.arange(nx) + 0.5) * h, (np.arange(ny) + 0.5) * h)
    tx, ty = x.ravel(), y.ravel()
    if kind == "culled":
        f[rng.uniform(size=f.shape) < 0.02] = 0.0
    elif kind == "extra":
        a = rng.uniform(0, 2 * np.pi, 500)
        tx = np.concatenate([tx, 0.25 + 0.1 * np.cos(a), tx[:70]])
        ty = np.concatenate([ty, 0.25 + 0.1 * np.sin(a), ty[:70]])
    elif kind == "subset":
        pick = rng.choice(tx.size, tx.size // 2, replace=False)
        tx, ty = tx[pick], ty[pick]
    fd, txd, tyd = to_dev(f, tx, ty)
    import paper_1610_04398_amd as pp
    got = []
    for waves in ("0", "1000000000"):
        monkeypatch.setenv("PP_COMPACT", waves)
        s = pp.Solver(0)
        try:
            out = [to_host(s.solve_grid(fd, h, txd, tyd, p=6, theta=theta, leaf_max=leaf_max, precision=precision))]
            out.append(s.debug_array("NEAR"))
            out.append(np.array([s.stats()["n_p2p_pairs"]]))
            got.append(out)
        finally:
            s.close()
    for a, b in zip(*got):
        assert np.array_equal(a, b)
