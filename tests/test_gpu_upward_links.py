"""The upward pass below the tree's dense prefix table, where a workgroup finds its cells by child links: the
same multipoles bit for bit as with the table, and a forest whose extra top levels push its requests' cells below
the table gives each request its lone result bit for bit (P2M by 64 x 64-node cells, and M2M at every level)."""

import numpy as np
import pytest

from gpu_common import to_dev, to_host

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,count,leaf_max", [
    (1100, 5, 64),  # 2^11-node roots two levels down: the 8-node blocks lie at level 10 of the forest
    (2100, 2, 64),  # 2^12, one level down
    (512, 5, 8),    # leaves of 2 x 2 nodes: M2M from level 10
])
def test_batch_equals_lone_below_the_table(n, count, leaf_max):
    import torch

    import paper_1610_04398_amd as pp
    rng = np.random.Generator(np.random.PCG64((n, count)))
    gen = torch.Generator(device="cuda").manual_seed(n)
    fs, txs, tys = [], [], []
    for r in range(count):
        f = torch.rand(n, n, dtype=torch.float64, device="cuda", generator=gen) - 0.5
        if r % 2:  # another depth than its neighbours': a dense corner beside isolated nodes
            keep = torch.rand(n, n, device="cuda", generator=gen) < 1e-4
            keep[: n // 5, n // 2:] = True
            f = f * keep
        fs.append(f.contiguous())
        a = rng.uniform(0, 2 * np.pi, 700)
        tx, ty = to_dev(0.5 + 0.2 * np.cos(a), 0.4 + 0.15 * np.sin(a))
        txs.append(tx)
        tys.append(ty)
    s, lone = pp.Solver(0), pp.Solver(0)
    try:
        outs = s.solve_grid_batch(fs, 1.0 / n, txs, tys, leaf_max=leaf_max)
        for r in range(count):
            want = to_host(lone.solve_grid(fs[r], 1.0 / n, txs[r], tys[r], leaf_max=leaf_max))
            assert np.array_equal(to_host(outs[r]), want), (r, np.max(np.abs(to_host(outs[r]) - want)))
    finally:
        s.close()
        lone.close()


@pytest.mark.parametrize("n", [64, 200, 520])
@pytest.mark.parametrize("p", [5, 12, 20])
@pytest.mark.parametrize("leaf_max", [8, 64, 300])
@pytest.mark.parametrize("levels", [0, 2, 5])
def test_links_equal_table(monkeypatch, n, p, leaf_max, levels):
    import paper_1610_04398_amd as pp
    rng = np.random.Generator(np.random.PCG64((n, p, levels)))
    f = rng.standard_normal((n, n))
    f[rng.uniform(size=f.shape) < 0.3] = 0.0
    f[n // 2:, n // 3:] = 0.0
    f[n - 2, n - 3] = 1.0  # a wide leaf of one node
    tx, ty = rng.uniform(0, 1, 900), rng.uniform(0, 1, 900)
    tx[:400] = 0.3 + rng.uniform(0, 4 / n, 400)
    ty[:400] = 0.2 + rng.uniform(0, 4 / n, 400)
    fd, txd, tyd = to_dev(f, tx, ty)
    got = []
    for dense in (9, levels):
        monkeypatch.setenv("PP_DENSE_LEVELS", str(dense))
        s = pp.Solver(0)
        try:
            out = to_host(s.solve_grid(fd, 1.0 / n, txd, tyd, p=p, leaf_max=leaf_max, precision="fp64"))
            has = s.debug_array("CELL_SE") > s.debug_array("CELL_SB")
            got.append((out, s.debug_array("MULTIPOLE").reshape(-1, 2 * (p + 1))[has], s.debug_array("CELL_LEVEL")))
        finally:
            s.close()
    for a, b in zip(*got):
        assert np.array_equal(a, b)
