"""Which launch carries a solve's near field follows from how its targets lie (on nodes or not, crowded or not),
leaf_max and the number of waves; none of it may show in the results.

The tables of log2(r^2) and ln(r^2) over node offsets against the pairwise loop of the same kernel: moving one
target of every leaf beside its node sends the leaf's other targets through the loop, for list entries on both
sides of the tables' reach.  Targets off the nodes, partly on them, in crowded cells and in leaves of every size:
the default route against the one-stream schedule and the two-stream one."""

import numpy as np
import pytest

from gpu_common import to_dev, to_host

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("nx,ny", [(96, 96), (101, 87), (200, 136)])
@pytest.mark.parametrize("theta", [0.2, 0.3, 0.4, 0.5, 0.8])
@pytest.mark.parametrize("precision", ["mixed", "fp64"])
def test_table_equals_pairwise_loop(nx, ny, theta, precision):
    import paper_1610_04398_amd as pp
    rng = np.random.Generator(np.random.PCG64((nx, ny)))
    h = 1.0 / max(nx, ny)
    f = rng.standard_normal((ny, nx))
    i, j = np.meshgrid(np.arange(nx), np.arange(ny))
    x, y = ((i + 0.5) * h).ravel(), ((j + 0.5) * h).ravel()
    moved = ((i % 8 == 3) & (j % 8 == 5)).ravel()
    fd, xd, yd, xm = to_dev(f, x, y, np.where(moved, x + 0.25 * h, x))
    got = []
    for tx in (xd, xm):
        s = pp.Solver(0)
        try:
            s.solve_grid(fd, h, tx, yd, p=6, theta=theta, precision=precision)
            perm = s.debug_array("TGT_PERM")
            got.append((perm, s.debug_array("NEAR").reshape(-1, perm.size)))
            if tx is xd:  # corner offsets of the list entries, in nodes
                D = int(np.ceil(np.log2(max(nx, ny))))
                side = 1 << (D - s.debug_array("CELL_LEVEL"))
                corner = np.stack([s.debug_array("CELL_IX") * side, s.debug_array("CELL_IY") * side])
                off, cnt, src = (s.debug_array(f"P2P_{k}") for k in ("OFF", "CNT", "SRC"))
                leaf = s.debug_array("TGT_LEAF")
                d = [np.abs(corner[:, [c]] - corner[:, src[off[c]:off[c] + cnt[c]]]).max(axis=0)
                     for c in np.unique(leaf) if side[c] == 8]
                far = np.concatenate(d)
        finally:
            s.close()
    reach = 24 if precision == "mixed" else 16
    assert (far <= reach).any()
    assert (far > reach).any() or theta > (0.3 if precision == "mixed" else 0.4)
    (perm, a), (perm2, b) = got
    assert np.array_equal(perm, perm2)
    keep = ~moved[perm]
    assert np.array_equal(a[:, keep], b[:, keep]) and not np.array_equal(a, b)


def _targets(kind, n, rng):
    h = 1.0 / n
    a = rng.uniform(0, 2 * np.pi, 1500)
    ell = 0.5 + 0.3 * np.cos(a), 0.5 + 0.1 * np.sin(a)
    if kind == "ellipse":
        return ell
    if kind == "random":
        return rng.uniform(0, 1, (2, n * n))
    if kind == "crowded":  # 400 targets of one finest cell beside leaves of a few
        return tuple(np.concatenate([e, (0.25 * n // 1 + rng.uniform(0, 1, 400)) * h]) for e in ell)
    x = (np.arange(n) + 0.5) * h
    if kind == "rounded nodes":  # a rounding error away from some of them
        x = np.arange(n) * h + 0.5 * h
        assert 0 < np.mean(x != (np.arange(n) + 0.5) * h) < 1
    x, y = np.tile(x, n), np.repeat(x, n)
    if kind == "rounded nodes":
        return x, y
    if kind == "mostly nodes":
        off = rng.uniform(size=x.size) < 0.3
        return np.where(off, x + 0.3 * h, x), y
    return np.where(rng.uniform(size=x.size) < 0.7, x + 0.3 * h, x), y  # "some nodes"


@pytest.mark.parametrize("kind", ["ellipse", "random", "crowded", "mostly nodes", "some nodes", "rounded nodes"])
@pytest.mark.parametrize("leaf_max", [8, 64, 300])
@pytest.mark.parametrize("precision", ["mixed", "fp64"])
@pytest.mark.parametrize("method", ["fmm", "treecode"])
def test_routes_agree(monkeypatch, kind, leaf_max, precision, method):
    import paper_1610_04398_amd as pp
    n = 136
    rng = np.random.Generator(np.random.PCG64((n, leaf_max)))
    f = rng.standard_normal((n, n))
    f[rng.uniform(size=f.shape) < 0.05] = 0.0
    f[:, : n // 4] = 0.0
    tx, ty = _targets(kind, n, rng)
    fd, gd, txd, tyd = to_dev(f, 0.5 * f, tx, ty)
    kw = dict(p=8, leaf_max=leaf_max, precision=precision, method=method)
    got = []
    for waves in (None, "0", "1000000000"):
        if waves is not None:
            monkeypatch.setenv("PP_COMPACT", waves)
        s = pp.Solver(0)
        try:
            out = [to_host(s.solve_grid(fd, 1.0 / n, txd, tyd, **kw)), s.debug_array("NEAR")]
            out.append(to_host(s.solve_grid_resident(gd, txd, tyd)))
            out.append(to_host(s.solve_grid_noalloc(fd, 1.0 / n, txd, tyd, **kw)))
            got.append(out)
        finally:
            s.close()
    assert np.array_equal(got[0][0], got[0][3])
    for other in got[1:]:
        for a, b in zip(got[0], other):
            assert np.array_equal(a, b)


@pytest.mark.parametrize("count", [64, 65, 256, 257])
@pytest.mark.parametrize("n", [136, 520])
@pytest.mark.parametrize("precision", ["mixed", "fp64"])
def test_routes_agree_at_the_edges_of_a_wave(monkeypatch, count, n, precision):
    """The fullest leaf holds one or four waves' targets, or one more, in the dense table and below it."""
    import paper_1610_04398_amd as pp
    h = 1.0 / n
    rng = np.random.Generator(np.random.PCG64((n, count)))
    f = rng.standard_normal((n, n))
    cell = (n // 3 + rng.uniform(0.05, 0.95, (2, count))) * h
    tx, ty = (np.concatenate([c, rng.uniform(0, 1, 1200)]) for c in cell)
    fd, gd, txd, tyd = to_dev(f, 0.5 * f, tx, ty)
    got = []
    for waves in (None, "0", "1000000000"):
        if waves is not None:
            monkeypatch.setenv("PP_COMPACT", waves)
        s = pp.Solver(0)
        try:
            got.append([to_host(s.solve_grid(fd, h, txd, tyd, p=8, precision=precision)),
                        to_host(s.solve_grid_resident(gd, txd, tyd))])
        finally:
            s.close()
    for other in got[1:]:
        for a, b in zip(got[0], other):
            assert np.array_equal(a, b)
