"""The one-stream schedule of small solves (lists + P2M + target preparation in one launch, the first M2M launch
with the near field, the downward pass with the finalize step) against the two-stream schedule: the same lists,
sums and orders, so outputs, multipoles and locals are equal bit for bit.  Depths at which one, two and three
M2M launches follow the blocks, every number of 16-column tiles, both precisions and methods, both list radii,
and counts of near-field waves on either side of the rule."""

import numpy as np
import pytest

from gpu_common import to_dev, to_host

pytestmark = pytest.mark.gpu


def _case(n, m, kind):
    rng = np.random.Generator(np.random.PCG64((n, m)))
    f = rng.standard_normal((n, n))
    if kind == "sparse":
        f[rng.uniform(size=f.shape) < 0.97] = 0.0
    elif kind == "band":
        f[:, n // 4:] = 0.0
    a = rng.uniform(0, 2 * np.pi, m)
    tx, ty = 0.5 + 0.3 * np.cos(a), 0.5 + 0.2 * np.sin(a)
    tx[: m // 4], ty[: m // 4] = rng.uniform(0, 1, (2, m // 4))
    return f, tx, ty


@pytest.mark.parametrize("n,m,kind", [(33, 40, "full"), (64, 1, "full"), (65, 3000, "sparse"), (129, 700, "band"),
                                      (520, 1500, "sparse"), (1025, 900, "band")])
@pytest.mark.parametrize("p", [8, 16, 20])
@pytest.mark.parametrize("method,precision,theta", [("fmm", "mixed", 0.5), ("fmm", "fp64", 0.4),
                                                    ("treecode", "mixed", 0.5), ("treecode", "fp64", 0.6)])
def test_compact_equals_two_streams(monkeypatch, n, m, kind, p, method, precision, theta):
    f, tx, ty = _case(n, m, kind)
    fd, fd2, txd, tyd = to_dev(f, 0.5 * f, tx, ty)
    import paper_1610_04398_amd as pp
    got = []
    for waves in ("0", "2048", "1000000000"):
        monkeypatch.setenv("PP_COMPACT", waves)
        with_rule = pp.Solver(0)
        try:
            kw = dict(p=p, theta=theta, leaf_max=64, precision=precision, method=method)
            out = [to_host(with_rule.solve_grid(fd, 1.0 / n, txd, tyd, **kw)) for _ in range(3)]
            # defined where a cell has sources (multipoles) or targets (locals)
            src = with_rule.debug_array("CELL_SE") > with_rule.debug_array("CELL_SB")
            tgt = with_rule.debug_array("CELL_TE") > with_rule.debug_array("CELL_TB")
            arrays = [with_rule.debug_array("MULTIPOLE").reshape(src.size, -1)[src]]
            if method == "fmm":
                arrays.append(with_rule.debug_array("LOCAL").reshape(tgt.size, -1)[tgt])
            out.append(to_host(with_rule.solve_grid_resident(fd2, txd, tyd)))
            got.append(out + arrays)
        finally:
            with_rule.close()
    for other in got[1:]:
        for a, b in zip(got[0], other):
            assert np.array_equal(a, b)
