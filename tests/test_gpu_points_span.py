"""Scattered points whose span no root square can hold (it overflows FP64, or is below 1e-280) are refused with
the same status and text on both sides of the joint sort's limit of 131,072 points;
the solver then works as a fresh one."""

import numpy as np
import pytest

from gpu_common import to_dev, to_host

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [3, 131072, 131073])
@pytest.mark.parametrize("ends,target,text", [
    ((-1e308, 1e308), 0.0, "span is not finite"),
    ((-1e308, 1e308), 1e308, "span is not finite"),
    ((0.0, 1e-290), 0.0, "less than 1e-280"),
    ((0.0, np.inf), 0.0, "non-finite"),
])
def test_span_refused(n, ends, target, text):
    import paper_1610_04398_amd as pp
    x = np.full(n, ends[0])
    x[1] = ends[1]
    sx, sy, w, tx, ty = to_dev(x, np.zeros(n), np.ones(n), np.array([target]), np.zeros(1))
    s, fresh = pp.Solver(0), pp.Solver(0)
    try:
        with pytest.raises(pp.PPError, match=text) as e:
            s.solve_points(sx, sy, w, tx, ty)
        assert e.value.status == -1
        sx, sy, w, tx, ty = to_dev([0.0, 1.0], [0.0, 0.0], [1.0, 1.0], [3.0], [0.0])
        assert np.array_equal(*(to_host(q.solve_points(sx, sy, w, tx, ty)) for q in (s, fresh)))
    finally:
        s.close()
        fresh.close()
