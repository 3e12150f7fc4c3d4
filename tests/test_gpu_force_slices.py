"""Force sums split over workgroups (up to 16 bodies, 64 slices of 256 panels each) and one workgroup per body
beyond that: empty bodies, bodies at and around the edges of a slice and of 64 slices, 16 and 17 bodies, and
repeated calls (the slices' arrival counters return to zero).  The per-panel forces equal the plain formulas bit
for bit; the sums are compensated throughout, so they are the exactly rounded ones to a few eps of the net
force plus eps^2 of the sum of moduli times its length: 1e-15 of that sum
bounds both (2e-15 for the drag, whose projection rounds six times on either side)."""

import numpy as np
import pytest

from oracle import assembly, forces

from gpu_common import to_dev, to_host

pytestmark = pytest.mark.gpu

SEGMENTS = [[1], [255, 0, 256, 257, 1], [4096], [64 * 256 - 1, 64 * 256, 64 * 256 + 1], [40000, 3], [0] * 15 + [513],
            [700] * 16, [700] * 17, [1, 300, 0] * 20]


@pytest.mark.parametrize("lengths", SEGMENTS)
@pytest.mark.parametrize("host", [False, True])
def test_sums_match_oracle(lengths, host):
    seg = np.concatenate([[0], np.cumsum(lengths)])
    m, n = int(seg[-1]), 50
    h, mu = 1.0 / n, 0.3
    rng = np.random.Generator(np.random.PCG64(m))
    p, nx, ny = rng.standard_normal((3, m))
    ds = rng.uniform(0, 1, m)
    lx, ly = rng.uniform(-0.1, 1.1, (2, m))
    u, v = rng.standard_normal((2, n, n))
    dev = to_dev(p, nx, ny, ds, lx, ly, u, v)
    if host:
        dev = [p, nx, ny, ds, lx, ly, u, v]
    pd, nxd, nyd, dsd, lxd, lyd, ud, vd = dev
    import paper_1610_04398_amd as pp
    want = [forces.surface_forces(p, nx, ny, ds, seg, 0.3, -0.1, 1.2, 0.08),
            assembly.viscous_forces(u, v, h, 0.0, 0.0, lx, ly, nx, ny, ds, seg, mu, 0.3, -0.1, 1.2, 0.08)]
    kw = dict(rho=1.2, area=0.08)
    s = pp.Solver(0)
    try:
        for again in range(2):
            for pointwise in (True, False):
                got = [s.surface_forces(pd, nxd, nyd, dsd, seg, u=(0.3, -0.1), pointwise=pointwise, **kw),
                       s.viscous_forces(ud, vd, h, lxd, lyd, nxd, nyd, dsd, seg, mu=mu, uinf=(0.3, -0.1),
                                        pointwise=pointwise, **kw)]
                for g, (dfx, dfy, sums) in zip(got, want):
                    if pointwise:
                        g, gx, gy = g
                        gx, gy = (gx, gy) if host else (to_host(gx), to_host(gy))
                        assert np.array_equal(gx, dfx) and np.array_equal(gy, dfy)
                    for a, r, lo, hi in zip(g, sums, seg[:-1], seg[1:]):
                        scale = float(np.sum(np.abs(dfx[lo:hi])) + np.sum(np.abs(dfy[lo:hi])))
                        for k, tol in (("fx", 1e-15), ("fy", 1e-15), ("drag", 2e-15)):
                            assert abs(a[k] - r[k]) <= tol * scale, (k, a[k], r[k])
    finally:
        s.close()
