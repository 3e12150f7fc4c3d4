"""Source and force calls that name no stream, with inputs still being written on the null stream or on a blocking
stream of the caller's: the calls see the finished inputs, and their results are there when they return (panels and
sums on host or device, up to 16 bodies and more)."""

import ctypes
import glob
import os

import numpy as np
import pytest

pytestmark = pytest.mark.gpu


def _streams():
    """The null stream, and a blocking stream made with the HIP runtime that torch has loaded."""
    import torch
    torch.cuda.init()
    yield "null", torch.cuda.default_stream()
    lib = glob.glob(os.path.join(os.path.dirname(torch.__file__), "lib", "libamdhip64.so*"))
    hip = ctypes.CDLL(lib[0] if lib else "libamdhip64.so")
    handle = ctypes.c_void_p()
    assert hip.hipStreamCreate(ctypes.byref(handle)) == 0
    yield "blocking", torch.cuda.ExternalStream(handle.value)


@pytest.mark.parametrize("nseg", [1, 16, 17])
def test_inputs_in_flight(nseg):
    import torch

    import paper_1610_04398_amd as pp
    n, m = 256, 5000
    gen = torch.Generator(device="cuda").manual_seed(nseg)
    rnd = lambda *s: torch.rand(*s, dtype=torch.float64, device="cuda", generator=gen)  # noqa: E731
    u, v, p, nx, ny, ds = rnd(n, n), rnd(n, n), rnd(m), rnd(m), rnd(m), rnd(m)
    lx, ly = rnd(m), rnd(m)
    seg = np.linspace(0, m, nseg + 1).astype(np.int64)
    big = rnd(4096, 4096)
    s = pp.Solver(0)
    try:
        def results(u_, p_, host):
            a = [t.cpu().numpy() if host else t for t in (p_, nx, ny, ds)]
            f = s.pressure_source(u_, v, 1.0 / n, stream=0)
            fs, dx, dy = s.surface_forces(*a, seg, pointwise=True, stream=0)
            fv, vx, vy = s.viscous_forces(u_, v, 1.0 / n, lx, ly, nx, ny, ds, seg, pointwise=True, stream=0)
            return [np.asarray(t.cpu()) if torch.is_tensor(t) else np.asarray(t) for t in (f, dx, dy, vx, vy)] + [
                np.array([[d[k] for k in ("fx", "fy", "drag", "cd")] for d in q]) for q in (fs, fv)]

        for host in (False, True):
            want = results(3.0 * u, 3.0 * p, host)
            for name, stream in _streams():
                torch.cuda.synchronize()
                u2, p2 = torch.zeros_like(u), torch.zeros_like(p)
                torch.cuda.synchronize()
                with torch.cuda.stream(stream):
                    for _ in range(40):  # milliseconds of work before the inputs are written
                        big.mul_(1.0000001)
                    torch.mul(u, 3.0, out=u2)
                    torch.mul(p, 3.0, out=p2)
                for a, b in zip(results(u2, p2, False) if not host else results(u2, p2, True), want):
                    assert np.array_equal(a, b), name
    finally:
        torch.cuda.synchronize()
        s.close()
