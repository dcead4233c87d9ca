"""Coupled runs long enough to replay a captured graph of steps."""
import ctypes

import numpy as np
import pytest

from gpu_util import to_dev
from paper_1911_03225_amd import workloads as W

pytestmark = pytest.mark.gpu

LOAD = dict(strain_rate13=2e-3, tau0=0.005, mobility=1.0, mu=1.0, lam=1.5, layer_h=3.0, cell_l3=24.0,
            dt_max=0.25, eps13=0.02, tau_y=0.01, beta=1e-2)


@pytest.fixture(scope="module")
def fdm():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1911_03225_amd import fdm as F
    F.load_library()
    return F


def _case(nx=72, ny=56):
    phi, a11, a12 = W.plateau_rings(nx, ny, seed=5, count=4, rmin=6.0, rmax=14.0)
    return float(phi.mean()), a11, a12


def _replays(fdm, ctx):
    f = fdm.load_library().fdm_debug_coupled_replays   # (the library's counter for this test)
    f.argtypes, f.restype = [ctypes.c_void_p], ctypes.c_int64
    return f(ctx.handle)


@pytest.mark.parametrize("precision,laws", [("fp32", ["threshold"]), ("fp32", ["wiggly"]),
                                            ("fp32", ["threshold", "wiggly"]), ("fp64", ["threshold"]),
                                            ("fp64", ["wiggly"])])
def test_a_fresh_context_replays(fdm, precision, laws):
    """The first call of 200 steps replays graphs, with either law and with
    the other law's run before it: nothing is allocated while capturing."""
    mean, a11, a12 = _case()
    dt = np.float64 if precision == "fp64" else np.float32
    t11, t12 = to_dev(a11, dt), to_dev(a12, dt)
    ctx = fdm.fdm_transport_init(fdm.desc(72, 56, cfl=0.4, v0=-1.0), options={"precision": precision})
    for law in laws:
        before = _replays(fdm, ctx)
        fdm.fdm_run(ctx, t11, t12, 200, 200, loading=fdm.loading(phi_mean=mean, law=law, **LOAD))
        n = _replays(fdm, ctx) - before
        assert n >= 12, (law, n)
    fdm.fdm_destroy(ctx)


@pytest.mark.parametrize("chunk,least", [(1, 199), (4, 49), (8, 24), (15, 12), (20, 19)])
def test_short_chunks_replay(fdm, chunk, least):
    """A chunk below sixteen steps is one replay, a longer one whole shares of
    it: of 200 steps none but the first chunk's and a short last one's, and a
    step or two a chunk, are enqueued kernel by kernel."""
    mean, a11, a12 = _case()
    t11, t12 = to_dev(a11, np.float32), to_dev(a12, np.float32)
    ctx = fdm.fdm_transport_init(fdm.desc(72, 56, cfl=0.4, v0=-1.0))
    fdm.fdm_run(ctx, t11, t12, 200, chunk, loading=fdm.loading(phi_mean=mean, **LOAD))
    n = _replays(fdm, ctx)
    fdm.fdm_destroy(ctx)
    assert n >= least, n


@pytest.mark.parametrize("precision,law,time_order", [("fp32", "threshold", 2), ("fp32", "wiggly", 2),
                                                      ("fp32", "threshold", 1), ("fp64", "threshold", 3),
                                                      ("fp64", "wiggly", 2)])
def test_replayed_steps_give_the_bits_of_direct_ones(fdm, precision, law, time_order):
    """200 steps in twenty calls too short to replay anything, against one
    call, and two calls of the same context, in chunks that are whole shares
    of a graph, that leave steps over, and that wait after every step: the
    same state and scalars bit for bit, with the diagnostics of every chunk
    read between the replays."""
    mean, a11, a12 = _case()
    cfl = 0.25 if time_order == 1 else 0.4
    dt = np.float64 if precision == "fp64" else np.float32

    def run(calls, n, chunk):
        t11, t12 = to_dev(a11, dt), to_dev(a12, dt)
        ctx = fdm.fdm_transport_init(fdm.desc(72, 56, cfl=cfl, v0=-1.0, time_order=time_order),
                                     options={"precision": precision})
        h = dict(phi_mean=mean, eps13=LOAD["eps13"])
        for _ in range(calls):
            load = dict(LOAD, law=law, phi_mean=h["phi_mean"], eps13=h["eps13"])
            h = fdm.fdm_run(ctx, t11, t12, n, chunk, loading=fdm.loading(**load))[-1][0]
        r = _replays(fdm, ctx)
        fdm.fdm_destroy(ctx)
        return h, t11.cpu().numpy(), t12.cpu().numpy(), r

    ref, r11, r12, replays = run(20, 10, 10)
    assert replays == 0 and ref["step"] == 200
    for calls, n, chunk in ((1, 200, 200), (1, 200, 40), (1, 200, 17), (1, 200, 16), (1, 200, 7), (1, 200, 1),
                            (2, 100, 25)):
        h, g11, g12, replays = run(calls, n, chunk)
        # (float64 runs replay from 160 steps and chunks of four on)
        assert (replays > 0) == (precision == "fp32" or (n >= 160 and chunk >= 4)), (chunk, replays)
        assert np.array_equal(g11, r11) and np.array_equal(g12, r12), (calls, chunk)
        for k in ("step", "t", "dt", "eps13", "sigma13", "phi_mean", "vmax", "sum_abs"):
            assert h[k] == ref[k], (calls, chunk, k, h[k], ref[k])
