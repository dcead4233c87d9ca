"""One-row problems (ny = 1): several steps a launch under the AUTO schedule
and through the allocation-free entry, against the plain schedule's stage
launches, bit for bit (the same operations), for every integrator, scheme,
velocity and precision, widths around the written columns of a wave and step
counts around what a launch takes."""
import numpy as np
import pytest

from gpu_util import gpu_run, to_dev

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def fdm():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1911_03225_amd import fdm as F
    F.load_library()
    return F


KINDS = {
    "uniform": dict(v0=-0.8),
    "field": dict(),
    "prescribed": dict(velocity="prescribed", V=(0.7, -0.4)),
}


def _data(nx):
    rng = np.random.default_rng(nx)
    a11, a12 = (rng.standard_normal((1, nx)).astype(np.float32) for _ in range(2))
    a12[0, nx // 3: nx // 2] = 0.0
    a11[0, nx // 4: nx // 2] = 0.0
    return a11, a12, rng.uniform(-1, 1, (1, nx)).astype(np.float32)


@pytest.mark.parametrize("nx,steps", [(1, 3), (2, 2), (31, 9), (32, 16), (33, 17), (64, 5), (97, 40), (2048, 33)])
@pytest.mark.parametrize("order,scheme", [(1, "semidiscrete"), (2, "semidiscrete"), (3, "semidiscrete"),
                                          (1, "fully_discrete")])
@pytest.mark.parametrize("kind", sorted(KINDS))
def test_line_equals_stage_launches_bitwise(fdm, nx, steps, order, scheme, kind):
    a11, a12, v0f = _data(nx)
    kw = dict(KINDS[kind], limiter="mc", cfl=0.25, time_order=order, scheme=scheme, dx=0.5)
    if kind == "field":
        kw["v0_field"] = v0f
    for precision in ("fp32", "fp64_arith", "fp64"):
        _, a = gpu_run(a11, a12, steps, options={"precision": precision}, **dict(kw))
        _, p = gpu_run(a11, a12, steps, options={"precision": precision, "schedule": "plain"}, **dict(kw))
        assert np.array_equal(a[-1][1], p[-1][1]) and np.array_equal(a[-1][2], p[-1][2]), precision


@pytest.mark.parametrize("limiter", ["none", "minmod", "theta", "superbee"])
def test_line_limiters_chunks_and_noalloc(fdm, limiter):
    import torch
    a11, a12, _ = _data(300)
    kw = dict(limiter=limiter, theta=1.3, cfl=0.4, v0=1.0)
    _, p = gpu_run(a11, a12, 24, options={"schedule": "plain"}, **kw)
    t11, t12 = to_dev(a11), to_dev(a12)
    ctx = fdm.fdm_transport_init(fdm.desc(300, 1, **kw))
    fdm.fdm_run(ctx, t11, t12, 24, 7)
    torch.cuda.synchronize()
    fdm.fdm_destroy(ctx)
    n11, n12 = to_dev(a11), to_dev(a12)
    fdm.fdm_transport_step_noalloc(fdm.desc(300, 1, **kw), n11, n12, 23)
    fdm.fdm_transport_step_noalloc(fdm.desc(300, 1, **kw), n11, n12, 1)
    torch.cuda.synchronize()
    for g11, g12 in ((t11, t12), (n11, n12)):
        assert np.array_equal(g11.cpu().numpy(), p[-1][1]) and np.array_equal(g12.cpu().numpy(), p[-1][2])
