"""The autotuner on an AUTO context of one row, whose steps go by the one-row
kernel whatever the tiling."""
import numpy as np
import pytest

from gpu_util import to_dev

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def fdm():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1911_03225_amd import fdm as F
    F.load_library()
    return F


@pytest.mark.parametrize("precision,time_order", [("fp32", 2), ("fp32", 1), ("fp64", 2)])
@pytest.mark.parametrize("trial_steps", [1, 5])
def test_one_trial_and_the_context_stays(fdm, precision, time_order, trial_steps):
    """One trial, named as the context is, and no height of the trials stays
    behind: a coupled run's tiling, and so the sums of its mean slip, are
    those of a context that was not tuned."""
    rng = np.random.default_rng(4)
    phi = np.repeat(np.sin(2 * np.pi * np.arange(700) / 700) + 0.1 * rng.standard_normal(700), 1)[None, :]
    a12 = (np.roll(phi, -1, 1) - phi).astype(np.float32)
    dt = np.float64 if precision == "fp64" else np.float32
    load = fdm.loading(layer_h=3.0, cell_l3=24.0, tau0=0.001, eps13=0.02)
    out = []
    for tune in (True, False):
        t11, t12 = to_dev(np.zeros_like(a12), dt), to_dev(a12, dt)
        ctx = fdm.fdm_transport_init(fdm.desc(700, 1, cfl=0.25, time_order=time_order),
                                     options={"precision": precision})
        rows = fdm.fdm_tile_rows(ctx)
        if tune:
            trials = fdm.fdm_autotune(ctx, t11, t12, trial_steps=trial_steps)
            assert len(trials) == 1 and trials[0]["tile_rows"] == rows and trials[0]["seconds_per_step"] > 0
            assert trials[0]["schedule"] == ("fused" if precision == "fp32" else "plain")
        assert fdm.fdm_tile_rows(ctx) == rows
        fdm.fdm_transport_step(ctx, t11, t12, 7)
        h = fdm.fdm_run(ctx, t11, t12, 5, 5, loading=load)[-1][0]
        out.append((t11.cpu().numpy(), t12.cpu().numpy(), h["phi_mean"]))
        fdm.fdm_destroy(ctx)
    assert np.array_equal(out[0][0], out[1][0]) and np.array_equal(out[0][1], out[1][1]) and out[0][2] == out[1][2]
