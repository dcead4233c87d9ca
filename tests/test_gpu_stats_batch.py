"""Diagnostics of batches (fdm_transport_stats on several instances)."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def fdm():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1911_03225_amd import fdm as F
    F.load_library()
    return F


def test_more_instances_than_a_grid_dimension_holds(fdm):
    """70000 instances: a launch's second dimension ends at 65535."""
    import torch
    n, nx, ny = 70000, 3, 2
    g = torch.Generator(device="cuda").manual_seed(1)
    a = torch.rand(n, ny, nx, device="cuda", generator=g)
    b = torch.rand(n, ny, nx, device="cuda", generator=g)
    ctx = fdm.fdm_transport_init([fdm.desc(nx, ny)] * n)
    t11, t12 = list(a), list(b)
    s11, s12 = a.double().sum((1, 2)).cpu().numpy(), b.double().sum((1, 2)).cpu().numpy()
    got = fdm.fdm_transport_stats(ctx, t11, t12)
    fdm.fdm_transport_step(ctx, t11, t12, 1)   # (no error stays behind)
    fdm.fdm_destroy(ctx)
    # six float values: their sums in double are exact to a few units of 2^-53 of 6
    assert np.allclose([s["sum11"] for s in got], s11, rtol=0, atol=1e-14)
    assert np.allclose([s["sum12"] for s in got], s12, rtol=0, atol=1e-14)
