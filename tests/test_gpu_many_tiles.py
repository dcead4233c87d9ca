"""A batch whose fused tiles (56 columns) are more than one launch takes, at a
tile height that the stage kernels' tiles (60 columns) fit."""
import pytest

pytestmark = pytest.mark.gpu


def test_auto_takes_the_stage_kernels():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1911_03225_amd import fdm
    n, nx, ny = 17, 60, 1 << 20   # at one row a tile 17 x 2^20 tiles of 60 columns, twice that of 56; 2^25 fit
    descs = [fdm.desc(nx, ny, cfl=0.4)] * n
    with pytest.raises(fdm.FdmError) as e:
        fdm.fdm_transport_init(descs, options={"schedule": "fused", "tile_rows": 1})
    assert e.value.status == fdm.FDM_ERR_INVALID_ARG
    ctx = fdm.fdm_transport_init(descs, options={"tile_rows": 1})
    assert fdm.fdm_tile_rows(ctx, n - 1) == 1
    g = torch.Generator(device="cuda").manual_seed(1)
    t11 = [torch.randn(ny, nx, device="cuda", generator=g) for _ in range(n)]
    t12 = [torch.randn(ny, nx, device="cuda", generator=g) for _ in range(n)]
    a, b = t11[-1].clone(), t12[-1].clone()
    fdm.fdm_transport_step(ctx, t11, t12, 1)
    torch.cuda.synchronize()
    fdm.fdm_destroy(ctx)
    ctx = fdm.fdm_transport_init(descs[0])
    fdm.fdm_transport_step(ctx, a, b, 1)
    torch.cuda.synchronize()
    fdm.fdm_destroy(ctx)
    assert torch.equal(a, t11[-1]) and torch.equal(b, t12[-1])
