"""Wiggly-law runs in float64, whose solve returns tau13 and phi from one
complex transform, at lengths that take every form of the transforms:
powers of two and not, odd row lengths (one column is its own mirror, not
two), direct sums of a prime, tables left in memory.  Bars as in
test_gpu_coupled.py: 1e-10 against the float64 oracle."""
import numpy as np
import pytest

from gpu_util import to_dev
from oracle import coupled as CP
from paper_1911_03225_amd import workloads as W

pytestmark = pytest.mark.gpu

LOAD = dict(strain_rate13=2e-3, tau0=0.005, mobility=1.0, mu=1.0, lam=1.5, layer_h=3.0, cell_l3=24.0,
            dt_max=0.25, eps13=0.02, law="wiggly", tau_y=0.01, beta=1e-3)


@pytest.fixture(scope="module")
def fdm():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1911_03225_amd import fdm as F
    F.load_library()
    return F


def run(fdm, a11, a12, n_steps, chunk, phi_mean, **load):
    import torch
    ny, nx = a11.shape
    t11, t12 = to_dev(a11, np.float64), to_dev(a12, np.float64)
    ctx = fdm.fdm_transport_init(fdm.desc(nx, ny, cfl=0.4, v0=-1.0), options={"precision": "fp64"})
    hist = fdm.fdm_run(ctx, t11, t12, n_steps, chunk, loading=fdm.loading(phi_mean=phi_mean, **dict(LOAD, **load)))
    torch.cuda.synchronize()
    fdm.fdm_destroy(ctx)
    return [h[0] for h in hist], t11.cpu().numpy(), t12.cpu().numpy()


# 64 x 128: powers of two; 96 x 80; 75 x 48: odd row; 93 x 76: primes 31 and 19
# by direct sums; 56 x 1440: columns whose tables stay in memory
SIZES = [(64, 128), (96, 80), (75, 48), (93, 76), (56, 1440)]


@pytest.mark.parametrize("nx,ny", SIZES)
def test_two_runs_give_the_same_bits_and_follow_the_oracle(fdm, nx, ny):
    """Every value of the spectrum has one writer: a run repeats bit for bit,
    whatever its chunks."""
    phi, a11, a12 = W.plateau_rings(nx, ny, seed=5, count=4, rmin=6.0, rmax=14.0)
    n, mean = 24, float(phi.mean())
    hist, g11, g12 = run(fdm, a11, a12, n, 12, mean)
    for chunk in (12, 12, 5):
        h, r11, r12 = run(fdm, a11, a12, n, chunk, mean)
        assert np.array_equal(g11, r11) and np.array_equal(g12, r12), chunk
        for k in ("t", "dt", "eps13", "sigma13", "phi_mean", "vmax"):
            assert h[-1][k] == hist[-1][k], (chunk, k)
    o11, o12, ohist = CP.coupled_run(a11, a12, n, 12, cfl=0.4, dx=1.0, phi_mean=mean, **LOAD)
    for g, o in zip(hist, ohist):
        for k in ("t", "eps13", "phi_mean", "sigma13"):
            assert g[k] == pytest.approx(o[k], rel=1e-10, abs=1e-13), (k, g[k], o[k])
    den = np.abs(a11).sum() + np.abs(a12).sum()
    assert (np.abs(g11 - o11).sum() + np.abs(g12 - o12).sum()) / den < 1e-10


@pytest.mark.parametrize("power", [30, -30])
def test_units_of_stress_do_not_matter(fdm, power):
    """The same problem with every stress times a power of two and the
    mobility divided by it takes the same steps bit for bit: phi does not
    lose digits to a stress of another magnitude, nor the stress to phi."""
    nx, ny = 96, 80
    phi, a11, a12 = W.plateau_rings(nx, ny, seed=5, count=4, rmin=6.0, rmax=14.0)
    mean, s = float(phi.mean()), 2.0 ** power
    hist, g11, g12 = run(fdm, a11, a12, 24, 12, mean)
    h, r11, r12 = run(fdm, a11, a12, 24, 12, mean, mu=LOAD["mu"] * s, lam=LOAD["lam"] * s, tau_y=LOAD["tau_y"] * s,
                      mobility=LOAD["mobility"] / s)
    assert np.array_equal(g11, r11) and np.array_equal(g12, r12)
    for k in ("t", "dt", "eps13", "phi_mean", "vmax"):
        assert h[-1][k] == hist[-1][k], k
    assert h[-1]["sigma13"] == hist[-1]["sigma13"] * s


def test_stresses_in_pascals_follow_the_oracle(fdm):
    nx, ny = 75, 48
    phi, a11, a12 = W.plateau_rings(nx, ny, seed=5, count=4, rmin=6.0, rmax=14.0)
    load = dict(LOAD, mu=80e9, lam=120e9, tau_y=0.8e9, mobility=1.0 / 80e9)
    hist, g11, g12 = run(fdm, a11, a12, 24, 12, float(phi.mean()), **load)
    o11, o12, ohist = CP.coupled_run(a11, a12, 24, 12, cfl=0.4, dx=1.0, phi_mean=float(phi.mean()), **load)
    for g, o in zip(hist, ohist):
        for k in ("t", "eps13", "phi_mean", "sigma13"):
            assert g[k] == pytest.approx(o[k], rel=1e-10), (k, g[k], o[k])
    den = np.abs(a11).sum() + np.abs(a12).sum()
    assert (np.abs(g11 - o11).sum() + np.abs(g12 - o12).sum()) / den < 1e-10
