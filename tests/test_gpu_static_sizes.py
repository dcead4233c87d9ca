"""The static solve's own transforms at the lengths where a pass can go wrong:
every radix and mixtures, single passes, one node, primes (direct sums),
lines whose tables do not fit beside them in LDS and lines that do not fit at
all, thin shapes of both kinds, against the float64 oracle.

Bars: the transforms of a line of n round like log2(n) units in the last
place in the 2-norm and the low modes of phi carry that error n / (2 pi)
times; tau13 itself divides it out again (K falls off with |xi|), so 4 log2(N)
units in the last place (6e-8 or 1.1e-16) are allowed, four times what a
solve of either library measures."""
import numpy as np
import pytest

from gpu_util import to_dev
from oracle import static as S
from paper_1911_03225_amd import workloads as W

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def fdm():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1911_03225_amd import fdm as F
    F.load_library()
    return F


SIZES = [(1, 1), (1, 64), (64, 1), (2, 3), (5, 8), (9, 7), (16, 25), (49, 50), (61, 64), (64, 62), (128, 96),
         (256, 100), (360, 243), (320, 125), (1000, 63), (509, 48), (4096, 8), (16, 2048), (2053, 6), (6, 5000)]


@pytest.mark.parametrize("nx,ny", SIZES)
@pytest.mark.parametrize("precision", ["fp32", "fp64"])
def test_sizes_match_oracle(fdm, nx, ny, precision):
    import torch
    rng = np.random.default_rng(nx * 10007 + ny)
    a11, a12 = W.densities_from_phi(rng.standard_normal((ny, nx)))
    h, n3 = 3, 40
    dt = np.float64 if precision == "fp64" else np.float32
    d = fdm.static_desc(nx, ny, layer_h=float(h), cell_l3=float(n3), eps13=0.01, phi_mean=0.2, precision=precision)
    out = fdm.fdm_static_solve(d, to_dev(a11, dt), to_dev(a12, dt))
    torch.cuda.synchronize()
    ref = S.static_tau13(a11, a12, 1.0, 1.0, 1.0, 1.5, h, n3, 0.01, 0.2)
    err = np.linalg.norm(out.cpu().numpy().astype(np.float64) - ref) / np.linalg.norm(ref)
    eps = 1.1e-16 if precision == "fp64" else 6e-8
    assert err <= 4 * max(1.0, np.log2(nx * ny)) * eps, err
