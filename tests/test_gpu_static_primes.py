"""The static solve on both sides of the longest prime line it sums directly
(2887 and 2897 nodes), against the float64 oracle.  Bars as in
test_gpu_static_sizes.py: 4 log2(N) units in the last place in the 2-norm."""
import numpy as np
import pytest

from gpu_util import to_dev
from oracle import static as S
from paper_1911_03225_amd import workloads as W

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("nx,ny", [(2887, 6), (2897, 6), (6, 2887), (6, 2897)])
def test_prime_lines_match_oracle(nx, ny):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1911_03225_amd import fdm
    rng = np.random.default_rng(nx * 10007 + ny)
    a11, a12 = W.densities_from_phi(rng.standard_normal((ny, nx)))
    d = fdm.static_desc(nx, ny, layer_h=3.0, cell_l3=40.0, eps13=0.01, phi_mean=0.2)
    out = fdm.fdm_static_solve(d, to_dev(a11), to_dev(a12))
    torch.cuda.synchronize()
    ref = S.static_tau13(a11, a12, 1.0, 1.0, 1.0, 1.5, 3, 40, 0.01, 0.2)
    err = np.linalg.norm(out.cpu().numpy().astype(np.float64) - ref) / np.linalg.norm(ref)
    assert err <= 4 * np.log2(nx * ny) * 6e-8, err
