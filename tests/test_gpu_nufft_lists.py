"""The NUFFT's gridding lists: threads per line of sight on either side of the
channel counts where small grids get one per point, lists of none, few and
many entries per point, on whole and 1/8 grids, and the 2048-point passes,
against the direct FP64 sum under the bar of test_gpu_nufft.py (1e-5 of
max |F|)."""
import numpy as np
import pytest

import oracle
import paper_1810_06250_amd as rs
from gpu_util import dev32, host, note
from synthetic import make_small_cube

pytestmark = pytest.mark.gpu


@pytest.fixture(autouse=True)
def _gpu():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    rs.load_library()
    oracle.build(force=False)


# The 120-168 MHz band covers 0.97 dphi of the circle (plus 8 cells): all of the
# grid at 1.0, at most 1/8 of 128 points and more at 0.05.
@pytest.mark.parametrize("dphi", [1.0, 0.05])
@pytest.mark.parametrize("nlos,nchan,nphi", [
    (37, 255, 16), (37, 256, 16), (5, 4096, 9),           # 32 points
    (19, 255, 32), (19, 256, 32), (3, 4096, 20),          # 64
    (21, 191, 64), (21, 192, 64), (3, 4096, 40),          # 128
    (21, 383, 128), (21, 384, 128), (3, 4096, 70),        # 256
    (9, 3, 200), (9, 400, 200), (3, 4096, 250),           # 512
    (5, 1, 600), (5, 64, 600), (5, 700, 1024),            # 2048
    (5, 40, 1500), (5, 100, 4001)])                       # 4096, 8192
def test_gridding_lists(nlos, nchan, nphi, dphi):
    note(f"nufft lists {nlos} x {nchan} x {nphi} step {dphi}")
    c = make_small_cube(nlos, nchan, 3, seed=nphi + nchan, nflag=nchan // 20, nsrc=nlos // 3 + 1,
                        phi_max=dphi * nphi / 2)
    phi = dphi * (np.arange(nphi) - nphi // 3)
    Q, U = np.float32(c["Q"]), np.float32(c["U"])
    Q[:, c["weights"] == 0] = np.nan
    plan = rs.Plan(c["lambda2"], c["weights"], phi)
    Fq, Fu, _ = plan.execute_nufft(dev32(Q), dev32(U))
    Fq, Fu = host(Fq), host(Fu)
    rq, ru = oracle.fdf(Q.astype(np.float64), U.astype(np.float64), c["lambda2"], c["weights"], phi)
    assert np.max(oracle.per_los_error(Fq, Fu, rq, ru)) <= 1e-5
    plan.close()
