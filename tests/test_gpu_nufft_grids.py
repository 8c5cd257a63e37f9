"""The NUFFT's short grids (a band that occupies at most 1/8 or 1/64 of the
grid) and its LOS-per-workgroup split, at every grid size, against the direct
FP64 sum under the bar of test_gpu_nufft.py (1e-5 of max |F|)."""
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


# nphi -> grid 128 .. 8192; the 120-168 MHz band covers 0.97 dphi of the circle
# (plus 8 cells): dphi 0.05 fits 1/8 of the grid, 0.002 fits 1/64 from 1024 on.
@pytest.mark.parametrize("dphi", [0.05, 0.002])
@pytest.mark.parametrize("nphi", [63, 100, 256, 401, 1000, 2001, 4001])
@pytest.mark.parametrize("nlos,nchan", [(1, 40), (37, 300)])
def test_short_grids(nlos, nchan, nphi, dphi):
    note(f"nufft short grid {nlos} x {nchan} x {nphi} step {dphi}")
    c = make_small_cube(nlos, nchan, 3, seed=nphi + nlos, nflag=nchan // 20, nsrc=nlos // 3 + 1, phi_max=dphi * nphi / 2)
    phi = 1.5 + dphi * np.arange(nphi)
    Q, U = np.float32(c["Q"]), np.float32(c["U"])
    plan = rs.Plan(c["lambda2"], c["weights"], phi)
    Fq, Fu, Fa = plan.execute_nufft(dev32(Q), dev32(U), want_abs=True)
    Fq, Fu, Fa = host(Fq), host(Fu), host(Fa)
    rq, ru = oracle.fdf(Q.astype(np.float64), U.astype(np.float64), c["lambda2"], c["weights"], phi)
    assert np.max(oracle.per_los_error(Fq, Fu, rq, ru)) <= 1e-5
    np.testing.assert_allclose(Fa, np.hypot(Fq, Fu), rtol=1e-6, atol=1e-30)
    plan.close()


def test_many_channels_on_a_small_grid():
    """3000 channels on a 512-point grid: the c_j then fill the LDS that several
    lines of sight would share."""
    note("nufft 3000 channels")
    c = make_small_cube(9, 3000, 3, seed=4, nflag=100, nsrc=4)
    phi = np.linspace(-60, 60, 241)
    Q, U = np.float32(c["Q"]), np.float32(c["U"])
    plan = rs.Plan(c["lambda2"], c["weights"], phi)
    Fq, Fu, _ = plan.execute_nufft(dev32(Q), dev32(U))
    rq, ru = oracle.fdf(Q.astype(np.float64), U.astype(np.float64), c["lambda2"], c["weights"], phi)
    assert np.max(oracle.per_los_error(host(Fq), host(Fu), rq, ru)) <= 1e-5
    plan.close()
