"""FP32 transforms at the edges of the rule that sends few channels and few phi to
the kernel that generates its phases, against the oracle: uniform and irregular
grids in both layouts, flagged and non-finite channels, a ragged last tile of
lines of sight, and the adjoint on a uniform phi grid."""
import numpy as np
import pytest

import oracle
import paper_1810_06250_amd as rs
from gpu_util import SCALE_TOL, dev32, host, note
from synthetic import FREQ_MAJOR, LOS_MAJOR, make_small_cube

pytestmark = pytest.mark.gpu

# (nlos, nchan, nphi): the last size of each part of the rule and the next one.
SHAPES = [(70, 1, 1), (129, 3, 96), (200, 8, 96), (200, 8, 97), (65, 9, 64), (130, 16, 64), (130, 16, 65),
          (67, 17, 33), (130, 24, 32), (63, 25, 32), (8200, 7, 20)]


@pytest.fixture(autouse=True)
def _gpu():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    rs.load_library()
    oracle.build(force=False)


@pytest.mark.parametrize("layout", [LOS_MAJOR, FREQ_MAJOR], ids=["los", "freq"])
@pytest.mark.parametrize("grid", ["uniform", "irregular"])
@pytest.mark.parametrize("shape", SHAPES, ids=lambda s: "x".join(map(str, s)))
def test_transform(grid, layout, shape):
    note(f"few channels FP32 {shape} {grid} layout={layout}")
    nlos, nchan, nphi = shape
    c = make_small_cube(nlos, nchan, 3, seed=nlos + nchan, nflag=nchan // 4, nsrc=nlos // 8 + 1)
    phi = -41.0 + 1.7 * np.arange(nphi)
    if grid == "irregular":
        phi = phi + np.random.default_rng(nphi).uniform(-0.4, 0.4, nphi)
    Q, U = np.float32(c["Q"]), np.float32(c["U"])
    Q[:, c["weights"] == 0] = np.nan
    U[3, int(np.flatnonzero(c["weights"] > 0)[0])] = np.inf  # spoils LOS 3 alone
    pick = np.setdiff1d(np.r_[0:min(nlos, 70), max(0, nlos - 70):nlos], [3])
    q64, u64 = Q[pick].astype(np.float64), U[pick].astype(np.float64)
    rq, ru = oracle.fdf(q64, u64, c["lambda2"], c["weights"], phi)
    size = np.maximum(np.hypot(rq, ru).max(1), oracle.incoherent_scale(q64, u64, c["weights"]))
    if layout == FREQ_MAJOR:
        Q, U = np.ascontiguousarray(Q.T), np.ascontiguousarray(U.T)
    plan = rs.Plan(c["lambda2"], c["weights"], phi)
    Fq, Fu, Fa = (host(x) for x in plan.execute(dev32(Q), dev32(U), layout, rs.RMSYNTH_FP32, want_abs=True))
    err = np.hypot(Fq[pick] - rq, Fu[pick] - ru).max(1)
    assert np.max(err / size) <= SCALE_TOL["fp32"]
    np.testing.assert_allclose(Fa[pick], np.hypot(Fq[pick].astype(np.float64), Fu[pick]), rtol=4e-7, atol=1e-30)
    assert not np.isfinite(Fq[3]).any() and not np.isfinite(Fu[3]).any()
    plan.close()


@pytest.mark.parametrize("nlos,nchan,nphi", [(70, 640, 16), (70, 641, 16), (130, 300, 17), (65, 300, 2), (8200, 257, 5),
                                             (70, 32, 24), (70, 33, 24), (130, 9, 25)])
def test_adjoint(nlos, nchan, nphi):
    note(f"few phi FP32 adjoint {nlos} x {nphi} -> {nchan}")
    c = make_small_cube(2, nchan, 3, seed=nchan)
    phi = -50.0 + 3.1 * np.arange(nphi)
    C = np.float32(np.random.default_rng(nchan).standard_normal((2, nlos, nphi)))
    plan = rs.Plan(c["lambda2"], c["weights"], phi)
    Pq, Pu = plan.adjoint(dev32(C[0]), dev32(C[1]), rs.RMSYNTH_FP32)
    pick = np.unique(np.r_[0:min(nlos, 70), max(0, nlos - 70):nlos])
    D = C[:, pick].astype(np.float64)
    rq, ru = oracle.adjoint(D[0], D[1], c["lambda2"], c["weights"], phi)
    err = np.hypot(host(Pq)[pick] - rq, host(Pu)[pick] - ru).max(1)
    size = np.maximum(np.hypot(rq, ru).max(1), np.sqrt((D ** 2).sum((0, 2))))
    assert np.max(err / size) <= SCALE_TOL["fp32"]
    plan.close()
