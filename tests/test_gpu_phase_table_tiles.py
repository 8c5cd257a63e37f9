"""The 128-column tiles of the phase-table form (two to a workgroup, one below
the other), which irregular grids take in both layouts where 256-column tiles
would pad more: full and half-height tiles of lines of sight, an odd number of
them, stored F and the fused peaks."""
import numpy as np
import pytest

import oracle
import paper_1810_06250_amd as rs
from gpu_util import SCALE_TOL, dev32, host, note
from synthetic import FREQ_MAJOR, LOS_MAJOR, make_small_cube
from test_gpu_search import KEYS, _search_vs_execute

pytestmark = pytest.mark.gpu

# 100 phi: wide tiles in half height, narrow ones in half and in full height, an
# odd and an even number of them; the same with a ragged third tile (300, 384) and
# five tiles instead of three (600).
SHAPES = [(33, 9, 100), (8300, 11, 100), (16383, 9, 90), (16449, 20, 100), (16385, 21, 128), (65, 40, 300),
          (4097, 12, 300), (8200, 23, 300), (8193, 17, 384), (129, 33, 600), (5441, 8, 600), (40, 1, 1)]


@pytest.fixture(autouse=True)
def _gpu():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    rs.load_library()
    oracle.build(force=False)


def _case(nlos, nchan, nphi):
    c = make_small_cube(nlos, nchan, 3, seed=nlos + nchan, nflag=nchan // 8, nsrc=nlos // 8 + 1)
    phi = np.sort(np.random.default_rng(nphi).uniform(-100, 100, nphi))
    Q, U = np.float32(c["Q"]), np.float32(c["U"])
    Q[:, c["weights"] == 0] = np.nan
    if nlos > 4:
        U[3, int(np.flatnonzero(c["weights"] > 0)[0])] = np.inf  # spoils LOS 3 alone
    return c, phi, Q, U


@pytest.mark.parametrize("prec", list(rs.PRECISIONS))
@pytest.mark.parametrize("layout", [LOS_MAJOR, FREQ_MAJOR], ids=["los", "freq"])
@pytest.mark.parametrize("shape", SHAPES, ids=lambda s: "x".join(map(str, s)))
def test_narrow_tiles(prec, layout, shape):
    note(f"narrow table tiles {shape} layout={layout} {prec}")
    nlos, nchan, nphi = shape
    c, phi, Q, U = _case(*shape)
    pick = np.setdiff1d(np.r_[0:min(nlos, 70), max(0, nlos - 70):nlos], [3])
    plan = rs.Plan(c["lambda2"], c["weights"], phi)
    rq, ru = oracle.fdf(Q[pick].astype(np.float64), U[pick].astype(np.float64), c["lambda2"], c["weights"], phi)
    if layout == FREQ_MAJOR:
        Q, U = np.ascontiguousarray(Q.T), np.ascontiguousarray(U.T)
    Fq, Fu, _ = plan.execute(dev32(Q), dev32(U), layout, rs.PRECISIONS[prec])
    Fq, Fu = host(Fq), host(Fu)
    assert np.max(oracle.per_los_error(Fq[pick], Fu[pick], rq, ru)) <= SCALE_TOL[prec]
    if nlos > 4:
        assert not np.isfinite(Fq[3]).any() and not np.isfinite(Fu[3]).any()
    plan.close()


@pytest.mark.parametrize("prec", ["bf16x3", "fp16x3"])
@pytest.mark.parametrize("layout", [LOS_MAJOR, FREQ_MAJOR], ids=["los", "freq"])
@pytest.mark.parametrize("shape", SHAPES, ids=lambda s: "x".join(map(str, s)))
def test_fused_peaks_on_narrow_tiles(prec, layout, shape):
    """Search and execute_peaks give bit for bit what execute and peaks give."""
    note(f"narrow table tiles, peaks {shape} layout={layout} {prec}")
    nlos, nchan, nphi = shape
    c, phi, Q, U = _case(*shape)
    plan = rs.Plan(c["lambda2"], c["weights"], phi)
    if layout == FREQ_MAJOR:
        Q, U = np.ascontiguousarray(Q.T), np.ascontiguousarray(U.T)
    Q, U = dev32(Q), dev32(U)
    out, Fq, Fu = _search_vs_execute(plan, Q, U, layout, prec, nlos)
    gq, gu, _, pk = plan.execute_peaks(Q, U, layout, rs.PRECISIONS[prec])
    np.testing.assert_array_equal(host(gq), Fq)
    np.testing.assert_array_equal(host(gu), Fu)
    for k in KEYS:
        np.testing.assert_array_equal(host(pk[k]), out[k], err_msg=k)
    if nlos > 4:
        assert out["idx"][3] == -1
    plan.close()
