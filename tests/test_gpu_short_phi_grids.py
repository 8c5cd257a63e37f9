"""Uniform grids of at most 128 phi: one tile of 64 mirrored pairs, on the first
two of four waves in small calls and on two waves, in pairs of tiles, in large
ones (half and full height, an odd number of tiles), against the oracle; the
same bits whatever the size of the call; fused peaks against execute + peaks."""
import numpy as np
import pytest

import oracle
import paper_1810_06250_amd as rs
from gpu_util import SCALE_TOL, dev32, host, note
from synthetic import FREQ_MAJOR, LOS_MAJOR, make_small_cube
from test_gpu_search import KEYS, _search_vs_execute

pytestmark = pytest.mark.gpu

# Channels: below a quad (single values), quads, ragged quads, K-steps of 16 with
# every remainder of 4.
SHAPES = [(40, 1, 1), (40, 3, 2), (70, 4, 63), (8257, 2, 128), (8257, 7, 64), (8193, 36, 65), (16449, 5, 127),
          (16400, 3, 100), (16449, 16, 20), (16385, 49, 128), (129, 130, 128)]


@pytest.fixture(autouse=True)
def _gpu():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    rs.load_library()
    oracle.build(force=False)


def _case(nlos, nchan, nphi, layout):
    c = make_small_cube(nlos, nchan, 3, seed=nlos + nchan, nflag=nchan // 5, nsrc=nlos // 8 + 1)
    phi = -37.0 + 1.3 * np.arange(nphi)
    Q, U = np.float32(c["Q"]), np.float32(c["U"])
    Q[:, c["weights"] == 0] = np.nan
    U[3, int(np.flatnonzero(c["weights"] > 0)[0])] = np.inf  # spoils LOS 3 alone
    return rs.Plan(c["lambda2"], c["weights"], phi), c, phi, Q, U


def _dev(X, layout):
    return dev32(np.ascontiguousarray(X.T) if layout == FREQ_MAJOR else X)


@pytest.mark.parametrize("prec", list(rs.PRECISIONS))
@pytest.mark.parametrize("layout", [LOS_MAJOR, FREQ_MAJOR], ids=["los", "freq"])
@pytest.mark.parametrize("shape", SHAPES, ids=lambda s: "x".join(map(str, s)))
def test_short_grids(prec, layout, shape):
    note(f"short phi grid {shape} layout={layout} {prec}")
    nlos = shape[0]
    plan, c, phi, Q, U = _case(*shape, layout)
    pick = np.setdiff1d(np.r_[0:min(nlos, 70), max(0, nlos - 70):nlos], [3])
    rq, ru = oracle.fdf(Q[pick].astype(np.float64), U[pick].astype(np.float64), c["lambda2"], c["weights"], phi)
    Fq, Fu, Fa = plan.execute(_dev(Q, layout), _dev(U, layout), layout, rs.PRECISIONS[prec], want_abs=True)
    Fq, Fu, Fa = host(Fq), host(Fu), host(Fa)
    # a handful of channels cancels: the error is taken relative to the larger of
    # max |F| and K sqrt(sum w^2 |P|^2)
    size = np.maximum(np.hypot(rq, ru).max(1), oracle.incoherent_scale(
        Q[pick].astype(np.float64), U[pick].astype(np.float64), c["weights"]))
    err = np.hypot(Fq[pick] - rq, Fu[pick] - ru).max(1)
    assert np.max(err / size) <= SCALE_TOL[prec]
    np.testing.assert_allclose(Fa[pick], np.hypot(Fq[pick].astype(np.float64), Fu[pick]), rtol=4e-7, atol=1e-30)
    assert not np.isfinite(Fq[3]).any() and not np.isfinite(Fu[3]).any()
    part = slice(nlos - 33, nlos)
    gq, gu, _ = plan.execute(_dev(Q[part], layout), _dev(U[part], layout), layout, rs.PRECISIONS[prec])
    np.testing.assert_array_equal(host(gq), Fq[part])
    np.testing.assert_array_equal(host(gu), Fu[part])
    plan.close()


@pytest.mark.parametrize("prec", ["bf16x3", "fp16x3"])
@pytest.mark.parametrize("layout", [LOS_MAJOR, FREQ_MAJOR], ids=["los", "freq"])
@pytest.mark.parametrize("shape", SHAPES, ids=lambda s: "x".join(map(str, s)))
def test_fused_peaks(prec, layout, shape):
    note(f"short phi grid, peaks {shape} layout={layout} {prec}")
    nlos = shape[0]
    plan, _, _, Q, U = _case(*shape, layout)
    Q, U = _dev(Q, layout), _dev(U, layout)
    out, Fq, Fu = _search_vs_execute(plan, Q, U, layout, prec, nlos)
    least = rs.rmsynth_search_workspace_size(plan.handle, 128, layout, rs.PRECISIONS[prec])
    _search_vs_execute(plan, Q, U, layout, prec, nlos, workspace_bytes=least)
    gq, gu, _, pk = plan.execute_peaks(Q, U, layout, rs.PRECISIONS[prec])
    np.testing.assert_array_equal(host(gq), Fq)
    np.testing.assert_array_equal(host(gu), Fu)
    for k in KEYS:
        np.testing.assert_array_equal(host(pk[k]), out[k], err_msg=k)
    assert out["idx"][3] == -1
    plan.close()


@pytest.mark.parametrize("prec", list(rs.PRECISIONS))
@pytest.mark.parametrize("nlos,nchan,nphi", [(40, 90, 77), (8257, 128, 33), (16400, 65, 20)])
def test_adjoint_onto_uniform_channels(prec, nlos, nchan, nphi):
    """Channels uniform in lambda^2 are the adjoint's uniform grid."""
    note(f"short grid of channels {nlos} x {nchan} x {nphi} {prec}")
    lam = np.linspace(0.03, 0.19, nchan)
    phi = -50.0 + 3.1 * np.arange(nphi)
    C = np.float32(np.random.default_rng(nchan).standard_normal((2, nlos, nphi)))
    plan = rs.Plan(lam, np.ones(nchan), phi)
    Pq, Pu = plan.adjoint(dev32(C[0]), dev32(C[1]), rs.PRECISIONS[prec])
    pick = np.unique(np.r_[0:min(nlos, 70), max(0, nlos - 70):nlos])
    D = C[:, pick].astype(np.float64)
    rq, ru = oracle.adjoint(D[0], D[1], lam, np.ones(nchan), phi)
    err = np.hypot(host(Pq)[pick] - rq, host(Pu)[pick] - ru).max(1)
    size = np.maximum(np.hypot(rq, ru).max(1), np.sqrt((D ** 2).sum((0, 2))))
    assert np.max(err / size) <= SCALE_TOL[prec]
    plan.close()
