"""The mirrored-pair transform (uniform phi grids) at the edges of its tiles:
64 LOS, 256 phi (32 pairs per wave), 16 channels per K-step in quads, the three
ways Q/U are read, every precision, against the oracle."""
import numpy as np
import pytest

import oracle
import paper_1810_06250_amd as rs
from gpu_util import SCALE_TOL, dev32, host, note
from synthetic import FREQ_MAJOR, LOS_MAJOR, make_small_cube

pytestmark = pytest.mark.gpu


@pytest.fixture(autouse=True)
def _gpu():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    rs.load_library()


# (nlos, nchan, nphi): one below, at and above each tile edge; nchan 4 n reads
# quads, odd nchan single values; 15-17, 31-36 and 47-49 channels end the
# K-loop after one, two and three steps and leave every remainder.
EDGES = [(63, 15, 255), (64, 16, 256), (65, 17, 257), (1, 31, 511), (128, 32, 512), (3, 33, 513),
         (66, 36, 300), (129, 47, 223), (64, 48, 225), (70, 49, 289), (5, 20, 40)]


@pytest.mark.parametrize("prec", list(rs.PRECISIONS))
@pytest.mark.parametrize("layout", [LOS_MAJOR, FREQ_MAJOR], ids=["los", "freq"])
@pytest.mark.parametrize("shape", EDGES, ids=lambda s: "x".join(map(str, s)))
def test_tile_edges(prec, layout, shape):
    nlos, nchan, nphi = shape
    note(f"mirrored {shape} layout={layout} {prec}")
    c = make_small_cube(nlos, nchan, nphi, seed=nlos + 3 * nchan + nphi, nflag=nchan // 12, nsrc=nlos // 8 + 1)
    plan = rs.Plan(c["lambda2"], c["weights"], c["phi"])
    Q, U = np.float32(c["Q"]), np.float32(c["U"])
    rq, ru = oracle.fdf(Q.astype(np.float64), U.astype(np.float64), c["lambda2"], c["weights"], c["phi"])
    if layout == FREQ_MAJOR:
        Q, U = np.ascontiguousarray(Q.T), np.ascontiguousarray(U.T)
    Fq, Fu, Fa = plan.execute(dev32(Q), dev32(U), layout, rs.PRECISIONS[prec], want_abs=True)
    Fq, Fu, Fa = host(Fq), host(Fu), host(Fa)
    assert np.max(oracle.per_los_error(Fq, Fu, rq, ru)) <= SCALE_TOL[prec]
    # |F| is the FP32 square root of the FP32 sum of squares of what is stored
    np.testing.assert_allclose(Fa, np.hypot(Fq.astype(np.float64), Fu), rtol=4e-7, atol=0)
    plan.close()


@pytest.mark.parametrize("prec", list(rs.PRECISIONS))
@pytest.mark.parametrize("nchan,skip", [(1, 0), (2, 1), (3, 3), (4, 1), (5, 0), (6, 2), (7, 3), (18, 1), (19, 0),
                                        (33, 2), (36, 3), (66, 1), (111, 3)])
def test_row_quads(prec, nchan, skip):
    """LOS-major rows are read as quads of any alignment, the last from the row's
    last 4 channels: bases `skip` floats off, NaN on both sides of the cube, a
    channel of weight 0 holding NaN, full and half-height tiles."""
    note(f"row quads {nchan} channels, {skip} floats off, {prec}")
    import torch
    for nlos, nphi in ((70, 60), (8300, 300)):
        c = make_small_cube(nlos, nchan, 3, seed=nchan + nlos, nflag=nchan // 8, nsrc=8)
        phi = np.linspace(-80.0, 90.0, nphi)
        Q, U = np.float32(c["Q"]), np.float32(c["U"])
        Q[:, c["weights"] == 0] = np.nan
        dev = []
        for X in (Q, U):
            buf = torch.full((skip + X.size + 5,), float("nan"), dtype=torch.float32, device="cuda")
            dev.append(buf[skip:skip + X.size].view(nlos, nchan))
            dev[-1].copy_(torch.from_numpy(X))
        pick = np.r_[0:70, nlos - 70:nlos]
        plan = rs.Plan(c["lambda2"], c["weights"], phi)
        rq, ru = oracle.fdf(Q[pick].astype(np.float64), U[pick].astype(np.float64), c["lambda2"], c["weights"], phi)
        Fq, Fu, _ = plan.execute(dev[0], dev[1], LOS_MAJOR, rs.PRECISIONS[prec])
        assert np.max(oracle.per_los_error(host(Fq)[pick], host(Fu)[pick], rq, ru)) <= SCALE_TOL[prec]
        plan.close()


@pytest.mark.parametrize("layout", [LOS_MAJOR, FREQ_MAJOR], ids=["los", "freq"])
@pytest.mark.parametrize("nlos", [1, 65, 4097, 65600])
@pytest.mark.parametrize("nchan", [1, 8, 33, 129, 257])
def test_half_scale_sees_every_channel(layout, nlos, nchan):
    """The per-LOS scale of the IEEE-half split is found by up to 16 waves that
    share the channels: LOS l has its one large value, 1e7 times the others (half
    overflows at 65504 unscaled), in channel l % nchan, of Q and U in turn."""
    note(f"half scale {nlos} x {nchan} layout={layout}")
    rng = np.random.default_rng(nchan)
    Q, U = (np.float32(1e-2 * rng.uniform(-1, 1, (nlos, nchan))) for _ in "QU")
    l = np.arange(nlos)
    for X, at in ((Q, l[0::2]), (U, l[1::2])):
        X[at, at % nchan] = 1e5
    c = make_small_cube(2, nchan, 3, seed=nchan)
    phi = np.linspace(-40.0, 50.0, 21)
    plan = rs.Plan(c["lambda2"], c["weights"], phi)
    pick = np.unique(np.r_[0:min(nlos, 300), max(0, nlos - 300):nlos])
    rq, ru = oracle.fdf(Q[pick].astype(np.float64), U[pick].astype(np.float64), c["lambda2"], c["weights"], phi)
    if layout == FREQ_MAJOR:
        Q, U = np.ascontiguousarray(Q.T), np.ascontiguousarray(U.T)
    Fq, Fu, _ = plan.execute(dev32(Q), dev32(U), layout, rs.RMSYNTH_SPLIT_FP16)
    assert np.max(oracle.per_los_error(host(Fq)[pick], host(Fu)[pick], rq, ru)) <= SCALE_TOL["fp16x3"]
    plan.close()


@pytest.mark.parametrize("prec", list(rs.PRECISIONS))
@pytest.mark.parametrize("nlos,nchan,nphi", [(1, 3, 2), (31, 40, 31), (33, 255, 32), (64, 256, 33), (65, 257, 255),
                                             (63, 64, 256), (66, 100, 257), (40, 130, 513), (9000, 70, 300)])
def test_folded_adjoint_edges(prec, nlos, nchan, nphi):
    """The adjoint on a uniform phi grid folds pairs of phi in K-tiles of at most
    256 (whole multiples of 32, padded below phi_0), 64 LOS x 256 channels per
    workgroup (32 LOS when there are few): one, two and three K-tiles with
    every remainder, against the direct FP64 sum.  Errors are taken relative
    to max(max |P|, sqrt(sum |C|^2)), the bound of a sum of independent
    products."""
    note(f"folded adjoint {nlos} x {nchan} x {nphi} {prec}")
    c = make_small_cube(2, nchan, 3, seed=nphi)
    phi = np.linspace(-90.0, 95.0, nphi)
    rng = np.random.default_rng(nlos + nphi)
    C = np.float32(rng.standard_normal((2, nlos, nphi)))
    plan = rs.Plan(c["lambda2"], c["weights"], phi)
    Pq, Pu = plan.adjoint(dev32(C[0]), dev32(C[1]), rs.PRECISIONS[prec])
    pick = np.unique(np.r_[0:min(nlos, 70), max(0, nlos - 70):nlos])
    D = C[:, pick].astype(np.float64)
    rq, ru = oracle.adjoint(D[0], D[1], c["lambda2"], c["weights"], phi)
    err = np.hypot(host(Pq)[pick] - rq, host(Pu)[pick] - ru).max(1)
    size = np.maximum(np.hypot(rq, ru).max(1), np.sqrt((D ** 2).sum((0, 2))))
    assert np.max(err / size) <= SCALE_TOL[prec]
    plan.close()


@pytest.mark.parametrize("prec", list(rs.PRECISIONS))
@pytest.mark.parametrize("nlos,nchan", [(70, 40), (33, 300), (8300, 130)])
@pytest.mark.parametrize("nphi", [1, 3, 5, 15, 17, 47, 129, 259])
def test_folded_pairs_at_row_ends(prec, nlos, nchan, nphi):
    """The folded adjoint reads two neighbouring phi at a time; those that start
    below phi_0 are read from phi_0 on.  A LOS of NaN must spoil no other."""
    note(f"folded pairs {nlos} x {nchan} x {nphi} {prec}")
    c = make_small_cube(2, nchan, 3, seed=nphi)
    phi = np.linspace(-70.0, 95.0, nphi)
    C = np.float32(np.random.default_rng(nlos + nphi).standard_normal((2, nlos, nphi)))
    C[:, 1] = np.nan
    plan = rs.Plan(c["lambda2"], c["weights"], phi)
    Pq, Pu = plan.adjoint(dev32(C[0]), dev32(C[1]), rs.PRECISIONS[prec])
    assert not np.isfinite(host(Pq)[1]).any() and not np.isfinite(host(Pu)[1]).any()
    pick = np.unique(np.r_[0, 2:min(nlos, 40), max(2, nlos - 40):nlos])
    D = C[:, pick].astype(np.float64)
    rq, ru = oracle.adjoint(D[0], D[1], c["lambda2"], c["weights"], phi)
    err = np.hypot(host(Pq)[pick] - rq, host(Pu)[pick] - ru).max(1)
    size = np.maximum(np.hypot(rq, ru).max(1), np.sqrt((D ** 2).sum((0, 2))))
    assert np.max(err / size) <= SCALE_TOL[prec]
    plan.close()


@pytest.mark.parametrize("prec", list(rs.PRECISIONS))
@pytest.mark.parametrize("layout", [LOS_MAJOR, FREQ_MAJOR], ids=["los", "freq"])
@pytest.mark.parametrize("nlos,nchan,nphi", [(1, 7, 40), (31, 8, 255), (33, 9, 256), (64, 16, 257), (65, 23, 100),
                                             (9001, 25, 513)])
def test_phase_table_edges(prec, layout, nlos, nchan, nphi):
    """Irregular grids contract 8 channels per K-step against the plan's phase
    table: one below, at and above a K-step, one to four of them, ragged LOS
    and phi tiles, channels of weight 0 holding NaN, both heights of LOS tile."""
    note(f"phase table {nlos} x {nchan} x {nphi} layout={layout} {prec}")
    c = make_small_cube(nlos, nchan, 3, seed=nlos + nchan, nflag=nchan // 8, nsrc=nlos // 8 + 1)
    phi = np.sort(np.random.default_rng(nphi).uniform(-100, 100, nphi))
    Q, U = np.float32(c["Q"]), np.float32(c["U"])
    Q[:, c["weights"] == 0] = np.nan
    pick = np.unique(np.r_[0:min(nlos, 70), max(0, nlos - 70):nlos])
    plan = rs.Plan(c["lambda2"], c["weights"], phi)
    rq, ru = oracle.fdf(Q[pick].astype(np.float64), U[pick].astype(np.float64), c["lambda2"], c["weights"], phi)
    if layout == FREQ_MAJOR:
        Q, U = np.ascontiguousarray(Q.T), np.ascontiguousarray(U.T)
    Fq, Fu, _ = plan.execute(dev32(Q), dev32(U), layout, rs.PRECISIONS[prec])
    assert np.max(oracle.per_los_error(host(Fq)[pick], host(Fu)[pick], rq, ru)) <= SCALE_TOL[prec]
    plan.close()
