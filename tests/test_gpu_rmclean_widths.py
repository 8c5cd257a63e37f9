"""RM-CLEAN at the edges of its register layouts: one element per lane more than
a width holds, a grid that ends inside the last element, more LOS than one
workgroup; and equal maxima, of which the lowest index is picked."""
import numpy as np
import pytest

import oracle
from oracle import rmclean as orc
import test_gpu_rmclean as base
from synthetic import band_lambda2, noise_sigma_F
from gpu_util import note

pytestmark = pytest.mark.gpu
_gpu = base._gpu


@pytest.mark.parametrize("nphi", [3, 64, 256, 257, 385, 513, 641, 769, 1025, 1281, 1537, 1793, 2049, 2561, 3073,
                                  3585, 4096])
def test_widths(nphi):
    """A valid run on every LOS (F = C * R + r, the stop, the restored spectrum) and
    the FP64 iteration's picks where those are clear, within test_gpu_rmclean's
    bar.  On the finest grids neighbours tie and no LOS need be clear."""
    note(f"rmclean width {nphi}")
    lam = band_lambda2(700.0, 1800.0, 300)
    w = np.ones(lam.size)
    w[::17] = 0.0
    phi = (np.arange(nphi) - nphi // 3) * (400.0 / nphi)
    Fq, Fu = base._cube(lam, w, phi, 7, 1e-3, seed=nphi)
    cutoff = 5 * noise_sigma_F(1e-3, w)
    g = base._run(lam, w, phi, Fq, Fu, 0.1, cutoff, 60)
    eps_R, R2, dphi = base._table_error(lam, w, phi)
    fwhm, _ = oracle.plan_info(lam, w)
    F = Fq.astype(np.float64) + 1j * Fu
    ref = orc.rmclean(F.real, F.imag, R2, dphi, 0.1, cutoff, 60, fwhm)
    clear = (ref["pick_margin"] > 1e-4) & (ref["stop_margin"] > 1e-4)
    bar = 2 * (np.maximum(g["niter"], ref["niter"]) + 1) * (eps_R + 2.0 ** -21) * np.abs(F).max(axis=1)
    resid, cc, rest = g["rq"] + 1j * g["ru"], g["cq"] + 1j * g["cu"], g["Rq"] + 1j * g["Ru"]
    np.testing.assert_array_equal(g["niter"][clear], ref["niter"][clear])
    for a, b in ((resid, ref["resid"]), (cc, ref["cc"]), (rest, ref["restored"])):
        assert np.all(np.abs(a - b).max(axis=1)[clear] <= bar[clear])
    k = np.arange(nphi)
    conv = np.stack([[np.sum(c * R2[(nphi - 1) + i - k]) for i in k] for c in cc])
    assert np.all(np.abs(conv + resid - F).max(axis=1) <= bar)
    done = g["niter"] < 60
    assert np.all(np.abs(resid[done]).max(axis=1, initial=0.0) < cutoff * (1 + 1e-4))
    beam = orc.restoring_beam(dphi * (k[:, None] - k[None, :]), fwhm)
    assert np.all(np.abs(rest - (resid + cc @ beam.T)).max(axis=1) <= bar)


@pytest.mark.parametrize("nphi", [130, 700, 2001])
def test_equal_maxima(nphi):
    """One iteration on spectra of one value at two places and 0 elsewhere: the
    component is gain times that value, exactly, at the lower place."""
    note(f"rmclean equal maxima {nphi}")
    rng = np.random.default_rng(nphi)
    n = 64
    at = np.sort(np.stack([rng.choice(nphi, 2, replace=False) for _ in range(n)]), axis=1)
    at[:3] = [[0, nphi - 1], [1, 65], [63, 64]]
    v = np.float32(0.75)
    Fq = np.zeros((n, nphi), np.float32)
    Fu = np.zeros((n, nphi), np.float32)
    Fq[np.arange(n), at[:, 0]] = v
    Fu[np.arange(n), at[:, 1]] = v  # the same power with another phase
    g = base._run(band_lambda2(700.0, 1800.0, 128), np.ones(128), np.linspace(-300, 300, nphi), Fq, Fu, 0.5, 0.1, 1)
    want = np.zeros((n, nphi), np.float32)
    want[np.arange(n), at[:, 0]] = np.float32(0.5) * v
    np.testing.assert_array_equal(g["cq"], want)
    np.testing.assert_array_equal(g["cu"], 0)
    np.testing.assert_array_equal(g["niter"], 1)
