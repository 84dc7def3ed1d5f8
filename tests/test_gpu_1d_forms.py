"""The 1-D kernel at one lane a replica against 16, over what the lane-split tests
leave out (needs an MI355X): the harmonic potential, the unrestrained ensemble
(exponents quadratic in xi), a pull, histograms at the most bins held in LDS and
one more, samples outside them.  The first replicas of window 1 (whose reverse
exponent is quadratic here) agree bit for bit; histograms add up to the samples."""
import numpy as np
import pytest

import paper_1105_4840_amd as ppp
import ppp_inputs

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")

FEW, MANY = 37, 44445          # three ensembles: 16 lanes a replica, and one


def _records(p):
    h = ppp.ppp_create(p)
    try:
        ws = ppp.workspace(h)
        ppp.ppp_begin(h, ws)
        ppp.ppp_advance(h, 50)
        ppp.ppp_advance(h, 10 ** 9)
        blob = ppp.ppp_checkpoint(h)
        ppp.ppp_finalize(h)
        res = ppp.ppp_get_result(h, p)
    finally:
        ppp.ppp_destroy(h)
    n = 3 * p["n_replicas"]
    dt = np.float64 if p["precision"] == "fp64" else np.float32
    state = np.frombuffer(blob, dtype=dt, count=2 * n, offset=16)
    at = 16 + -(-state.nbytes // 256) * 256
    acc = np.frombuffer(blob, dtype=np.float64, count=16 * n, offset=at).reshape(3, -1, 16)
    return state.reshape(3, -1, 2), acc, res


@pytest.mark.parametrize("precision", ["fp64", "fp32"])
@pytest.mark.parametrize("bins", [64, 16384, 16385])
@pytest.mark.parametrize("every,pull", [(1, 0), (2, 20), (7, 0)])
def test_one_lane_and_sixteen_agree(precision, bins, every, pull):
    print(f"case 1-D forms {precision} bins={bins} every={every} pull={pull}", flush=True)
    p = ppp_inputs.config_harmonic_1d(n_steps=203, seed=4, precision=precision)
    # bins that some samples miss, a bound that some replicas cross
    p.update({"lambda": [-1.0, -0.9], "free_ensemble": True, "n_equil": 30, "n_pull": pull, "sample_every": every,
              "w_half_bins": 0, "n_blocks": 4, "xi_min": -1.1, "xi_bin": 0.3 / bins, "xi_nbins": bins, "xi_bound": 1.35})
    s1, a1, _ = _records(dict(p, n_replicas=FEW))
    s2, a2, res = _records(dict(p, n_replicas=MANY))
    assert 0 < a1[0, :, 13].sum() and 0 < a1[0, :, 14].sum()          # some below, some above the bins
    assert np.array_equal(s1[0], s2[0, :FEW]) and np.array_equal(a1[0], a2[0, :FEW])
    inside = res["n_samples"] - res["xi_under_over"].sum(axis=1).astype(np.int64)
    assert np.array_equal(res["xi_hist"].astype(np.int64).sum(axis=1), inside)
    # the other ensembles: every replica that was not frozen has all its samples, and the
    # maxima of 2a are twice those of a
    for w in (1, 2):
        a = a2[w]
        full = a[:, 15] == 0
        assert np.array_equal(a[full, 0], np.full(full.sum(), float(len(range(30 + every, 204, every)))))
        assert np.array_equal(a[:, 7], 2.0 * a[:, 5]) and np.array_equal(a[:, 11], 2.0 * a[:, 9])


@pytest.mark.parametrize("precision", ["fp64", "fp32"])
def test_short_trajectories_are_the_start_of_long_ones(precision):
    """A few steps run at one lane a replica, more at sixteen: the same positions."""
    p = ppp_inputs.config_1d(n_replicas=131, n_steps=400, n_windows=3, seed=6, precision=precision)
    p.update({"n_equil": 3, "sample_every": 4})
    h = ppp.ppp_create(p)
    try:
        ws = ppp.workspace(h)
        for window, replica in ((0, 0), (1, 130), (2, 77)):
            long = ppp.ppp_trajectory(h, ws, window, replica, 400, 1).cpu().numpy()
            for n in (1, 4, 16, 33):
                short = ppp.ppp_trajectory(h, ws, window, replica, n, 1).cpu().numpy()
                assert np.isfinite(short).all() and np.array_equal(short, long[:n + 1]), (window, replica, n)
    finally:
        ppp.ppp_destroy(h)
