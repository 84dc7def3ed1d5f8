"""Leave-one-out errors of the estimators where a lane holds several jackknife
blocks (more than 64 of them), where blocks are uneven or empty, and where one
block outweighs all others (needs an MI355X)."""
import struct

import numpy as np
import pytest

import paper_1105_4840_amd as ppp
import ppp_inputs
import oracle
from oracle import estimators

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


def _problem(replicas, blocks, **kw):
    p = ppp_inputs.config_1d(n_replicas=replicas, n_steps=400, n_windows=3, seed=5, precision="fp64")
    p.update({"lambda": [-1.0, -0.9, -0.8], "n_equil": 20, "w_half_bins": 0, "n_blocks": blocks, "xi_min": -2.5,
              "xi_bin": 5.0 / 64, "xi_nbins": 64}, **kw)
    return p


@pytest.mark.parametrize("replicas,blocks", [(203, 64), (203, 65), (203, 130), (331, 300), (193, 193)])
def test_many_blocks_match_the_oracle(replicas, blocks):
    """With frozen replicas, so that blocks hold different numbers of samples (the
    last case has a block per replica).  Positions agree with the oracle's to some
    1e-12, a leave-one-out value of order one then to 1e-11, and a standard error,
    sqrt((B - 1) / B sum of squares), to sqrt(B) 1e-11."""
    print(f"case jackknife R={replicas} B={blocks}", flush=True)
    p = _problem(replicas, blocks, free_ensemble=True, xi_bound=1.3)
    res, _ = ppp.run(p)
    xi, kept, _ = oracle.run(p)
    ref = estimators.estimate(p, xi, kept)
    frozen = int(ref["n_blown_up"].sum()) + ref["turn_on"]["free_blown"]
    print(f"  frozen {frozen}, without samples {int((kept == 0).sum())}", flush=True)
    assert frozen > 3
    assert np.array_equal(res["n_samples"], ref["n_samples"]) and np.array_equal(res["n_blown_up"], ref["n_blown_up"])
    tol = dict(rtol=1e-9, atol=np.sqrt(blocks) * 1e-11)
    for key in ("dF_je_se", "dF_fluct_se", "dF_gauss_se", "dF_com_se"):
        assert np.isfinite(ref[key]).all() and np.allclose(res[key], ref[key], **tol), key
    assert np.allclose(res["G_se"], ref["G_se"], **tol)
    for key in ("eq5_first_se", "eq6_first_se", "eq5_last_se", "eq6_last_se", "eq10_log_se"):
        assert np.isclose(res["turn_on"][key], ref["turn_on"][key], **tol), key


@pytest.mark.parametrize("blocks", [32, 70])
@pytest.mark.parametrize("size", [1e3, 1e7, 1e60])
def test_one_block_outweighs_the_others(size, blocks):
    """One replica's record in a checkpoint gets moments as of samples near `size`;
    the errors of Eqs. 13 and 14 against the same sums in 64-bit-mantissa floats.
    A leave-one-out moment formed as total minus block is off by rounding of the
    total there, which the error, as large as the total's share, does not show:
    each value is good to some 100 roundings of the largest."""
    R, s = 70, 3
    print(f"case jackknife outlier {size} B={blocks}", flush=True)
    p = _problem(R, blocks)
    h = ppp.ppp_create(p)
    try:
        ws = ppp.workspace(h)
        ppp.ppp_begin(h, ws)
        ppp.ppp_advance(h, 10 ** 9)
        blob = bytearray(ppp.ppp_checkpoint(h))
        at = 16 + -(-(2 * s * R * 8) // 256) * 256
        acc = np.frombuffer(blob, dtype=np.float64, count=16 * s * R, offset=at).reshape(s, R, 16).copy()
        acc[1, 41, 1] = size * acc[1, 41, 0] * 0.75
        acc[1, 41, 2] = size * size * acc[1, 41, 0]
        blob[at:at + acc.nbytes] = acc.tobytes()
        assert struct.unpack_from("<q", blob, 8)[0] == p["n_steps"]
        ppp.ppp_restore(h, ws, bytes(blob))
        ppp.ppp_finalize(h)
        res = ppp.ppp_get_result(h, p)
    finally:
        ppp.ppp_destroy(h)
    q = acc.astype(np.longdouble)
    block = (np.arange(R) * blocks) // R
    k, kT = p["k"], p["kT"]
    fl, ga = [], []
    for b in range(blocks):
        n, s1, s2 = (q[:, block != b, f].sum(axis=1) for f in range(3))
        m = s1 / n
        var = (s2 - n * m * m) / (n - 1)
        dl = np.diff(np.asarray(p["lambda"], dtype=np.longdouble))
        f = -k * dl * m[:-1]
        fl.append(np.cumsum(f))
        ga.append(np.cumsum(f + k * dl * dl / 2 * (1 - k * var[:-1] / kT)))
    for key, v in (("dF_fluct_se", fl), ("dF_gauss_se", ga)):
        v = np.array(v)
        want = np.sqrt((blocks - 1) / blocks * ((v - v.mean(axis=0)) ** 2).sum(axis=0)).astype(np.float64)
        assert np.allclose(res[key][1:], want, rtol=1e-12, atol=0), (key, res[key][1:] / want - 1)
