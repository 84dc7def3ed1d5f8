"""The 1-D kernel's lane split (needs an MI355X): 16, 8, 4, 2 or 1 lanes per replica
by the number of replicas, normals drawn in tiles of 64 down to 4 steps.

A replica's trajectory and record depend on its number alone, so the first
replicas of window 1 must come out the same bit for bit whatever the number of
replicas (hence of lanes) and however the run is cut into launches; the
smallest problem is held against the oracle."""
import numpy as np
import pytest

import paper_1105_4840_amd as ppp
import ppp_inputs
import oracle

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")

# replicas per window (two windows): one size for each lane count, each ragged
SIZES = [37, 3001, 5003, 33333, 66666]


def _problem(replicas, precision, every, **kw):
    p = ppp_inputs.config_1d(n_replicas=replicas, n_steps=391, n_windows=2, seed=9, precision=precision)
    p.update({"lambda": [-1.0, -0.9], "n_equil": 5, "sample_every": every, "w_half_bins": 0, "n_blocks": 4,
              "integrator_1d": every % 2, "xi_min": -1.2, "xi_bin": 0.4 / 64, "xi_nbins": 64}, **kw)
    return p


def _records(prob, cuts=()):
    """(state, accumulators) of every replica after the run, from a checkpoint, and the results."""
    h = ppp.ppp_create(prob)
    try:
        ws = ppp.workspace(h)
        ppp.ppp_begin(h, ws)
        for n in cuts:
            ppp.ppp_advance(h, n)
        ppp.ppp_advance(h, 10 ** 9)
        blob = ppp.ppp_checkpoint(h)
        ppp.ppp_finalize(h)
        res = ppp.ppp_get_result(h, prob)
    finally:
        ppp.ppp_destroy(h)
    n = len(prob["lambda"]) * prob["n_replicas"]
    dt = np.float64 if prob["precision"] == "fp64" else np.float32
    state = np.frombuffer(blob, dtype=dt, count=2 * n, offset=16).reshape(n, 2)
    at = 16 + -(-state.nbytes // 256) * 256
    return state, np.frombuffer(blob, dtype=np.float64, count=16 * n, offset=at).reshape(n, 16), res


@pytest.mark.parametrize("precision", ["fp64", "fp32"])
@pytest.mark.parametrize("every", [1, 3, 4, 10, 200])
def test_records_do_not_depend_on_the_lane_split_or_the_launches(precision, every):
    print(f"case 1-D lanes {precision} every {every}", flush=True)
    # a bound near the well's edge freezes some of the replicas part way
    small = _problem(SIZES[0], precision, every, xi_bound=1.25)
    st, acc, _ = _records(small)
    frozen = int(acc[:SIZES[0], 15].sum())
    print(f"  frozen {frozen} of {SIZES[0]}", flush=True)
    for n in SIZES:
        p = _problem(n, precision, every, xi_bound=1.25)
        for cuts in ((), (1, 2, 3, 13, 64, 17, 100)):
            s2, a2, _ = _records(p, cuts)
            assert np.array_equal(s2[:SIZES[0]], st[:SIZES[0]]), (n, cuts)
            assert np.array_equal(a2[:SIZES[0]], acc[:SIZES[0]]), (n, cuts)


@pytest.mark.parametrize("every", [1, 3, 4, 10, 200])
def test_records_match_the_oracle(every):
    print(f"case 1-D lanes against the oracle, every {every}", flush=True)
    p = _problem(SIZES[0], "fp64", every)
    _, acc, res = _records(p, (7, 60))
    xi, kept, _ = oracle.run(p)
    xi = np.asarray(xi).reshape(2 * SIZES[0], -1)
    lam = np.repeat(p["lambda"], SIZES[0])[:, None]
    d = xi - lam
    # accumulated rounding of a few hundred fp64 terms of order one
    assert np.array_equal(acc[:, 0], np.full(2 * SIZES[0], xi.shape[1]))
    assert np.allclose(acc[:, 1], d.sum(axis=1), rtol=0, atol=1e-11)
    assert np.allclose(acc[:, 2], (d * d).sum(axis=1), rtol=0, atol=1e-11)
    assert np.allclose(acc[:, 3], xi.min(axis=1), rtol=0, atol=1e-12)
    assert np.allclose(acc[:, 4], xi.max(axis=1), rtol=0, atol=1e-12)
    dl = p["lambda"][1] - p["lambda"][0]
    bk = p["k"] / p["kT"]
    for rows, a, at in ((slice(0, SIZES[0]), bk * dl * (d - 0.5 * dl), 5),
                        (slice(SIZES[0], None), -bk * dl * (d + 0.5 * dl), 9)):
        for q in (1.0, 2.0):
            ref = np.log(np.sum(np.exp(q * a[rows]), axis=1))
            got = acc[rows, at] + np.log(acc[rows, at + 1])
            assert np.allclose(got, ref, rtol=0, atol=1e-11), (at, q)
            at += 2
    under = (xi < p["xi_min"]).sum(axis=1)
    assert np.array_equal(acc[:, 13], under)
    assert int(res["xi_hist"].sum()) + int(res["xi_under_over"].sum()) == xi.size
