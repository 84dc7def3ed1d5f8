"""Which steps the 1-D kernel samples when step numbers come near 2^32 (needs an
MI355X).  n_steps may be anything below 2^32 and sample_every any positive int32,
so the next sampled step can lie beyond 2^32.

A checkpoint's step count is moved to just before the step in question, so a case
takes some hundred steps.  The samples of a launch have to be the steps n with
n > n_equil and n - n_equil a multiple of sample_every, counted in Python."""
import struct

import numpy as np
import pytest

import paper_1105_4840_amd as ppp
import ppp_inputs

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")

TOP = 2 ** 32
CASES = [
    # n_steps, n_equil, sample_every, first launch's start, launch lengths
    (3_100_000_000, 3_000_000_000, 2_000_000_000, 3_000_000_000 + 2_000_000_000 - TOP - 40, (100,)),
    (2_200_000_000, 2_199_999_999, 2 ** 31 - 1, 2_199_999_999 + 2 ** 31 - 1 - TOP - 70, (130, 65)),
    (TOP - 1, TOP - 2, 2 ** 31 - 1, TOP - 2 + 2 ** 31 - 1 - TOP - 8, (64, 64)),
    (TOP - 1, 10 ** 9, 2 ** 31 - 1, 10 ** 9 + 2 ** 31 - 1 - 30, (20, 70)),   # one sample, the next beyond 2^32
    (TOP - 1, TOP - 150, 10, TOP - 1 - 300, (77, 1000)),                     # up to the very last step
    (TOP - 1, TOP - 150, 3, TOP - 1 - 300, (1000,)),
]


@pytest.mark.parametrize("precision", ["fp64", "fp32"])
@pytest.mark.parametrize("replicas", [37, 66666])     # 16 lanes a replica and one
@pytest.mark.parametrize("case", CASES, ids=lambda c: f"{c[0]}-{c[1]}-{c[2]}")
def test_sampled_steps_near_two_to_the_32(case, replicas, precision):
    n_steps, n_equil, every, start, launches = case
    print(f"case sampled steps {case} replicas={replicas} {precision}", flush=True)
    p = ppp_inputs.config_1d(n_replicas=replicas, n_steps=n_steps, n_windows=2, precision=precision)
    p.update({"lambda": [-1.0, -0.9], "n_equil": n_equil, "sample_every": every, "w_half_bins": 0, "n_blocks": 4,
              "xi_min": -2.5, "xi_bin": 5.0 / 64, "xi_nbins": 64})
    h = ppp.ppp_create(p)
    try:
        ws = ppp.workspace(h)
        ppp.ppp_begin(h, ws)
        ppp.ppp_advance(h, 1)
        blob = ppp.ppp_checkpoint(h)
        ppp.ppp_restore(h, ws, blob[:8] + struct.pack("<q", start) + blob[16:])
        for n in launches:
            ppp.ppp_advance(h, n)
        done = ppp.ppp_steps_done(h)
        blob = ppp.ppp_checkpoint(h)
    finally:
        ppp.ppp_destroy(h)
    assert done == min(n_steps, start + sum(launches))
    want = sum(1 for n in range(start + 1, done + 1) if n > n_equil and (n - n_equil) % every == 0)
    n = 2 * replicas
    at = 16 + -(-(2 * n * (8 if precision == "fp64" else 4)) // 256) * 256
    acc = np.frombuffer(blob, dtype=np.float64, count=16 * n, offset=at).reshape(n, 16)
    assert np.array_equal(acc[:, 15], np.zeros(n))
    assert np.array_equal(acc[:, 0], np.full(n, float(want)))
