"""The chain kernels with the Lennard-Jones rounds in assembly (needs an MI355X).

ppp_eval_forces runs the compiled rounds with energies for every shape, so what the
fp32 runs of the shapes 8x4 to 64x4 compute is held here: one step of theirs, whose
length makes the displacement the force, against the oracle."""
import numpy as np
import pytest

import paper_1105_4840_amd as ppp
import ppp_inputs
import oracle

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")

f32 = np.float32


def _run(prob, G):
    """(state, accumulators) of every replica after the run, from a checkpoint."""
    h = ppp.ppp_create(prob)
    try:
        ws = ppp.workspace(h)
        ppp.ppp_begin(h, ws)
        ppp.ppp_advance(h, 10 ** 9)
        blob = ppp.ppp_checkpoint(h)
    finally:
        ppp.ppp_destroy(h)
    n = len(prob["lambda"]) * prob["n_replicas"]
    state = np.frombuffer(blob, dtype=f32, count=24 * G * n, offset=16).reshape(n, 6, 4 * G)
    at = 16 + -(-state.nbytes // 256) * 256
    return state, np.frombuffer(blob, dtype=np.float64, count=16 * n, offset=at).reshape(n, 16)


@pytest.mark.parametrize("G", [8, 16, 32, 64])
@pytest.mark.parametrize("short", [0, 1, 3])
def test_one_step_is_the_oracles_force(G, short, tmp_path, monkeypatch):
    """Without friction and almost without heat the first BAOAB step moves a bead by
    dt^2 F(x_0) / 2m (and dt v_0, small): at dt = 1 the fp32 positions then hold the forces to some 1e-7
    of the largest, and the compiled kernels' bound of 1e-5 applies to them."""
    n = 4 * G - short
    table = tmp_path / "tune.txt"
    table.write_text(f"{n} 0 {G} 4\n")
    monkeypatch.setenv("PPP_TUNE_TABLE", str(table))
    for seed in range(3):
        print(f"case one step {G}x4 N={n} seed={seed}", flush=True)
        x0 = ppp_inputs.random_chain_coords(n, 1, seed=100 * G + seed)[0].astype(f32).astype(np.float64)
        end = float(np.linalg.norm(x0[-1] - x0[0]))
        R = 4 * (64 // G) + 1                               # one workgroup and a replica more in either window
        p = ppp_inputs.config_chain_small(n, n_replicas=R, n_steps=1, n_windows=2, precision="fp32")
        p.update({"init_coords": x0, "lambda": [end - 0.1, end + 0.1], "n_equil": 0, "sample_every": 1, "gamma": 0.0,
                  "kT": 1e-8, "dt": 1.0, "xi_bound": 1e12, "w_half_bins": 0, "n_blocks": 2})
        state, acc = _run(p, G)
        assert np.array_equal(acc[:, 0], np.ones(2 * R))
        for w in range(2):
            for r in range(R):
                path = oracle.trajectory(p, w, r, 1)        # with the replica's own small velocities
                want = (path[1] - path[0]).reshape(n, 3)
                moved = state[w * R + r, :3, :n].T.astype(np.float64) - x0
                assert np.linalg.norm(moved - want) <= 1e-5 * np.linalg.norm(want), (w, r)
