"""The chain kernels with the Lennard-Jones rounds in assembly, and their compiled
twins of the 64x4 shape (needs an MI355X).

ppp_eval_forces runs the compiled rounds with energies for every shape, so what the
fp32 runs of the shapes 8x4 to 64x4 compute is held here: one step of theirs, whose
length makes the displacement the force, against the oracle.  The 64x4 shape has a
direct and a persistent kernel of either kind, chosen by the work at hand: each has
to leave the same states, records and results."""
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


@pytest.mark.parametrize("n", [129, 200, 256])
def test_direct_kernels_of_the_64x4_shape_agree(n):
    """One and six workgroups a CU take the assembly; two, or a histogram of more than
    48 KB, the compiled kernel.  A replica's trajectory depends on its number alone."""
    cus = torch.cuda.get_device_properties(0).multi_processor_count
    x0 = ppp_inputs.random_chain_coords(n, 1, seed=n)[0]
    end = float(np.linalg.norm(x0[-1] - x0[0]))
    few = 5
    got = {}
    # replicas of two windows, four to a workgroup
    for name, replicas, bins in (("assembly, 1 a CU", few, 512), ("compiled, 2 a CU", 4 * cus - 3, 512),
                                 ("assembly, 6 a CU", 11 * cus + 3, 512), ("compiled, large histogram", 11 * cus + 3, 13000),
                                 ("compiled, 2 a CU, large histogram", 4 * cus - 3, 13000)):
        print(f"case 64x4 direct N={n} {name}", flush=True)
        p = ppp_inputs.config_chain_small(n, n_replicas=replicas, n_steps=23, n_windows=2, precision="fp32")
        p.update({"init_coords": x0, "lambda": [end - 0.1, end + 0.1], "sample_every": 3, "n_equil": 2, "w_half_bins": 0,
                  "xi_min": 0.0, "xi_bin": (end + 3.0) / bins, "xi_nbins": bins})
        s, a = _run(p, 64)
        assert np.isfinite(s).all() and np.array_equal(a[:, 0], np.full(len(a), 7.0))
        got[name] = s[:few].copy(), a[:few].copy()
    s0, a0 = got["assembly, 1 a CU"]
    for name, (s, a) in got.items():
        assert np.array_equal(s, s0) and np.array_equal(a, a0), name


@pytest.mark.parametrize("wide", [False, True])
def test_batches_of_long_chains_equal_single_runs(wide):
    """The persistent kernels of the 64x4 shape: compiled where the longest items set the
    time, in assembly from 4.5 times the longest item's work per CU on."""
    cus = torch.cuda.get_device_properties(0).multi_processor_count
    probs = []
    for i, n in enumerate((150, 256, 40, 100)):
        p = ppp_inputs.config_chain_small(n, n_replicas=9, n_steps=24, n_windows=3, seed=50 + i, precision="fp32")
        p.update({"sample_every": 2, "n_equil": 3, "n_blocks": 3, "w_half_bins": 400, "w_bin": 0.1})
        probs.append(p)
    if wide:
        p = dict(probs[1], n_replicas=6 * cus, seed=60)     # three windows of 1.5 workgroups a CU each
        probs.append(p)
    npair = [0.5 * p["n_beads"] ** 2 + 20.0 * p["n_beads"] for p in probs]
    work = sum(c * p["n_replicas"] * 3 for c, p in zip(npair, probs))
    longest = max(c * min(p["n_replicas"], 4 if p["n_beads"] > 128 else 8 if p["n_beads"] > 64 else 16) for c, p in zip(npair, probs))
    print(f"case batch of long chains wide={wide}: work / longest per CU {work / longest / cus:.2f}", flush=True)
    assert (work >= 4.5 * cus * longest) == wide
    h = ppp.ppp_batch_create(probs)
    try:
        ws = ppp.workspace(h)
        for _ in range(2):                                  # the graph twice
            ppp.ppp_run(h, ws)
            got = [ppp.ppp_batch_get_result(h, p, i) for i, p in enumerate(probs)]
            for p, g in zip(probs, got):
                ref, _ = ppp.run(p)
                for key, v in ref.items():
                    if isinstance(v, np.ndarray):
                        assert np.array_equal(v, g[key], equal_nan=v.dtype.kind == "f"), (p["n_beads"], key)
    finally:
        ppp.ppp_destroy(h)
