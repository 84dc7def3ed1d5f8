"""The assembly rounds of the fp32 chain kernels with four beads a lane.

On the CPU the generated lines are run on 64 simulated lanes against the plain
loop they stand for, bit for bit; a result used before its wait, or too close
behind a compare or a reciprocal, fails the test.  On the GPU the kernels that
use them are held against the kernels that do not, on crowded conformations."""
import os
import re
import runpy

import numpy as np
import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
f32 = np.float32


def _fma(a, b, c):
    # one rounding to double, one to float, on both sides of the comparison
    return (a.astype(np.float64) * b.astype(np.float64) + c.astype(np.float64)).astype(f32)


class Lanes:
    """64 lanes' vector registers, the mask and the in-order LDS queue."""

    def __init__(self, rc2, n):
        self.v = {}
        self.pending, self.rc2, self.n = [], rc2, n
        self.vcc, self.vcc_age, self.rcp = None, 99, (None, 99)

    def read(self, name):
        x = int(name[1:])
        assert x not in [d for d, _ in self.pending], f"v{x} read before its LDS result is waited for"
        assert x != self.rcp[0] or self.rcp[1] >= 1, f"v{x} read right behind v_rcp"
        return self.v[x]

    def write(self, name, value):
        x = int(name[1:])
        assert x not in [d for d, _ in self.pending], f"v{x} written with an LDS result in flight"
        self.v[x] = value.astype(f32) if value.dtype != np.int64 else value

    def run(self, lines):
        pc = 0
        while pc < len(lines):
            op, *a = re.split(r"[ ,]+", lines[pc])
            pc += 1
            if op == "1:":
                top = pc
                continue
            self.vcc_age += 1
            self.rcp = (self.rcp[0], self.rcp[1] + 1)
            if op == "s_waitcnt":
                keep = int(re.search(r"\d+", a[0]).group())
                while len(self.pending) > keep:
                    x, val = self.pending.pop(0)
                    self.v[x] = val
            elif op == "ds_bpermute_b32":
                val = self.read(a[2])[self.read(a[1]) >> 2]
                assert int(a[0][1:]) not in [d for d, _ in self.pending]
                self.pending.append((int(a[0][1:]), val))
            elif op == "v_sub_f32":
                self.write(a[0], self.read(a[1]) - self.read(a[2]))
            elif op == "v_mul_f32":
                self.write(a[0], self.read(a[1]) * self.read(a[2]))
            elif op == "v_fmac_f32":
                self.write(a[0], _fma(self.read(a[1]), self.read(a[2]), self.read(a[0])))
            elif op == "v_fma_f32":
                self.write(a[0], _fma(self.read(a[1]), self.read(a[2]), self.read(a[3])))
            elif op == "v_rcp_f32":
                self.write(a[0], f32(1) / self.read(a[1]))
                self.rcp = (int(a[0][1:]), -1)
            elif op == "v_cmp_gt_f32":
                self.vcc, self.vcc_age = self.rc2 > self.read(a[2]), -1
            elif op == "v_cndmask_b32":
                assert self.vcc_age >= 2, "mask used too early"
                self.write(a[0], np.where(self.vcc, self.read(a[2]), f32(0)))
            elif op == "s_sub_u32":
                self.n -= 1
            elif op == "s_cbranch_scc1":
                pc = top if self.n != 0 else pc
            else:
                assert op in ("s_cmp_lg_u32", "s_nop"), op
        assert not self.pending


@pytest.mark.parametrize("G", [8, 16, 32, 64])
def test_generated_rounds_equal_the_plain_loop(G):
    gen = runpy.run_path(os.path.join(ROOT, "paper_1105_4840_amd", "lj_rounds.py"))
    lines, clobbered, (P, Q, F, Gr, addr, lA, lB) = gen["rounds"]()
    rng = np.random.default_rng(G)
    n = (G - 1) // 2 - 1
    lane = np.arange(64)
    src = (lane // G) * G + (lane % G + G - 1) % G
    A, Bc, rc2 = f32(48.0), f32(24.0), f32(6.25)
    p, q, f, g = (rng.uniform(-s, s, (3, 4, 64)).astype(f32) for s in (2.5, 2.5, 9.0, 9.0))
    m = Lanes(rc2, n - 1)
    for rows, x in ((P, p), (Q, q), (F, f), (Gr, g)):
        for c in range(3):
            for b in range(4):
                m.v[rows[c][b]] = x[c, b].copy()
    m.v[addr], m.v[lA], m.v[lB] = src.astype(np.int64) << 2, np.full(64, A), np.full(64, -Bc)
    used = {r for rows in (P, Q, F, Gr) for row in rows for r in row} | {addr, lA, lB}
    assert not used & set(clobbered)
    assert {int(x) for line in lines for x in re.findall(r"\bv(\d+)\b", line)} <= used | set(clobbered)
    m.run(lines)
    for _ in range(n):
        q, g = q[:, :, src], g[:, :, src]
        for b1 in range(4):
            for b2 in range(4):
                d = p[:, b1] - q[:, b2]
                r2 = _fma(d[2], d[2], _fma(d[0], d[0], d[1] * d[1]))
                i = f32(1) / r2
                i6 = i * i * i
                fac = np.where(r2 < rc2, i6 * i * _fma(np.full(64, A), i6, np.full(64, -Bc)), f32(0))
                for c in range(3):
                    f[c, b1] = _fma(fac, d[c], f[c, b1])
                    g[c, b2] = _fma(fac, d[c], g[c, b2])
    for c in range(3):
        for b in range(4):
            assert np.array_equal(m.v[F[c][b]], f[c, b]) and np.array_equal(m.v[Gr[c][b]], g[c, b]), (c, b)


def _records(ppp, prob, G):
    """(state, accumulators) of window 1's replicas after the run, from a checkpoint."""
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


@pytest.mark.gpu
@pytest.mark.parametrize("G", [8, 16, 32, 64])
@pytest.mark.parametrize("short", [0, 2, 5])
def test_kernels_with_and_without_rounds_agree(G, short, tmp_path, monkeypatch):
    """From a crowded conformation, ragged workgroups: a run small enough for the
    compiled rounds against one large enough for the generated ones.  A replica's
    trajectory depends on its number alone, so the first replicas of window 1 have
    to end in the same state with the same record, bit for bit."""
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_1105_4840_amd as ppp
    import ppp_inputs
    n = 4 * G - short
    print(f"case lj rounds {G}x4 N={n}", flush=True)
    table = tmp_path / "tune.txt"
    table.write_text(f"{n} 1 {G} 4\n{n} 0 {G} 4\n")
    monkeypatch.setenv("PPP_TUNE_TABLE", str(table))
    x0 = ppp_inputs.random_chain_coords(n, 1, seed=G + short)[0]
    end = float(np.linalg.norm(x0[-1] - x0[0]))
    cus = torch.cuda.get_device_properties(0).multi_processor_count
    per_wg = 4 * (64 // G)
    few, many = per_wg + 1, (5 * cus * per_wg) // 2 + 3      # workgroups: 3 a window, then 5 per CU
    got = []
    for replicas in (few, many):
        prob = ppp_inputs.config_chain_small(n, n_replicas=replicas, n_steps=23, n_windows=2, precision="fp32")
        prob.update({"init_coords": x0, "lambda": np.array([end - 0.1, end + 0.1]), "sample_every": 3, "n_equil": 2})
        got.append(_records(ppp, prob, G))
    (s1, a1), (s2, a2) = got
    assert np.isfinite(s1[:few]).all() and np.array_equal(s1[:few], s2[:few])
    assert np.array_equal(a1[:few, 0], np.full(few, 7.0))
    assert np.array_equal(a1[:few], a2[:few])
