"""Writes the Newton-3 rotation rounds of the fp32 chain kernels in gfx950 assembly.

One round pulls the j-beads and (minus) their reactions one lane on and evaluates
the 4 x 4 pairs of a lane; csrc/ppp_chain_force.hpp holds the same arithmetic in
the same order in C++ for every other case (`lj_block`) and uses this one where it
is built for the device in fp32, without energies, for groups of 8 lanes and more.

Bound: VALU issue, 20 instructions a pair, no memory.  Measured on MI355X with two
wavefronts a SIMD, in cycles per wavefront-instruction: v_sub, v_mul and v_fmac
with vector operands 2.4; v_fma with three different registers 2.9, and 4.7 when
all three lie in registers of one parity (the register file has an even and an odd
bank); v_cmp and v_cndmask 3.2 each; v_rcp 8.2.  So:
  - differences, reciprocals and constants lie in even registers, squares and force
    factors in odd ones, so that no triple shares a parity (a quarter of the
    compiler's did);
  - the reactions are kept with their sign turned, so both beads take the 4-byte
    v_fmac instead of a v_fma with a negated operand (rounding is symmetric);
  - the pairs are software-pipelined: a new one starts every 20 instructions, each
    instruction of a pair at its own place modulo 20 (`_places`), so the slow
    instructions are spread evenly and every result is at least GAP instructions
    old when it is used.  Four pairs are in flight;
  - a j-bead is pulled on as soon as the round's last pair has taken its
    difference, a reaction as soon as the last pair has added to it, one bead's
    pairs before their next use.
A pair's last instructions fall into the next round: the first round stands before the
loop without them, and the last pairs are finished after it.

The loop alone, measured at GAP = 4, cycles a pair at 2 / 3 / 4 wavefronts a SIMD: the
compiler's code for lj_block 77 / 69 / 65, these rounds 66 / 59 / 56.  Kernel times at
GAP = 3 / 4 / 5 / 6, ms: 256 beads (21 windows of 4096, 30 steps) 37.5 / 36.9 / 36.6 /
36.6, 128 beads (21 x 2048, 100 steps) 16.3 / 16.1 / 15.9 / 16.0, 64 beads (21 x 4096,
150 steps) 13.4 / 13.2 / 13.1 / 13.1.  More pairs in flight cost registers.  The
compiler schedules its loop with more registers inside the kernels, so there the gain
comes with the third wavefront that the kernels using these rounds are built to fit:
256 beads, 41 windows of 4096 replicas, 30 steps: 76.7 -> 71.2 ms (79.4 at two
wavefronts); 128 beads, 21 windows of 2048, 100 steps: 18.3 -> 16.1; 64 beads, 21
windows of 4096, 150 steps: 14.4 -> 13.3.  With two beads a lane the exchanges take a
quarter of the instructions and the LDS, not the VALU, sets the pace (70 cycles a pair
either way; 32 beads 15.9 ms compiled, 16.7 with such rounds): those shapes have the
C++ loop alone.

Waits: LDS results return in order, so the count before a use is the number of LDS
instructions issued since (`lgkmcnt` counts to 15).  v_cmp to v_cndmask keeps the
two wait states a mask in VCC needs, v_rcp to its use the one of a transcendental.
"""
B = 4            # beads per lane
GAP = 6          # instructions between a result and its use
II = 20          # instructions per pair
IN_FLIGHT = 4    # pairs in flight (temporary registers for each)


def _places():
    """Issue place of each instruction of a pair, relative to its first."""
    deps = [("s1", []), ("s0", []), ("s2", []), ("m", [("s1", GAP)]), ("a0", [("m", GAP), ("s0", GAP)]),
            ("a2", [("a0", GAP), ("s2", GAP)]), ("rcp", [("a2", GAP)]), ("q1", [("rcp", GAP + 1)]), ("q2", [("q1", GAP)]),
            ("w", [("q2", GAP)]), ("u", [("q2", GAP), ("w", 0)]), ("f", [("w", GAP), ("u", GAP)]), ("cmp", [("f", -2)]),
            ("cnd", [("f", GAP), ("cmp", 3)])] + [(x, [("cnd", GAP)]) for x in ("f0", "f1", "f2", "g0", "g1", "g2")]
    place, used = {}, set()
    for name, ds in deps:
        t = max([0] + [place[d] + g for d, g in ds])
        while t % II in used:
            t += 1
        place[name] = t
        used.add(t % II)
    assert len(used) == II
    assert place["cnd"] - place["cmp"] < II          # one mask register
    assert max(place.values()) < IN_FLIGHT * II
    assert min(place[x] for x in ("s0", "s2")) > place["s1"] and min(place[x] for x in ("g1", "g2")) > place["g0"]
    return place


def rounds():
    """(assembly lines, clobbered vector registers, register numbers) of the loop."""
    place = _places()
    base = 40
    row = lambda k: [[base + 3 * B * k + B * c + b for b in range(B)] for c in range(3)]
    P, Q, F, G = row(0), row(1), row(2), row(3)
    addr = base + 12 * B
    lA, lB, t0 = addr + 2, addr + 4, addr + 6
    even = [t0 + 2 * k for k in range(4 * IN_FLIGHT)]
    odd = [t0 + 1 + 2 * k for k in range(2 * IN_FLIGHT)]
    D = [even[c * IN_FLIGHT:(c + 1) * IN_FLIGHT] for c in range(3)]
    I = even[3 * IN_FLIGHT:]
    R, S = odd[:IN_FLIGHT], odd[IN_FLIGHT:]
    n_pairs = B * B
    length = n_pairs * II

    def text(i, op):
        b1, b2 = divmod(i, B)
        k = i % IN_FLIGHT
        d, r, s, v = [D[c][k] for c in range(3)], R[k], S[k], I[k]
        c = int(op[1]) if op[1:].isdigit() else 0
        return {"s": f"v_sub_f32 v{d[c]}, v{P[c][b1]}, v{Q[c][b2]}",
                "m": f"v_mul_f32 v{r}, v{d[1]}, v{d[1]}",
                "a": f"v_fmac_f32 v{r}, v{d[c]}, v{d[c]}",
                "rcp": f"v_rcp_f32 v{v}, v{r}",
                "q1": f"v_mul_f32 v{s}, v{v}, v{v}",
                "q2": f"v_mul_f32 v{s}, v{s}, v{v}",
                "w": f"v_mul_f32 v{v}, v{s}, v{v}",
                "u": f"v_fma_f32 v{s}, v{lA}, v{s}, v{lB}",
                "f": f"v_mul_f32 v{s}, v{v}, v{s}",
                "cmp": f"v_cmp_gt_f32 vcc, %[rc2], v{r}",
                "cnd": f"v_cndmask_b32 v{s}, 0, v{s}, vcc",
                "F": f"v_fmac_f32 v{F[c][b1]}, v{s}, v{d[c]}",
                "G": f"v_fmac_f32 v{G[c][b2]}, v{s}, v{d[c]}"}[
                    op if op in ("m", "rcp", "q1", "q2", "w", "u", "f", "cmp", "cnd")
                    else {"s": "s", "a": "a", "f": "F", "g": "G"}[op[0]]]

    # (place in the round, next round?, text, LDS results needed, LDS result made)
    ops = []
    for i in range(n_pairs):
        for op, t in place.items():
            need = {"s1": ("q", i % B), "g0": ("g", i % B)}.get(op) if i < B else None
            ops.append((i * II + t, text(i, op), need, None))
    perm = lambda x: f"ds_bpermute_b32 v{x}, v{addr}, v{x}"
    for b in range(B):
        last = ((B - 1) * B + b) * II
        for c in range(3):
            ops.append((last + max(place[x] for x in ("s0", "s1", "s2")) + 0.1 + 0.01 * c, perm(Q[c][b]), None, ("q", b)))
            # at the start of the next round at the earliest: every round pulls once, the first one included
            ops.append((max(length, last + max(place[x] for x in ("g0", "g1", "g2"))) + 0.1 + 0.01 * c, perm(G[c][b]), None,
                        ("g", b)))
    body = sorted((t % length, t >= length, x, need, made) for t, x, need, made in ops)
    first = [o for o in body if not o[1] or o[4]]        # nothing of a round before it; the pulls
    start = [(0, False, perm(Q[c][b]), None, ("q", b)) for b in range(B) for c in range(3)]
    made, waits = [], {}
    for turn, ops in enumerate((start, first, body, body)):
        for k, (_, _, _, need, m) in enumerate(ops):
            if need is not None:
                newest = max(j for j, key in enumerate(made) if key == need)
                at = (min(turn, 2), k)
                waits[at] = min(15, waits.get(at, 15), len(made) - 1 - newest)
            if m is not None:
                made.append(m)

    def lines(turn, ops):
        for k, (_, _, x, _, _) in enumerate(ops):
            if (turn, k) in waits:
                yield f"s_waitcnt lgkmcnt({waits[turn, k]})"
            yield x

    out = [x for _, _, x, _, _ in start] + list(lines(1, first)) + ["1:"] + list(lines(2, body))
    out += ["s_sub_u32 %[n], %[n], 1", "s_cmp_lg_u32 %[n], 0", "s_cbranch_scc1 1b"]
    out += [x for _, later, x, _, m in body if later and m is None]      # the last pairs' tails
    out += ["s_waitcnt lgkmcnt(0)", "s_nop 1"]
    return out, sorted(sum(D, []) + I + R + S), (P, Q, F, G, addr, lA, lB)


def header():
    s = ["// Written by lj_rounds.py, which says what bounds these loops and why they are laid out so.",
         "#pragma once", "namespace ppp {"]
    lines, clobbered, (P, Q, F, G, addr, lA, lB) = rounds()
    vec = f"lj_vec{B}"
    reg = lambda row: f"{{v[{row[0]}:{row[-1]}]}}"
    s.append(f"typedef float {vec} __attribute__((ext_vector_type({B})));")
    arg = lambda n, const: f"{'const ' if const else ''}float (&{n})[{B}]"
    names = [(x + a, x == "p") for x in "pqfg" for a in "xyz"]
    s.append("__device__ __forceinline__ void lj_rounds(int rounds_after_first, int src_lane, float lA, float lB, float rc2, "
             + ", ".join(arg(n, c) for n, c in names) + ") {")
    for n, c in names:
        s.append(f"    {'const ' if c else ''}{vec} v{n} = {{" + ", ".join(f"{n}[{b}]" for b in range(B)) + "};")
    s.append("    asm volatile(")
    s += [f'        "{x}\\n\\t"' for x in lines]
    outs = [f'"+{reg(r[a])}"(v{x}{"xyz"[a]})' for x, r in (("f", F), ("g", G), ("q", Q)) for a in range(3)]
    s.append("        : " + ", ".join(outs) + ', [n] "+s"(rounds_after_first)')
    ins = [f'"{reg(P[a])}"(vp{"xyz"[a]})' for a in range(3)]
    s.append("        : " + ", ".join(ins) + f', "{{v{addr}}}"(src_lane << 2), "{{v{lA}}}"(lA), "{{v{lB}}}"(-lB), [rc2] "s"(rc2)')
    s.append('        : "vcc", "scc", ' + ", ".join(f'"v{x}"' for x in clobbered) + ");")
    for n in [x + a for x in "fg" for a in "xyz"]:
        s.append("    " + " ".join(f"{n}[{b}] = v{n}[{b}];" for b in range(B)))
    s.append("}")
    s.append("}  // namespace ppp")
    return "\n".join(s) + "\n"


if __name__ == "__main__":
    print(header())
