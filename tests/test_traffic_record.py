"""The sources that bench.py's traffic record is tied to: everything the chain kernels
are compiled from, the generator of their assembly included (no GPU needed)."""
import os
import re

import bench

PKG = os.path.join(bench.ROOT, "paper_1105_4840_amd")


def test_every_source_of_the_chain_kernels_is_in_the_digest():
    listed = {os.path.basename(n) for n in bench.KERNEL_SOURCES}
    todo, seen = ["ppp_sim.hip"], set()
    while todo:
        name = todo.pop()
        if name in seen:
            continue
        seen.add(name)
        path = os.path.join(PKG, "csrc", name)
        if not os.path.exists(path):
            name = {"ppp_lj_rounds.hpp": "lj_rounds.py"}.get(name, name)      # written at build time
            if name == "ppp.h":                                               # the C interface
                continue
            assert os.path.exists(os.path.join(PKG, name)), name
            assert name in listed, name
            continue
        assert name in listed, name
        todo += re.findall(r'#include "([^"]+)"', open(path).read())
    assert "lj_rounds.py" in listed


def test_the_digest_follows_the_generator(tmp_path, monkeypatch):
    before = bench.kernel_sources_digest()
    for n in bench.KERNEL_SOURCES:
        dst = tmp_path / "paper_1105_4840_amd" / n
        dst.parent.mkdir(parents=True, exist_ok=True)
        dst.write_bytes(open(os.path.join(PKG, n), "rb").read())
    monkeypatch.setattr(bench, "ROOT", str(tmp_path))
    assert bench.kernel_sources_digest() == before
    rounds = tmp_path / "paper_1105_4840_amd" / "lj_rounds.py"
    rounds.write_text(re.sub(r"^GAP = \d+", "GAP = 99", rounds.read_text(), flags=re.M))
    assert bench.kernel_sources_digest() != before
