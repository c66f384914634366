"""The colour sum in blocks under relabellings, as emitted, against J^dag N J."""
import re

import numpy as np
import pytest

from paper_2503_21935_amd.gen import wave5
from paper_2503_21935_amd.gen.colour import colour_matrix_exact
from paper_2503_21935_amd.gen.emit import GGEmitter


@pytest.mark.parametrize("n", [2, 3, 4])
def test_emitted_blocks_equal_the_quadratic_form(n):
    em = GGEmitter("x", n)
    J = np.random.default_rng(n).integers(-9, 10, size=(len(em.perms), 2)).astype(float)
    scope = {"fma": lambda a, b, c: a * b + c, "J": J}
    for line in em.emit_colour_blocks():
        line = line.split("//")[0].strip()
        if line in ("{", "}", ""):
            continue
        line = re.sub(r"J\[(\d+)\]\.([ri])", lambda m: f"J[{m[1]},{'ri'.index(m[2])}]", line.replace("const T ", ""))
        line = line.replace("return ", "result = ").replace("T acc", "acc").replace("T(", "(").rstrip(";")
        exec(line, scope)
    want = sum(J[:, c] @ np.array(em.num, dtype=float) @ J[:, c] for c in (0, 1))
    assert scope["result"] == want  # small integers: exact


def test_five_gluon_plan_equals_the_quadratic_form():
    """Signed sums over orbits, the emitted fast transform, and the blocks."""
    J = np.random.default_rng(5).integers(-9, 10, size=120).astype(float)
    want = J @ np.array(colour_matrix_exact(5)[0], dtype=float) @ J
    orbits, blocks = wave5.colour_plan()
    assert sorted(f for fl, _ in orbits for f in fl) == list(range(120))
    h = J.copy()
    for flows, rows in orbits:
        scope = {"h": J.copy()}
        for line in wave5.emit_butterfly(flows, rows, lambda f: f"h[{f}]"):
            for part in line.replace("const double ", "").rstrip(";").split(", "):
                exec(part, scope)
        h[flows] = scope["h"][flows]
        assert np.array_equal(h[flows], np.array(rows) @ J[flows])
    assert sum(h[pl] @ np.array(c) @ h[pl] for pl, c in blocks) == want
    shares = wave5.colour_waves(orbits, blocks)
    assert sorted(map(repr, (x for w in shares[0] for x in w))) == sorted(map(repr, orbits))
    assert sorted(map(repr, (x for w in shares[1] for x in w))) == sorted(map(repr, blocks))


def test_five_gluon_tables_write_every_entry_once():
    dests = {"W2": 2, "W4": 2, "W4S": 2}
    written = {}
    for name, rows in wave5.nodes().items():
        k = dests.get(name, 1)
        d = [v for r in rows for v in r[-k:]]
        assert len(set(d)) == len(d)
        assert all(0 <= v < wave5.L.END for r in rows for v in r)
        written[name] = set(d)
    assert not written["W4"] & written["W4S"] and not written["W5"] & (written["W5A"] | written["W5B"])
    flows = [f for p in wave5.PAIRS for f in wave5.slot_flows(p)]
    assert len(set(flows)) == 120
    # what a configuration's sums read has been written
    tree, ends, mid, rows, two = wave5.slot_entries((1, 3), {0: 1, 1: 0, 2: 1, 3: 1, 4: 0}, 1, 0)
    w3 = written["W3"]
    assert set(tree) <= written["W5"] | written["W5A"] | written["W5B"]
    assert set(ends) <= written["C1L"] | written["C1R"] | written["W4"] | written["W4S"]
    assert set(mid) <= written["CAE"] | w3
    assert set(rows) <= written["N2"] | written["N3"] and set(two) <= written["X3"] | written["N2"]
