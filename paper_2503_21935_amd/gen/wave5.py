"""Tables and colour code of the workgroup kernel for g g -> t tbar g g g
summed over spins with real polarisation vectors (csrc/me_wave5.h).

The kernel computes every wavefunction of one event once, as nodes of a few
kinds, and keeps them in LDS; which operands a node has, and which table
entries a configuration's colour-ordered amplitudes are made of, depends on
gluon labels and polarisation bits only and is tabulated here.  All offsets are
in double2 units of the workgroup's LDS block, two to a word: bits 4..17 and 18..31, so that the first one masked
and the second one shifted and masked are byte offsets.
"""
from __future__ import annotations

import itertools

from .colour import colour_matrix_exact, orderings

N = 5
THREADS = 768
ORDERED2 = list(itertools.permutations(range(N), 2))
ORDERED3 = list(itertools.permutations(range(N), 3))
PAIRS = list(itertools.combinations(range(N), 2))
TRIPLES = list(itertools.combinations(range(N), 3))
PERM3 = list(itertools.permutations(range(3)))


class Layout:
    """Regions of the LDS block (double2 units).  Those up to W2 (SMALL) are
    prepared for the next event, at WINDOW, while the present one still uses
    its own: inside W4, which is done with by then.  The colour sum takes J
    behind the window."""

    def __init__(self):
        o = 0
        for name, size in (("Q", 14), ("K", 60), ("F", 56), ("EPS", 20), ("N0", 16), ("C0", 16), ("N1", 160),
                           ("W2", 160), ("W3", 480), ("W4", 3840), ("N2", 1280)):
            setattr(self, name, o)
            o += size
        self.STAGE = o
        self.W5 = self.N3 = self.X3 = o            # 60 x 64 each
        self.CAE, self.C1 = o, o + 1280            # 20 x 64, 10 x 32
        self.END = o + 3840
        self.SMALL, self.WINDOW = self.W3, self.W4
        self.J = self.WINDOW + 512
        assert self.W4 <= self.WINDOW and self.SMALL <= 512 and self.J + 7680 <= self.END - 8
        assert self.END < 1 << 14


L = Layout()


def bits(p, labels):
    return sum(p[x] << i for i, x in enumerate(labels))


def q(a):
    return L.Q + 2 * a


def eps(a, p):
    return L.EPS + 4 * a + p[a]


def n0(e, s):
    return L.N0 + 8 * e + s


def n1(e, a, p, s):
    return L.N1 + 16 * (5 * e + a) + p[a] + 2 * s


def w2(x, y, p):
    return L.W2 + 8 * ORDERED2.index((x, y)) + p[x] + 2 * p[y]


def w3(x, y, z, p):
    """W(x, y, z) = W(z, y, x): by the set and its middle."""
    t = tuple(sorted((x, y, z)))
    return L.W3 + 48 * TRIPLES.index(t) + 16 * t.index(y) + bits(p, t)


def w4(order, p):
    t = tuple(sorted(order))
    m = next(a for a in range(N) if a not in t)
    rank = tuple(t.index(x) for x in order)
    return L.W4 + 32 * (24 * m + list(itertools.permutations(range(4))).index(rank)) + bits(p, t)


# five-gluon currents up to reflection (W is even under it)
W5_ORDERS = [o for o in orderings(N) if o < o[::-1]]
# those that start with gluon 0 are computed, the others follow from the shuffle identities
W5_DIRECT = [o for o in orderings(N) if o[0] == 0]


def w5(order, p):
    o = tuple(order)
    o = min(o, o[::-1])
    return L.W5 + 64 * W5_ORDERS.index(o) + bits(p, range(N))


def n2(e, x, y, p, s):
    """End e, gluon x absorbed first, then y."""
    return L.N2 + 32 * (20 * e + ORDERED2.index((x, y))) + p[x] + 2 * p[y] + 4 * s


def n3(x, y, z, p, s4):
    return L.N3 + 64 * ORDERED3.index((x, y, z)) + p[x] + 2 * p[y] + 4 * p[z] + 8 * s4


def c1(e, a, p, s3, s4):
    return L.C1 + 32 * (5 * e + a) + p[a] + 2 * s3 + 4 * s4


def cae(a, e, p, s3, s4):
    return L.CAE + 64 * ORDERED2.index((a, e)) + p[a] + 2 * p[e] + 4 * s3 + 8 * s4


def x3(a, b, c, p, s3):
    return L.X3 + 64 * ORDERED3.index((a, b, c)) + p[a] + 2 * p[b] + 4 * p[c] + 8 * s3


def pols(labels):
    """Polarisation assignments of some gluons, the first label's bit fastest."""
    for v in itertools.product((0, 1), repeat=len(labels)):
        yield dict(zip(labels, reversed(v)))


# F (and K = F - 26): pairs 0..9, triples 10..19, quads 20..24 (by the missing
# gluon), 25 p3 + p4, then the line: p3 - q_a, after pairs, p4 - q_a, before pairs
def f_pair(x, y):
    return L.F + PAIRS.index(tuple(sorted((x, y))))


def f_triple(t):
    return L.F + 10 + TRIPLES.index(tuple(sorted(t)))


def f_quad(t):
    return L.F + 20 + next(a for a in range(N) if a not in t)


def line(e, gl):
    return 15 * e + (gl[0] if len(gl) == 1 else 5 + PAIRS.index(tuple(sorted(gl))))


def momentum_coefficients():
    """Coefficients of (q0..q4, p3, p4) of the 56 summed momenta.  On the line
    the form with fewer beam momenta (q0, q1) is taken, which rounds less."""
    rows = []
    for s in PAIRS + TRIPLES + [tuple(x for x in range(N) if x != m) for m in range(N)]:
        rows.append([1 if a in s else 0 for a in range(N)] + [0, 0])
    rows.append([0] * N + [1, 1])
    for e in (0, 1):
        for s in [(a,) for a in range(N)] + PAIRS:
            rest = [x for x in range(N) if x not in s]
            if len(s) == 1 or sum(x < 2 for x in s) <= sum(x < 2 for x in rest):
                c = [-1 if a in s else 0 for a in range(N)] + ([1, 0] if e == 0 else [0, 1])
            else:
                c = [1 if a in rest else 0 for a in range(N)] + ([0, -1] if e == 0 else [-1, 0])
            rows.append(c)
    return rows


def nodes():
    """Operand lists of every kind of node."""
    out = {}
    out["W2"] = [[eps(x, p), eps(y, p), q(x), q(y), f_pair(x, y), w2(x, y, p), w2(y, x, p)]
                 for x, y in PAIRS for p in pols((x, y))]
    out["N1"] = [[n0(e, s), eps(a, p), L.K + 2 * line(e, (a,)), L.F + 26 + line(e, (a,)), n1(e, a, p, s)]
                 for e in (0, 1) for a in range(N) for s in (0, 1) for p in pols((a,))]
    rows = []
    for e in (0, 1):
        for x, y in ORDERED2:
            for s in (0, 1):
                for p in pols((x, y)):
                    # the pair current enters as W(x, y) from p3 and W(y, x) from p4
                    w = w2(x, y, p) if e == 0 else w2(y, x, p)
                    rows.append([n1(e, x, p, s), eps(y, p), n0(e, s), w, L.K + 2 * line(e, (x, y)),
                                 L.F + 26 + line(e, (x, y)), n2(e, x, y, p, s)])
    out["N2"] = rows
    rows = []
    for t in TRIPLES:
        for mid in t:
            a, c = [x for x in t if x != mid]
            for p in pols(t):
                rows.append([eps(a, p), eps(mid, p), eps(c, p), q(a), q(mid), q(c), w2(a, mid, p), w2(mid, c, p),
                             f_triple(t), w3(a, mid, c, p)])
    out["W3"] = rows
    direct, sums = [], []
    for m in range(N):
        t = [x for x in range(N) if x != m]
        for o in itertools.permutations(t[1:]):
            a, b, c, d = (t[0],) + o
            for p in pols(t):
                direct.append([eps(a, p), eps(b, p), eps(c, p), eps(d, p), q(a), q(b), q(c), q(d), w2(a, b, p),
                               w2(b, c, p), w2(c, d, p), w3(a, b, c, p), w3(b, c, d, p), f_quad(t),
                               w4((a, b, c, d), p), w4((d, c, b, a), p)])
                # W(b, a, c, d) = -[W(a, b, c, d) + W(a, c, b, d) + W(a, c, d, b)]
                sums.append([w4((a, b, c, d), p), w4((a, c, b, d), p), w4((a, c, d, b), p), w4((b, a, c, d), p),
                             w4((d, c, a, b), p)])
    out["W4"], out["W4S"] = direct, sums
    direct, sums = [], []
    for o in W5_DIRECT:
        for p in pols(range(N)):
            direct.append([eps(x, p) for x in o] + [q(x) for x in o]
                          + [w2(o[i], o[i + 1], p) for i in range(4)]
                          + [w3(*o[i:i + 3], p) for i in range(3)] + [w4(o[:4], p), w4(o[1:], p)]
                          + [w5(o, p)])
    for o in W5_ORDERS:
        k = o.index(0)
        if k == 0:
            continue
        # W(alpha, 0, beta) = (-1)^|alpha| sum of W(0, shuffles of alpha reversed with beta)
        if k > 2:
            o = o[::-1]
            k = o.index(0)
        if k == 4:
            raise ValueError("computed directly")
        al, be = o[:k][::-1], o[k + 1:]
        src = []
        for places in itertools.combinations(range(4), k):
            s, ia, ib = [], 0, 0
            for i in range(4):
                if i in places:
                    s.append(al[ia])
                    ia += 1
                else:
                    s.append(be[ib])
                    ib += 1
            src.append((0,) + tuple(s))
        for p in pols(range(N)):
            sums.append((k, [w5(s, p) for s in src] + [w5(o, p)]))
    out["W5"] = direct
    out["W5A"] = [r for k, r in sums if k == 1]   # minus the sum of four
    out["W5B"] = [r for k, r in sums if k == 2]   # the sum of six
    out["N3"] = [[n2(1, x, y, p, s), eps(z, p), n1(1, x, p, s), w2(z, y, p), n0(1, s), w3(z, y, x, p),
                  n3(x, y, z, p, s)] for x, y, z in ORDERED3 for s in (0, 1) for p in pols((x, y, z))]
    spins = [(s3, s4) for s4 in (0, 1) for s3 in (0, 1)]
    out["CAE"] = [[n1(0, a, p, s3), n1(1, e, p, s4), cae(a, e, p, s3, s4)]
                  for a, e in ORDERED2 for s3, s4 in spins for p in pols((a, e))]
    out["C1L"] = [[n1(0, a, p, s3), n0(1, s4), c1(0, a, p, s3, s4)]
                  for a in range(N) for s3, s4 in spins for p in pols((a,))]
    out["C1R"] = [[n0(0, s3), n1(1, a, p, s4), c1(1, a, p, s3, s4)]
                  for a in range(N) for s3, s4 in spins for p in pols((a,))]
    # L(a) W(bc) + ubar W(abc)
    out["X3"] = [[n1(0, a, p, s), w2(b, c, p), n0(0, s), w3(a, b, c, p), x3(a, b, c, p, s)]
                 for a, b, c in ORDERED3 for s in (0, 1) for p in pols((a, b, c))]
    return out


# The 120 flows by unordered first pair: unit u = 10 s4 + pair.  Each SIMD's
# three waves take two, two and one of the twenty units.


def slot_flows(pair):
    """(a, b, c, d, e) for the pair's two orders times the six orders of the rest."""
    rest = [x for x in range(N) if x not in pair]
    return [(pair[o], pair[1 - o]) + tuple(rest[i] for i in k) for o in (0, 1) for k in PERM3]


# stages of a configuration's sums and the entries each reads, per slot
def slot_entries(pair, p, s3, s4):
    rest = [x for x in range(N) if x not in pair]
    fl = slot_flows(pair)
    at = lambda o, k: fl[6 * o + k]  # noqa: E731
    tree = [w5(f, p) for f in fl]
    cur = []
    cur += [c1(0, pair[o], p, s3, s4) for o in (0, 1)]
    cur += [w4(at(o, k)[1:], p) for o in (0, 1) for k in range(6)]
    cur += [c1(1, rest[z], p, s3, s4) for z in range(3)]
    cur += [w4(at(o, k)[:4], p) for o in (0, 1) for k in range(6)]
    mid = [cae(pair[o], rest[z], p, s3, s4) for o in (0, 1) for z in range(3)]
    mid += [w3(*at(o, k)[1:4], p) for o in (0, 1) for k in range(6)]
    rows = [n2(0, pair[o], pair[1 - o], p, s3) for o in (0, 1)]
    rows += [n3(at(0, k)[4], at(0, k)[3], at(0, k)[2], p, s4) for k in range(6)]
    two = [x3(pair[o], pair[1 - o], rest[c], p, s3) for o in (0, 1) for c in range(3)]
    two += [n2(1, at(0, k)[4], at(0, k)[3], p, s4) for k in range(6)]
    return [tree, cur, mid, rows, two]


STAGE_SIZES = [12, 29, 18, 8, 12]


def words(entries, size):
    """Packed pairs, padded to whole int4."""
    w = [(entries[i] << 4) | ((entries[i + 1] if i + 1 < size else 0) << 18) for i in range(0, size, 2)]
    w = [v - (1 << 32) if v >> 31 else v for v in w]  # as int
    return w + [0] * (-len(w) % 4)


def table(name, rows):
    size = len(rows[0])
    packed = [words(r, size) for r in rows]
    quads = len(packed[0]) // 4
    out = [f"// {len(rows)} nodes, {size} offsets each, [int4 {quads}][node]",
           f"__device__ static const int4 tab_{name}[{quads * len(rows)}] = {{"]
    for k in range(quads):
        line_ = []
        for w in packed:
            line_.append("{" + ",".join(str(v) for v in w[4 * k:4 * k + 4]) + "}")
        for i in range(0, len(line_), 8):
            out.append("    " + ", ".join(line_[i:i + 8]) + ",")
    out.append("};")
    return out


# --------------------------------------------------------------------------
# Colour sum
# --------------------------------------------------------------------------

def colour_plan():
    """Blocks of the colour matrix.  N is unchanged when one relabelling acts on
    both orderings, and when both are reversed: sums and differences of J over
    the orbits of the Klein four-group on gluons 0..3 and of the reversal give
    eight blocks of 12 to 18 instead of one of 120.  Returns (orbits, blocks):
    orbit = (flows, sign rows), transformed value k of an orbit in place of its
    k-th flow; block = (places, coefficients)."""
    num, lcd = colour_matrix_exact(N)
    perms = orderings(N)
    kx = {s: i for i, s in enumerate(perms)}
    klein = [((0, 1, 2, 3, 4), (0, 0)), ((1, 0, 3, 2, 4), (1, 0)), ((2, 3, 0, 1, 4), (0, 1)),
             ((3, 2, 1, 0, 4), (1, 1))]
    chars = [(x, r) for x in itertools.product((0, 1), repeat=2) for r in (0, 1)]
    seen, orbits = set(), []
    members = {c: [] for c in chars}
    for s in perms:
        if s in seen:
            continue
        images = {}
        for g, ex in klein:
            for r in (0, 1):
                t = tuple(g[x] for x in s)
                t = t[::-1] if r else t
                images.setdefault(t, []).append((ex, r))
        seen |= set(images)
        flows = list(images)
        rows = []
        for x, rc in chars:
            sign = lambda ex, r: (-1) ** (ex[0] * x[0] + ex[1] * x[1] + r * rc)  # noqa: E731
            vals = [{sign(*h) for h in images[t]} for t in flows]
            if all(len(v) == 1 for v in vals):
                members[(x, rc)].append((len(orbits), len(rows)))
                rows.append([v.pop() for v in vals])
        assert len(rows) == len(flows)
        orbits.append(([kx[t] for t in flows], rows))
    blocks = []
    for c in chars:
        mem = members[c]
        if not mem:
            continue
        coef = []
        for oi, ri in mem:
            fi, si = orbits[oi][0], orbits[oi][1][ri]
            row = []
            for oj, rj in mem:
                fj, sj = orbits[oj][0], orbits[oj][1][rj]
                tot = sum(a * b * num[k][l] for k, a in zip(fi, si) for l, b in zip(fj, sj))
                row.append(tot / (len(fi) * len(fj)))
            coef.append(row)
        blocks.append(([orbits[o][0][r] for o, r in mem], coef))
    return orbits, blocks


def colour_waves(orbits, blocks, waves=6):
    """Orbits and blocks handed out to the waves of one configuration group."""
    def share(items, cost):
        load, got = [0] * waves, [[] for _ in range(waves)]
        for i in sorted(range(len(items)), key=lambda i: -cost(items[i])):
            w = min(range(waves), key=lambda w: load[w])
            load[w] += cost(items[i])
            got[w].append(items[i])
        return got
    return (share(orbits, lambda o: len(o[0]) * (3 if len(o[0]) == 8 else 2)),
            share(blocks, lambda b: len(b[0]) * (len(b[0]) + 1) // 2))


def emit_butterfly(flows, rows, at):
    """One orbit's signed sums in place, by a fast transform over sign bits."""
    out = []
    k = len(flows)
    for i, f in enumerate(flows):
        out.append(f"const double a{i} = {at(f)};")
    # rows are characters of an elementary 2-group: pairwise sums
    names = [f"a{i}" for i in range(k)]
    # index the flows by sign bits: flow j has the bit vector of its signs in generating rows
    gens, span = [], {tuple([1] * k): ()}
    for r in rows:
        t = tuple(r)
        if t not in span:
            gens.append(t)
            new = {}
            for v, c in span.items():
                new[tuple(x * y for x, y in zip(v, t))] = c + (len(gens) - 1,)
            span.update(new)
    ng = len(gens)
    assert 1 << ng == k
    slot = {}
    for j in range(k):
        b = sum((1 if gens[g][j] < 0 else 0) << g for g in range(ng))
        slot[b] = names[j]
    cur = [slot[b] for b in range(k)]
    n = 0
    for g in range(ng):
        nxt = list(cur)
        for b in range(k):
            if not b >> g & 1:
                x, y = cur[b], cur[b | 1 << g]
                out.append(f"const double t{n} = {x} + {y}, t{n + 1} = {x} - {y};")
                nxt[b], nxt[b | 1 << g] = f"t{n}", f"t{n + 1}"
                n += 2
        cur = nxt
    for i, r in enumerate(rows):
        c = span[tuple(r)]
        out.append(f"{at(flows[i])} = {cur[sum(1 << g for g in c)]};")
    return out


def emit_colour():
    orbits, blocks = colour_plan()
    osh, bsh = colour_waves(orbits, blocks)
    at = lambda f: f"J[{128 * f}]"  # noqa: E731
    out = ["// Signed sums of one part (real or imaginary) of J over orbits, in place: wave w of",
           "// a configuration group; J points at the lane's column of [flow][128].",
           "template <int W>", "MEV void colour_orbits(double* __restrict__ J) {"]
    for w, items in enumerate(osh):
        out.append(f"    {'if' if w == 0 else '} else if'} constexpr (W == {w}) {{")
        for flows, rows in items:
            out.append("        {")
            out += ["            " + s for s in emit_butterfly(flows, rows, at)]
            out.append("        }")
    out += ["    }", "}", "",
            "// wave W's blocks of J^T N J over the signed sums.",
            "template <int W>", "MEV double colour_quads(const double* __restrict__ J) {", "    double acc = 0.0;"]
    for w, items in enumerate(bsh):
        out.append(f"    {'if' if w == 0 else '} else if'} constexpr (W == {w}) {{")
        for places, coef in items:
            out.append("        {")
            for i, f in enumerate(places):
                out.append(f"            const double h{i} = {at(f)};")
            for i in range(len(places)):
                z = f"{coef[i][i]!r} * h{i}"
                for j in range(i + 1, len(places)):
                    assert coef[i][j] == coef[j][i]
                    if coef[i][j]:
                        z = f"fma({2 * coef[i][j]!r}, h{j}, {z})"
                out.append(f"            acc = fma(h{i}, {z}, acc);")
            out.append("        }")
    out += ["    }", "    return acc;", "}"]
    return out


def render():
    h = ["// Generated by paper_2503_21935_amd.gen.wave5: g g -> t tbar g g g, one event per workgroup.",
         "#pragma once", '#include "me_vertex.h"', "", "namespace w5 {", "", "enum {"]
    for k in ("Q", "K", "F", "EPS", "N0", "C0", "N1", "W2", "W3", "W4", "N2", "STAGE", "W5", "N3", "X3", "CAE", "C1",
              "END", "SMALL",
              "WINDOW", "J"):
        h.append(f"    S_{k} = {getattr(L, k)},")
    h.append("};")
    co = momentum_coefficients()
    h.append("// coefficients of (gluons 0..4, p3, p4) of the summed momenta, two bits each: 1 plus, 2 minus")
    h.append(f"__device__ static const int tab_K[{len(co)}] = {{")
    h.append("    " + ", ".join(str(sum((1 if c > 0 else 2 if c < 0 else 0) << 2 * i for i, c in enumerate(r)))
                                for r in co))
    h.append("};")
    nd = nodes()
    for name, rows in nd.items():
        for r in rows:
            if not all(0 <= v < L.END for v in r):
                raise ValueError(f"offset outside the block in {name}")
        h.append(f"enum {{ N_{name} = {len(rows)} }};")
        h += table(name, rows)
    quads = [len(words(list(range(n)), n)) // 4 for n in STAGE_SIZES]
    per = sum(quads)
    h.append("// int4 of each stage's entries, and where they start")
    for i, name in enumerate(("TREE", "ENDS", "MID", "ROWS", "TWO")):
        h.append(f"enum {{ Q_{name} = {quads[i]}, AT_{name} = {sum(quads[:i])} * 64 }};")
    h.append(f"// entries of configuration `lane` (bits 0..4 polarisations, 5 the spin of t): [unit 20][int4 {per}][lane]")
    h.append(f"enum {{ CFG_UNIT = {per} * 64 }};")
    h.append(f"__device__ static const int4 tab_cfg[{20 * per * 64}] = {{")
    for s4 in (0, 1):
        for pair in PAIRS:
            lanes = []
            for lane in range(64):
                p = {a: lane >> a & 1 for a in range(N)}
                ent = slot_entries(pair, p, lane >> 5 & 1, s4)
                if [len(e) for e in ent] != STAGE_SIZES or not all(0 <= v < L.END for e in ent for v in e):
                    raise ValueError("bad entries")
                lanes.append(sum((words(e, len(e)) for e in ent), []))
            for k in range(per):
                row = ["{" + ",".join(str(v) for v in w[4 * k:4 * k + 4]) + "}" for w in lanes]
                for i in range(0, 64, 8):
                    h.append("    " + ", ".join(row[i:i + 8]) + ",")
    h.append("};")
    kx = {s: i for i, s in enumerate(orderings(N))}
    h.append("// flow of each of a unit's sums: [pair 10][12]")
    h.append("__device__ static const int tab_flow[120] = {")
    for pair in PAIRS:
        h.append("    " + ", ".join(str(kx[f]) for f in slot_flows(pair)) + ",")
    h.append("};")
    h += emit_colour()
    h += ["", "}  // namespace w5"]
    return "\n".join(h) + "\n"
