"""What a user of this library has it do, as cases that can be timed.

Kinds of case (the public entry points of ``paper_2503_21935_amd``):

  eval      |M|^2 of a batch of phase-space points in float64
            (``MatrixElement.eval``), the step the library exists for;
  mixed     the same with the mixed-precision form chosen;
  channels  |M|^2 and the single-diagram weight of each event's channel;
  sample    flat phase-space points and their weights (``rambo``);
  train     an epoch's worth of surrogate training steps in one call, then the
            parameters read back, as a program does that keeps them;
  unweight  two-stage unweighting with the surrogate as its first stage.

Sizes are those of the benchmark and the tests: 2^20 points for the benchmark
process, 2^14 for a generator's own batch, a few dozen where an integrator asks
for single points; odd ones in between.  Inputs are flat phase-space points
made on the GPU from the seed, with torch alone.
"""
import itertools
import math

import numpy as np
import torch

import paper_2503_21935_amd as me

# final-state masses and energies (GeV) of the processes, as in ``inputs``
MT = 173.0
KIN = {
    "ee_mumu": (500.0, (0.0, 0.0)),
    "gg_tt": (13000.0, (MT, MT)),
    "gg_ttg": (13000.0, (MT, MT, 0.0)),
    "gg_ttgg": (13000.0, (MT, MT, 0.0, 0.0)),
    "gg_ttggg": (13000.0, (MT, MT, 0.0, 0.0, 0.0)),
    "gux_taptamux": (13000.0, (0.0,) * 3),
    "gux_taptamgux": (13000.0, (0.0,) * 4),
    "gux_taptamggux": (13000.0, (0.0,) * 5),
}
# operations of one event over all helicities with every wavefunction computed
# once (the library's own algorithmic count, bench.py's roofline figure)
FLOPS = {"ee_mumu": 2.6e3, "gg_tt": 1.0e4, "gg_ttg": 9.6e4, "gg_ttgg": 1.664e6, "gg_ttggg": 2.722e7,
         "gux_taptamux": 5.0e3, "gux_taptamgux": 3.7e4, "gux_taptamggux": 3.422e5}
# about what one sampled particle costs: two rounds of counter-based random
# numbers, a logarithm, a sine and cosine, the boost and the mass rescaling
SAMPLE_FLOPS = 300
BATCH, WIDTH, DEPTH, N_IN = 4096, 256, 4, 24
MLP_FLOPS = 2 * (N_IN * WIDTH + (DEPTH - 1) * WIDTH * WIDTH + WIDTH)
N_PARAMS = N_IN * WIDTH + WIDTH + (DEPTH - 1) * (WIDTH * WIDTH + WIDTH) + WIDTH + 1


def listed():
    return [
        # a smoke-size batch of the simplest process: launch and host path
        {"name": "eemumu_16k", "kind": "eval", "process": "ee_mumu", "events": 16384},
        # a large batch of the smallest gluon process
        {"name": "ggtt_1m", "kind": "eval", "process": "gg_tt", "events": 1 << 20},
        # single points asked for by an integrator: latency
        {"name": "ggttgg_48", "kind": "eval", "process": "gg_ttgg", "events": 48},
        # an event generator's own batch
        {"name": "ggttgg_16k", "kind": "eval", "process": "gg_ttgg", "events": 16384},
        # the benchmark workload
        {"name": "ggttgg_1m", "kind": "eval", "process": "gg_ttgg", "events": 1 << 20},
        # the heaviest process, an odd batch
        {"name": "ggttggg_50k", "kind": "eval", "process": "gg_ttggg", "events": 50021},
        # the Drell-Yan + 3 jets subprocess
        {"name": "dy3j_1m", "kind": "eval", "process": "gux_taptamggux", "events": 1 << 20},
        # the mixed-precision option on a generator's larger batch
        {"name": "mixed_ggttgg_128k", "kind": "mixed", "process": "gg_ttgg", "events": 1 << 17},
        # multi-channel integration: events of all channels in one call
        {"name": "channels_ggttgg_64k", "kind": "channels", "process": "gg_ttgg", "events": 1 << 16},
        # the points of such a batch, made on the GPU
        {"name": "sample_ggttgg_1m", "kind": "sample", "process": "gg_ttgg", "events": 1 << 20},
        # surrogate training
        {"name": "train_64", "kind": "train", "steps": 64},
        # unweighting a sample
        {"name": "unweight_1m", "kind": "unweight", "process": "gg_ttgg", "events": 1 << 20},
    ]


def _log_int(rng, lo, hi):
    return max(lo, min(hi, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def draw(rng):
    kind = rng.choice(["eval"] * 6 + ["mixed", "channels", "sample", "train", "unweight"])
    if kind == "train":
        return {"kind": kind, "steps": _log_int(rng, 4, 128)}
    if kind == "unweight":
        return {"kind": kind, "process": "gg_ttgg", "events": _log_int(rng, 4096, 1 << 20)}
    if kind == "mixed":
        return {"kind": kind, "process": "gg_ttgg", "events": _log_int(rng, 64, 1 << 18)}
    if kind == "channels":
        proc = rng.choice(["gg_tt", "gg_ttg", "gg_ttgg"])
        return {"kind": kind, "process": proc, "events": _log_int(rng, 64, 1 << (16 if proc == "gg_ttgg" else 19))}
    if kind == "sample":
        return {"kind": kind, "process": rng.choice(["gg_tt", "gg_ttgg", "gg_ttggg", "gux_taptamggux"]),
                "events": _log_int(rng, 256, 1 << 20)}
    proc = rng.choice(list(KIN) + ["gg_ttgg", "gg_ttgg", "gg_ttggg"])
    top = {"gg_ttggg": 1 << 16, "ee_mumu": 1 << 18}.get(proc, 1 << 20)
    return {"kind": kind, "process": proc, "events": _log_int(rng, 32, top)}


# --------------------------------------------------------------------------
# Inputs
# --------------------------------------------------------------------------

def _generator(seed):
    g = torch.Generator(device="cuda")
    g.manual_seed(int(seed) + 17)
    return g


def _flat_points(roots, masses, n, g):
    """n flat phase-space points: [n][2 + nf][4]."""
    u = torch.rand(n, len(masses), 4, dtype=torch.float64, device="cuda", generator=g).clamp_min(1e-300)
    return _map_points(roots, masses, u)


def _map_points(roots, masses, u):
    """RAMBO (Kleiss, Stirling, Ellis): uniforms [n][nf][4] to momenta."""
    n, nf = u.shape[:2]
    c, phi = 2 * u[..., 0] - 1, 2 * math.pi * u[..., 1]
    q0 = -torch.log(u[..., 2] * u[..., 3])
    st = torch.sqrt(1 - c * c)
    q = torch.stack([st * torch.cos(phi), st * torch.sin(phi), c], -1) * q0[..., None]
    del u, c, phi, st
    E, P = q0.sum(1), q.sum(1)
    m = torch.sqrt(E * E - (P * P).sum(-1))
    b, x, gam = -P / m[:, None], roots / m, E / m
    bq = (q * b[:, None]).sum(-1)
    e = x[:, None] * (gam[:, None] * q0 + bq)
    k = x[:, None, None] * (q + b[:, None] * (q0 + bq / (1 + gam)[:, None])[..., None])
    m2 = torch.tensor(masses, dtype=torch.float64, device="cuda") ** 2
    if max(masses) > 0:
        xi = torch.ones(n, 1, dtype=torch.float64, device="cuda")
        for _ in range(12):  # Newton on a convex increasing function, from its right
            en = torch.sqrt(m2 + (xi * e) ** 2)
            xi = xi - (en.sum(1, True) - roots) / (xi * e * e / en).sum(1, True)
        k = xi[..., None] * k
    out = torch.zeros(n, 2 + nf, 4, dtype=torch.float64, device="cuda")
    out[:, :2, 0] = 0.5 * roots
    out[:, 0, 3], out[:, 1, 3] = 0.5 * roots, -0.5 * roots
    out[:, 2:, 1:] = k
    out[:, 2:, 0] = torch.sqrt(m2 + (k * k).sum(-1))
    return out


def _points(process, n, seed):
    return _flat_points(*KIN[process], n, _generator(seed))


def _cuts(mom):
    """p_T > 20 GeV, |eta| < 5, Delta R > 0.4 on the final gluons."""
    p = mom[:, 4:, 1:]
    pt = torch.hypot(p[..., 0], p[..., 1])
    eta = torch.asinh(p[..., 2] / pt)
    phi = torch.atan2(p[..., 1], p[..., 0])
    ok = ((pt > 20.0) & (eta.abs() < 5.0)).all(1)
    for i, j in itertools.combinations(range(p.shape[1]), 2):
        dphi = (phi[:, i] - phi[:, j]).abs()
        dphi = torch.minimum(dphi, 2 * math.pi - dphi)
        ok &= torch.hypot(eta[:, i] - eta[:, j], dphi) > 0.4
    return ok


def _network(seed=1004):
    """The library's initial parameters of the surrogate (splitmix64, He-uniform)."""
    out, st = [], 0

    def uniform(n, fan_in):
        nonlocal st
        with np.errstate(over="ignore"):
            z = np.uint64(seed) + np.arange(st + 1, st + n + 1, dtype=np.uint64) * np.uint64(0x9E3779B97F4A7C15)
            z = (z ^ (z >> np.uint64(30))) * np.uint64(0xBF58476D1CE4E5B9)
            z = (z ^ (z >> np.uint64(27))) * np.uint64(0x94D049BB133111EB)
            z ^= z >> np.uint64(31)
        st += n
        return math.sqrt(6.0 / fan_in) * (2.0 * (z >> np.uint64(11)).astype(np.float64) / 2.0 ** 53 - 1.0)

    fan = N_IN
    for _ in range(DEPTH):
        out += [uniform(WIDTH * fan, fan).astype(np.float32).reshape(WIDTH, fan), np.zeros(WIDTH, np.float32)]
        fan = WIDTH
    return out + [uniform(WIDTH, WIDTH).astype(np.float32), np.zeros(1, np.float32)]


def _forward(theta, x):
    h = x
    for k in range(DEPTH):
        h = torch.nn.functional.silu(h @ theta[2 * k].T + theta[2 * k + 1])
    return h @ theta[-2] + theta[-1]


def _features(mom):
    s = (mom[:, 0] + mom[:, 1])
    roots = torch.sqrt(s[:, 0] ** 2 - (s[:, 1:] ** 2).sum(-1))
    return (mom.reshape(mom.shape[0], -1) / roots[:, None]).float()


def _train_data(case, seed):
    """Network inputs, standardised targets, the epoch's order and its rates."""
    n = 1 << 17
    g = _generator(seed)
    mom = _flat_points(*KIN["gg_ttgg"], n, g)
    t = -torch.log(torch.hypot(mom[:, 2:, 1], mom[:, 2:, 2])).sum(1)
    t = ((t - t.mean()) / t.std()).float()
    steps = case["steps"]
    rounds = -(-steps * BATCH // n)
    idx = torch.cat([torch.randperm(n, device="cuda", generator=g) for _ in range(rounds)])[:steps * BATCH]
    lr = 5e-4 * (1 + torch.cos(math.pi * torch.arange(steps, dtype=torch.float32, device="cuda") / steps))
    return _features(mom), t, idx.to(torch.int32).contiguous(), lr


def prepare(case, seed):
    kind = case["kind"]
    if kind == "train":
        x, t, idx, lr = _train_data(case, seed)
        return {"kind": kind, "net": me.Surrogate(n_in=N_IN, width=WIDTH, depth=DEPTH, seed=1004), "x": x, "t": t,
                "idx": idx, "lr": lr, "loss": torch.empty(case["steps"], dtype=torch.float32, device="cuda")}
    proc, n = case["process"], case["events"]
    if kind == "sample":
        return {"kind": kind, "kin": KIN[proc], "seed": int(seed) * 7919 + 3, "n": n}
    mom = _points(proc, n, seed)
    m = me.MatrixElement(proc)
    st = {"kind": kind, "me": m, "mom": mom}
    if kind == "mixed":
        m.set_precision(me.ME_MIXED, 1e-5)
    elif kind == "channels":
        st["chan"] = torch.randint(0, len(m.channels()), (n,), dtype=torch.int32, device="cuda",
                                   generator=_generator(seed + 1))
    elif kind == "unweight":
        # the maxima come from a calibration sample, here with the network's
        # float32 values from torch
        g = _generator(seed + 1)
        cal = _points(proc, 16384, seed + 2)
        theta = [torch.from_numpy(p).cuda() for p in _network()]
        y = _forward(theta, _features(cal)).double()
        sig, mu = 4.0 / float(y.std()), -4.0 * float(y.mean() / y.std())
        w = _cuts(cal).double()
        s, ex = torch.exp(sig * y + mu) * w, m.eval(cal) * w
        ok = s > 0
        st.update(net=me.Surrogate(n_in=N_IN, width=WIDTH, depth=DEPTH, seed=1004), w=_cuts(mom).double(),
                  u=torch.rand(n, 2, dtype=torch.float64, device="cuda", generator=g), mu=mu, sig=sig,
                  s_max=float(torch.quantile(s[ok], 0.999)), r_max=float(torch.quantile(ex[ok] / s[ok], 0.9)),
                  idx=torch.empty(n, dtype=torch.int32, device="cuda"),
                  wt=torch.empty(n, dtype=torch.float64, device="cuda"),
                  count=torch.zeros(2, dtype=torch.int32, device="cuda"))
    return st


def run(st):
    kind = st["kind"]
    if kind == "eval" or kind == "mixed":
        return st["me"].eval(st["mom"])
    if kind == "channels":
        return st["me"].eval_multichannel(st["mom"], st["chan"])
    if kind == "sample":
        return me.rambo(*st["kin"], st["seed"], st["n"])
    if kind == "train":
        st["net"].train_steps(st["x"], st["t"], st["idx"], BATCH, st["lr"], st["loss"])
        return {"loss": st["loss"], "params": st["net"].get_params()}
    me.unweight_two_stage(st["me"].ctx, st["net"].h, st["mom"], st["w"], st["mom"].shape[0], st["u"], st["mu"],
                          st["sig"], st["s_max"], st["r_max"], st["idx"], st["wt"], st["count"])
    kept = int(st["count"][1])
    # the accepted points come in any order: each one's weight at its event
    weights = torch.zeros_like(st["w"])
    weights[st["idx"][:kept].long()] = st["wt"][:kept]
    return {"weights": weights, "count": st["count"].clone()}


def work(case):
    if case["kind"] == "train":
        steps = case["steps"]
        # each batch's rows once, the parameters and moments in and out once
        return {"bytes": steps * BATCH * (N_IN + 1 + 1) * 4 + 6 * N_PARAMS * 4, "flops": 3 * MLP_FLOPS * steps * BATCH}
    n, proc = case["events"], case["process"]
    npart = 2 + len(KIN[proc][1])
    if case["kind"] == "unweight":
        # momenta, weights and uniforms in; the network on every point
        return {"bytes": n * (npart * 32 + 8 + 16), "flops": n * MLP_FLOPS}
    if case["kind"] == "sample":
        return {"bytes": n * (npart * 32 + 8), "flops": n * (npart - 2) * SAMPLE_FLOPS}
    extra = {"eval": 0, "mixed": 0, "channels": 12}[case["kind"]]
    return {"bytes": n * (npart * 32 + 8 + extra), "flops": n * FLOPS[proc]}


# --------------------------------------------------------------------------
# The same values in 64 bits, with torch alone
# --------------------------------------------------------------------------

ALPHA_S, INV_ALPHA, G_F, W_TOP, MZ, WZ = 0.118, 132.507, 1.16639e-5, 1.4915, 91.188, 2.4414
METRIC = (1.0, -1.0, -1.0, -1.0)


def _gamma():
    s = [np.eye(2), np.array([[0, 1], [1, 0]]), np.array([[0, -1j], [1j, 0]]), np.diag([1, -1])]
    return [np.block([[np.zeros((2, 2)), s[k]], [(1 if k == 0 else -1) * s[k], np.zeros((2, 2))]]).astype(complex)
            for k in range(4)]


GAMMA = _gamma()


def _cplx(a, dev):
    return torch.from_numpy(np.asarray(a, dtype=complex)).to(dev)


def _slash(w):
    """gamma.w as [..., 4, 4] of a (real or complex) contravariant vector [..., 4]."""
    return sum(METRIC[k] * w[..., k, None, None] * _cplx(GAMMA[k], w.device) for k in range(4))


def _row(f, a):
    return (f[..., :, None] * a).sum(-2)


def _dot(a, b):
    return a[..., 0] * b[..., 0] - a[..., 1] * b[..., 1] - a[..., 2] * b[..., 2] - a[..., 3] * b[..., 3]


def _spinors(p, m, anti):
    """u(p, s) or v(p, s), s = 0, 1, in the rest-frame spin basis: [n, 2, 4]."""
    r = 1 / math.sqrt(2.0)
    base = _cplx([[r, 0, -r, 0], [0, r, 0, -r]] if anti else [[r, 0, r, 0], [0, r, 0, r]], p.device)
    a = (-1 if anti else 1) * _slash(p) + m * torch.eye(4, dtype=torch.complex128, device=p.device)
    return (a[:, None] * base[None, :, None, :]).sum(-1) / torch.sqrt(p[:, 0] + m)[:, None, None]


def _bar(u):
    return (u.conj()[..., :, None] * _cplx(GAMMA[0], u.device)).sum(-2)


def _polarisations(k):
    """Two real transverse vectors without time component: [n, 2, 4]."""
    kt, kk = torch.hypot(k[:, 1], k[:, 2]), torch.sqrt((k[:, 1:] ** 2).sum(-1))
    axis = kt == 0
    cp = torch.where(axis, torch.ones_like(kt), k[:, 1] / torch.where(axis, torch.ones_like(kt), kt))
    sp = torch.where(axis, torch.zeros_like(kt), k[:, 2] / torch.where(axis, torch.ones_like(kt), kt))
    c, s, z = k[:, 3] / kk, kt / kk, torch.zeros_like(kt)
    return torch.stack([torch.stack([z, c * cp, c * sp, -s], -1), torch.stack([z, -sp, cp, z], -1)], 1)


def _vvv(x, qx, y, qy):
    return _dot(x, y)[..., None] * (qx - qy) + _dot(qx + 2 * qy, x)[..., None] * y - _dot(2 * qx + qy, y)[..., None] * x


def _ordered_amplitudes(q, eps, row, prow, mass, width, col, ins=None, qins=None):
    """Colour-ordered amplitudes of a quark line with gluons (Berends, Giele),
    momenta q flowing in, polarisations eps [n, 2, 4] with the coupling in
    them; with an insertion ins (a matrix [n, K, 4, 4] of momentum qins), once
    on the line.  {ordering: [n, 2 (row), 2 (each gluon in label order),
    (K,) 2 (col)]}, up to a common phase."""
    ng = len(q)
    n = q[0].shape[0]
    dims = [1] * ng

    def spread(v, labels):
        """[n, 2 per label in order, 4] -> [n, 1 or 2 per gluon 0..ng-1, 4]"""
        perm = sorted(range(len(labels)), key=lambda i: labels[i])
        v = v.permute([0] + [1 + i for i in perm] + [1 + len(labels)])
        shape = list(dims)
        for a in labels:
            shape[a] = 2
        return v.reshape([n] + shape + [4])

    Q = lambda s: sum(q[a] for a in s).reshape([n] + dims + [4])  # noqa: E731
    W = {}

    def current(s):
        if len(s) == 1:
            return spread(eps[s[0]], s)
        if s not in W:
            out = 0
            for j in range(1, len(s)):
                out = out - _vvv(current(s[:j]), Q(s[:j]), current(s[j:]), Q(s[j:]))
            for i in range(1, len(s) - 1):
                for j in range(i + 1, len(s)):
                    x, y, z = current(s[:i]), current(s[i:j]), current(s[j:])
                    out = out + 2 * _dot(x, z)[..., None] * y - _dot(y, z)[..., None] * x - _dot(x, y)[..., None] * z
            W[s] = out / _dot(Q(s), Q(s))[..., None]
        return W[s]

    eye = torch.eye(4, dtype=torch.complex128, device=q[0].device)
    S = {}

    def slash(s):
        if s not in S:
            S[s] = _slash(current(s))[:, None]  # a place for the row's spin
        return S[s]

    def prop(f, s, inserted):
        p = prow.reshape([n] + dims + [4]) - (Q(s) if s else 0)
        if inserted:
            p = p - qins.reshape([n] + dims + [4])
        den = _dot(p, p) - mass * mass + 1j * mass * width
        return -_row(f, (_slash(p) + mass * eye)[:, None]) / den[:, None, ..., None]

    if ins is None:
        L = {(): row.reshape([n, 2] + dims + [4])}

        def line(s):
            if s not in L:
                L[s] = prop(sum(_row(line(s[:j]), slash(s[j:])) for j in range(len(s))), s, False)
            return L[s]

        return {s: (sum(_row(line(s[:j]), slash(s[j:])) for j in range(ng))[..., None, :]
                    * col.reshape([n, 1] + dims + [2, 4])).sum(-1)
                for s in itertools.permutations(range(ng))}
    # with an insertion: one more axis (its K values) as part of the row's axis
    K = ins.shape[1]
    L0, L1 = {(): row.reshape([n, 2] + dims + [4])}, {}

    def line0(s):
        if s not in L0:
            L0[s] = prop(sum(_row(line0(s[:j]), slash(s[j:])) for j in range(len(s))), s, False)
        return L0[s]

    def insert(f):
        g = (f.unsqueeze(2)[..., :, None] * ins.reshape([n, 1, K] + dims + [4, 4])).sum(-2)
        return g.reshape([n, 2 * K] + list(g.shape[3:]))

    def line1(s):
        if s not in L1:
            L1[s] = prop(insert(line0(s)) + sum(_row(line1(s[:j]), slash(s[j:])) for j in range(len(s))), s, True)
        return L1[s]

    return {s: ((insert(line0(s)) + sum(_row(line1(s[:j]), slash(s[j:])) for j in range(ng)))[..., None, :]
                * col.reshape([n, 1] + dims + [2, 4])).sum(-1)
            for s in itertools.permutations(range(ng))}


_COLOUR = {}


def _colour(ng):
    """Colour matrix of the orderings, from the Gell-Mann matrices."""
    if ng in _COLOUR:
        return _COLOUR[ng]
    l = np.zeros((8, 3, 3), dtype=complex)
    for k, (i, j) in ((0, (0, 1)), (3, (0, 2)), (5, (1, 2))):
        l[k][i, j] = l[k][j, i] = 1
    for k, (i, j) in ((1, (0, 1)), (4, (0, 2)), (6, (1, 2))):
        l[k][i, j], l[k][j, i] = -1j, 1j
    l[2] = np.diag([1, -1, 0])
    l[7] = np.diag([1, 1, -2]) / math.sqrt(3)
    T = l / 2
    w = T
    for _ in range(ng - 1):
        w = np.einsum("...ij,bjk->...bik", w, T)
    perms = list(itertools.permutations(range(ng)))
    first = {p: float(np.vdot(w, np.transpose(w, list(np.argsort(p)) + [ng, ng + 1])).real) for p in perms}
    inv = [tuple(np.argsort(p)) for p in perms]
    _COLOUR[ng] = np.array([[first[tuple(inv[i][a] for a in t)] for t in perms] for i in range(len(perms))])
    return _COLOUR[ng]


def _colour_sum(J, ng):
    n = next(iter(J.values())).shape[0]
    a = torch.stack([J[p].reshape(n, -1) for p in itertools.permutations(range(ng))], 1)  # [n, flows, configurations]
    a = torch.view_as_real(a.permute(1, 0, 2).contiguous()).reshape(a.shape[1], -1)
    c = torch.from_numpy(_colour(ng)).to(a.device)
    return (a * (c @ a)).sum(0).reshape(n, -1).sum(1)


def _me2_gluons(mom):
    ng = mom.shape[1] - 2
    gs = math.sqrt(4 * math.pi * ALPHA_S)
    parts = [0, 1] + list(range(4, ng + 2))
    q = [mom[:, p] if p < 2 else -mom[:, p] for p in parts]
    eps = [gs * _polarisations(mom[:, p]) for p in parts]
    J = _ordered_amplitudes(q, eps, _bar(_spinors(mom[:, 2], MT, False)), mom[:, 2], MT, W_TOP,
                            _spinors(mom[:, 3], MT, True))
    return _colour_sum(J, ng) / (256.0 * math.factorial(ng - 2))


def _electroweak():
    alpha = 1 / INV_ALPHA
    mw2 = MZ ** 2 / 2 + math.sqrt(MZ ** 4 / 4 - math.pi * alpha * MZ ** 2 / (math.sqrt(2) * G_F))
    sw2 = 1 - mw2 / MZ ** 2
    e = math.sqrt(4 * math.pi * alpha)
    return e, e / math.sqrt(sw2 * (1 - sw2)), sw2


def _current(f, psi, left, right):
    """f gamma^mu (left P_L + right P_R) psi for all spins: [n, 2, 2, 4]."""
    w = torch.tensor([left, left, right, right], dtype=torch.complex128, device=f.device)
    return torch.stack([(_row(f, _cplx(GAMMA[k], f.device))[:, :, None] * (w * psi)[:, None]).sum(-1)
                        for k in range(4)], -1)


def _me2_eemumu(mom):
    e, gz, sw2 = _electroweak()
    gl, gr = -0.5 + sw2, sw2
    a = (_bar(_spinors(mom[:, 0], 0.0, True)), _spinors(mom[:, 1], 0.0, False))
    b = (_bar(_spinors(mom[:, 3], 0.0, False)), _spinors(mom[:, 2], 0.0, True))
    k = mom[:, 0] + mom[:, 1]
    s = _dot(k, k)[:, None, None, None, None]

    def contract(x, y):
        return _dot(x[:, :, :, None, None], y[:, None, None])

    amp = (e * e / s) * contract(_current(*a, 1, 1), _current(*b, 1, 1)) \
        + gz * gz / (s - MZ ** 2 + 1j * MZ * WZ) * contract(_current(*a, gl, gr), _current(*b, gl, gr))
    return (amp.abs() ** 2).reshape(mom.shape[0], -1).sum(1) / 4


def _me2_lepton_pair(mom):
    """g ubar -> tau+ tau- (gluons) ubar."""
    e, gz, sw2 = _electroweak()
    gs = math.sqrt(4 * math.pi * ALPHA_S)
    last = mom.shape[1] - 1
    gl = [0] + list(range(4, last))
    ng = len(gl)
    q = [mom[:, p] if p < 2 else -mom[:, p] for p in gl]
    eps = [gs * _polarisations(mom[:, p]) for p in gl]
    lp, lm = mom[:, 2], mom[:, 3]
    k = lp + lm
    k2 = _dot(k, k)[:, None, None]
    f, v = _bar(_spinors(lm, 0.0, False)), _spinors(lp, 0.0, True)
    jg = _current(f, v, 1, 1).reshape(-1, 4, 4)
    jz = _current(f, v, -0.5 + sw2, sw2).reshape(-1, 4, 4)
    qq, t3 = 2.0 / 3.0, 0.5
    photon = -qq * e * e / k2 * jg
    z = gz * gz / (k2 - MZ ** 2 + 1j * MZ * WZ) * jz
    pl = torch.diag(torch.tensor([1, 1, 0, 0], dtype=torch.complex128, device=mom.device))
    pr = torch.diag(torch.tensor([0, 0, 1, 1], dtype=torch.complex128, device=mom.device))
    ins = (_slash(photon + (t3 - qq * sw2) * z)[..., :, :, None] * pl).sum(-2) \
        + (_slash(photon - qq * sw2 * z)[..., :, :, None] * pr).sum(-2)
    # the row end is the incoming antiquark: momentum -p on the line
    J = _ordered_amplitudes(q, eps, _bar(_spinors(mom[:, 1], 0.0, True)), -mom[:, 1], 0.0, 0.0,
                            _spinors(mom[:, last], 0.0, True), ins, -k)
    return _colour_sum(J, ng) / (4 * 24 * math.factorial(ng - 1))


def _me2(process, mom):
    if process == "ee_mumu":
        return _me2_eemumu(mom)
    fn, chunk = (_me2_gluons, {4: 1 << 18, 5: 1 << 17, 6: 1 << 15, 7: 1 << 12}) if process.startswith("gg") else \
        (_me2_lepton_pair, {5: 1 << 17, 6: 1 << 16, 7: 1 << 14})
    step = chunk[mom.shape[1]]
    return torch.cat([fn(mom[o:o + step]) for o in range(0, mom.shape[0], step)])


def _train_exact(case, seed):
    x, t, idx, lr = _train_data(case, seed)
    x, t, idx = x.double(), t.double(), idx.long()
    theta = [torch.from_numpy(p).cuda().double().requires_grad_(True) for p in _network()]
    m, v = [torch.zeros_like(p) for p in theta], [torch.zeros_like(p) for p in theta]
    losses = []
    for k in range(case["steps"]):
        rows = idx[k * BATCH:(k + 1) * BATCH]
        loss = ((_forward(theta, x[rows]) - t[rows]) ** 2).mean()
        grads = torch.autograd.grad(loss, theta)
        losses.append(loss.detach())
        with torch.no_grad():
            for p, g, a, b in zip(theta, grads, m, v):
                a.mul_(0.9).add_(0.1 * g)
                b.mul_(0.999).add_(0.001 * g * g)
                p -= lr[k].double() * (a / (1 - 0.9 ** (k + 1))) / (torch.sqrt(b / (1 - 0.999 ** (k + 1))) + 1e-8)
    return {"loss": torch.stack(losses), "params": torch.cat([p.detach().reshape(-1) for p in theta]).cpu().numpy()}


def _philox(event, block, seed):
    """Philox4x32-10 (Salmon et al.) of counter (event, block, 0), two uniforms."""
    mask = 0xFFFFFFFF

    def mul(a, b):  # 32 x 32 -> high and low words
        low = a * (b & 0xFFFF)
        return ((a * (b >> 16) + (low >> 16)) >> 16) & mask, (a * b) & mask

    c = [event & mask, event >> 32, torch.full_like(event, block), torch.zeros_like(event)]
    k0, k1 = seed & mask, seed >> 32
    for _ in range(10):
        (h0, l0), (h1, l1) = mul(c[0], 0xD2511F53), mul(c[2], 0xCD9E8D57)
        c = [h1 ^ c[1] ^ k0, l1, h0 ^ c[3] ^ k1, l0]
        k0, k1 = (k0 + 0x9E3779B9) & mask, (k1 + 0xBB67AE85) & mask
    return [((((hi << 21) | (lo >> 11)).double() + 0.5) / 2.0 ** 53) for hi, lo in ((c[0], c[1]), (c[2], c[3]))]


def _sample_exact(roots, masses, seed, n):
    nf = len(masses)
    ev = torch.arange(n, dtype=torch.int64, device="cuda")
    u = torch.stack([torch.stack(_philox(ev, 2 * i, seed) + _philox(ev, 2 * i + 1, seed), -1) for i in range(nf)], 1)
    out = _map_points(roots, masses, u)
    k = torch.sqrt((out[:, 2:, 1:] ** 2).sum(-1))
    en = out[:, 2:, 0]
    w = (2 * math.pi) ** (4 - 3 * nf) * (math.pi / 2) ** (nf - 1) * roots ** (2 * nf - 4) \
        / (math.factorial(nf - 1) * math.factorial(nf - 2))
    w = w * torch.ones_like(k[:, 0])
    if max(masses) > 0:
        w = w * (k.sum(1) / roots) ** (2 * nf - 3) * (k / en).prod(1) * roots / (k * k / en).sum(1)
    return out, w


def exact(case, seed):
    kind = case["kind"]
    if kind == "train":
        return _train_exact(case, seed)
    if kind == "sample":
        return _sample_exact(*KIN[case["process"]], int(seed) * 7919 + 3, case["events"])
    if kind == "unweight":  # which points are kept is decided in 16 bits
        return None
    mom = _points(case["process"], case["events"], seed)
    me2 = _me2(case["process"], mom)
    # a single diagram's share has no value without the library's list of diagrams
    return (me2, None) if kind == "channels" else me2
