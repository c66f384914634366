"""The spin-summed float64 kernels with shared wavefunctions (run on an MI355X).

Sizes at the edges of the grid (8192 waves, or 1024 workgroups, that stride over the events; partly
filled waves of several events), the
indexed form, and a massless top, where the helicity filter drops the spin
pairs that vanish.  Against the oracle, event by event: both sides work in
float64 with the same momenta, so all but the ill-conditioned events agree to
1e-12 and those to 1e-9 (the largest deviation of two float64 evaluations on
2^20 flat points is 1.3e-9, at the 99.9th percentile 6e-13)."""
import numpy as np
import pytest

import oracle
from inputs import process_points, rambo

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def env():
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2503_21935_amd as me

    me.lib()
    return torch, me


def close(got, want):
    rel = np.abs(got / want - 1)
    assert np.all(np.isfinite(got)) and rel.max() <= 1e-9 and np.mean(rel > 1e-12) <= 0.02, rel.max()


@pytest.mark.parametrize("proc,n", [("gg_tt", 1), ("gg_tt", 127), ("gg_ttg", 9), ("gg_ttg", 4103),
                                    ("gg_ttgg", 1), ("gg_ttgg", 2), ("gg_ttgg", 8191), ("gg_ttgg", 8193),
                                    ("gg_ttgg", 20000), ("gg_ttggg", 1), ("gg_ttggg", 255), ("gg_ttggg", 1025),
                                    ("gux_taptamux", 1), ("gux_taptamux", 33), ("gux_taptamgux", 15),
                                    ("gux_taptamgux", 4099), ("gux_taptamggux", 7), ("gux_taptamggux", 2049)])
def test_edges_of_the_grid(env, proc, n):
    torch, me = env
    print(f"[wave] {proc} n={n}", flush=True)
    mom = process_points(proc, n, 61)
    m = me.MatrixElement(proc)
    out = torch.full((n + 64,), -7.0, dtype=torch.float64, device="cuda")
    me.me_eval(m.ctx, torch.from_numpy(mom).cuda(), n, out)
    torch.cuda.synchronize()
    out = out.cpu().numpy()
    assert np.all(out[n:] == -7.0)
    k = 40 if proc != "gg_ttggg" else 6  # the oracle takes about a second per g g -> t tbar g g g event and core
    sel = np.unique(np.r_[np.arange(min(n, k)), np.arange(max(0, n - k), n)])
    close(out[sel], oracle.me2(proc, mom[sel]))
    m.close()


@pytest.mark.parametrize("proc,n", [("gg_tt", 1000), ("gg_ttg", 1001), ("gg_ttgg", 9000), ("gg_ttgg", 777), ("gg_ttggg", 300)])
def test_indexed_form(env, proc, n):
    """A tolerance no float32 result meets sends every event through the
    indexed form: the same values bit for bit."""
    torch, me = env
    m = me.MatrixElement(proc)
    t = torch.from_numpy(process_points(proc, n, 62)).cuda()
    ref = m.eval(t)
    m.set_precision(me.ME_MIXED, 1e-14)
    got = m.eval(t)
    assert m.fallback_count() == n
    assert torch.equal(got, ref)
    m.close()


@pytest.mark.parametrize("proc", ["gg_tt", "gg_ttg", "gg_ttgg", "gg_ttggg"])
def test_massless_top(env, proc):
    torch, me = env
    nf = {"gg_tt": 2, "gg_ttg": 3, "gg_ttgg": 4, "gg_ttggg": 5}[proc]
    mom = rambo(200 if nf < 5 else 12, 13000.0, [0.0] * nf, 63)
    m = me.MatrixElement(proc, masses=(91.188, 2.4414, 0.0, 0.0))
    assert len(m.good_helicities()) < 1 << (nf + 2)
    got = m.eval(torch.from_numpy(mom).cuda()).cpu().numpy()
    close(got, oracle.me2(proc, mom, params=oracle.sm_params(mt=0.0, wt=0.0)))
    m.close()


def test_five_gluons_are_deterministic(env):
    """No sums with atomics: the same input twice gives the same bits."""
    torch, me = env
    m = me.MatrixElement("gg_ttggg")
    t = torch.from_numpy(process_points("gg_ttggg", 700, 64)).cuda()
    assert torch.equal(m.eval(t), m.eval(t))
    m.close()


@pytest.mark.parametrize("proc,n", [("gg_tt", 1), ("gg_tt", 65), ("gg_ttg", 1), ("gg_ttg", 9), ("gg_ttgg", 1),
                                    ("gg_ttgg", 2), ("gg_ttgg", 4097), ("gg_ttgg", 16387)])
def test_channel_weights_at_the_edges_of_the_grid(env, proc, n):
    """Every event in another channel; nothing written past the end.  Weights
    to 1e-10 relative, as ratios of sums of squares of the amplitudes."""
    torch, me = env
    print(f"[wave] channels {proc} n={n}", flush=True)
    mom = process_points(proc, n, 62)
    m = me.MatrixElement(proc)
    descs = m.channels()
    chan = np.random.default_rng(62).integers(0, len(descs), n).astype(np.int32)
    me2, alpha = (torch.full((n + 64,), -7.0, dtype=torch.float64, device="cuda") for _ in range(2))
    me.me_eval_multichannel(m.ctx, torch.from_numpy(mom).cuda(), torch.from_numpy(chan).cuda(), n, me2, alpha)
    torch.cuda.synchronize()
    me2, alpha = me2.cpu().numpy(), alpha.cpu().numpy()
    assert np.all(me2[n:] == -7.0) and np.all(alpha[n:] == -7.0)
    sel = np.unique(np.r_[np.arange(min(n, 40)), np.arange(max(0, n - 40), n)])
    odescs, sums = oracle.diagram_sums(proc, mom[sel])
    col = np.array([odescs.index(d) for d in descs])
    want = (sums / sums.sum(axis=1, keepdims=True))[np.arange(len(sel)), col[chan[sel]]]
    assert np.all(np.abs(alpha[sel] / want - 1) <= 1e-10)
    close(me2[sel], oracle.me2(proc, mom[sel]))
    m.close()


def test_channel_weights_with_helicities_dropped(env):
    """A massless top: the filter drops helicities whose |M|^2 vanishes though
    single diagrams do not; the weights are those over the kept ones and add up to 1."""
    torch, me = env
    m = me.MatrixElement("gg_ttg", masses=(91.188, 2.4414, 0.0, 0.0))
    assert len(m.good_helicities()) < 32
    mom = torch.from_numpy(rambo(300, 1500.0, [0.0] * 3, 63)).cuda()
    total = 0
    for c in range(len(m.channels())):
        total = total + m.eval_multichannel(mom, torch.full((300,), c, dtype=torch.int32, device="cuda"))[1]
    np.testing.assert_allclose(total.cpu().numpy(), 1.0, rtol=1e-12)
    m.close()


@pytest.mark.parametrize("proc,n", [("gg_tt", 1), ("gg_ttg", 1000), ("gg_ttgg", 1), ("gg_ttgg", 65), ("gg_ttgg", 4097),
                                    ("gg_ttgg", 66000)])
def test_mixed_form_with_its_helicities_parted(env, proc, n):
    """The parted form adds the same float32 values in the same order as one lane
    does: unflagged events bit for bit as the diagnostic call, which never parts
    them, gives, and the same number flagged."""
    torch, me = env
    print(f"[wave] parted {proc} n={n}", flush=True)
    base = process_points(proc, min(n, 3000), 65, precise=False)
    mom = torch.from_numpy(np.tile(base, (-(-n // len(base)), 1, 1))[:n].copy()).cuda()
    m = me.MatrixElement(proc)
    m.set_precision(me.ME_MIXED, 1e-5)
    raw, _, flag = m.eval_mixed_diag(mom)
    got = m.eval(mom)
    assert m.fallback_count() == int(flag.sum())
    keep = flag == 0
    assert torch.equal(got[keep], raw[keep])
    assert torch.equal(m.eval(mom), got)
    m.close()


@pytest.mark.parametrize("proc,n", [("gg_ttgg", 4097), ("gg_ttgg", 8193), ("gg_ttgg", 20000), ("gg_ttggg", 1025),
                                    ("gg_ttggg", 2050)])
def test_matrix_core_colour_sum_of_many_events(env, proc, n):
    """Blocks with two events set up together, blocks that stride over the events, and
    the staging of J used again behind the next event's preparation.  61 points over and
    over: every copy has the bits of the first, in whichever slot of a block; the two
    colour forms agree as two float64 evaluations do."""
    torch, me = env
    print(f"[wave] colour {proc} n={n}", flush=True)
    pts = process_points(proc, 61, 67)
    mom = torch.from_numpy(np.tile(pts, (-(-n // 61), 1, 1))[:n].copy()).cuda()
    m = me.MatrixElement(proc)
    got = {}
    for form in (me.ME_COLOUR_VALU, me.ME_COLOUR_MFMA):
        m.set_colour_form(form)
        out = torch.full((n + 64,), -7.0, dtype=torch.float64, device="cuda")
        me.me_eval(m.ctx, mom, n, out)
        assert bool((out[n:] == -7.0).all())
        first = out[:61]
        assert all(torch.equal(out[k:min(k + 61, n)], first[:min(61, n - k)]) for k in range(0, n, 61))
        got[form] = first.cpu().numpy()
    close(got[me.ME_COLOUR_MFMA], got[me.ME_COLOUR_VALU])
    close(got[me.ME_COLOUR_MFMA][:4], oracle.me2(proc, pts[:4]))
    m.close()


@pytest.mark.parametrize("proc,n", [("gg_tt", 300), ("gg_ttg", 300), ("gg_ttgg", 300), ("gg_ttggg", 60),
                                    ("gux_taptamux", 300), ("gux_taptamgux", 300), ("gux_taptamggux", 300)])
def test_lanes_setting_changes_nothing(env, proc, n):
    """Accepted for every process, in effect for e+ e- -> mu+ mu- alone."""
    torch, me = env
    m = me.MatrixElement(proc)
    mom = torch.from_numpy(process_points(proc, n, 68)).cuda()
    want = m.eval(mom)
    for lanes in (1, 4, 64, 0):
        m.set_helicity_lanes(lanes)
        assert torch.equal(m.eval(mom), want)
    m.close()


@pytest.mark.parametrize("proc,n", [("gg_tt", n) for n in (1, 15, 16, 17, 1000, 16383, 16384, 16385)]
                         + [("gg_ttg", n) for n in (1, 2, 3, 1000, 2047, 2048, 2049)])
def test_spin_pairs_on_lanes_and_in_turn(env, proc, n):
    """g g -> t tbar and g g -> t tbar g: calls of up to 16,384 and 2,048 events give each
    spin pair lanes of its own; the same bits as all pairs in turn, also through a list."""
    torch, me = env
    nf = {"gg_tt": 2, "gg_ttg": 3}[proc]
    pts = process_points(proc, 97, 69)
    mom = torch.from_numpy(np.tile(pts, (207, 1, 1))[:20000].copy()).cuda()
    m = me.MatrixElement(proc)
    want = m.eval(mom)
    close(want[:97].cpu().numpy(), oracle.me2(proc, pts))
    out = torch.full((n + 64,), -7.0, dtype=torch.float64, device="cuda")
    me.me_eval(m.ctx, mom, n, out)
    assert torch.equal(out[:n], want[:n]) and bool((out[n:] == -7.0).all())
    m.set_precision(me.ME_MIXED, 1e-14)
    assert torch.equal(m.eval(mom[:n]), want[:n]) and m.fallback_count() == n
    m.close()
    m = me.MatrixElement(proc, masses=(91.188, 2.4414, 0.0, 0.0))
    mom = torch.from_numpy(np.tile(rambo(97, 13000.0, [0.0] * nf, 63), (207, 1, 1))[:20000].copy()).cuda()
    assert torch.equal(m.eval(mom[:n]), m.eval(mom)[:n])
    m.close()
