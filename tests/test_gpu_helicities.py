"""Single helicities (me_eval_helicities) and the totals beside them (run on
an MI355X).

me_eval sums over real polarisation vectors, me_eval_helicities evaluates one
helicity after the other: the two share neither wavefunctions nor sums, so
that |M|^2 formed from the one checks the other.  Both are float64, so all
but the ill-conditioned events agree to 1e-12 and those to 1e-9.  Sizes on both sides
of the rule that spreads an event over lanes (fewer than half a turn of the chip,
65,536 lanes or, for five gluons, 16,384)."""
import math

import numpy as np
import pytest

from inputs import process_points, rambo

pytestmark = pytest.mark.gpu

# spins, colours and identical gluons: |M|^2 = sum of the helicities / this
AVERAGE = {"ee_mumu": 4, "gg_tt": 256, "gg_ttg": 256, "gg_ttgg": 512, "gg_ttggg": 1536,
           "gux_taptamux": 96, "gux_taptamgux": 96, "gux_taptamggux": 192}


@pytest.fixture(scope="module")
def env():
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2503_21935_amd as me

    me.lib()
    return torch, me


def close(got, want):
    rel = (got / want - 1).abs()
    assert bool(rel.isfinite().all()) and rel.max() <= 1e-9 and (rel > 1e-12).double().mean() <= 0.02, rel.max()


def tiled(torch, base, n):
    return torch.from_numpy(np.tile(base, (-(-n // len(base)), 1, 1))[:n].copy()).cuda()


@pytest.mark.parametrize("proc,n", [("ee_mumu", 1000), ("gg_tt", 1), ("gg_tt", 1000), ("gg_tt", 32769), ("gg_ttg", 65),
                                    ("gg_ttg", 70000), ("gg_ttgg", 1), ("gg_ttgg", 333), ("gg_ttgg", 32769),
                                    ("gg_ttggg", 3), ("gg_ttggg", 200), ("gg_ttggg", 8193), ("gux_taptamux", 1000),
                                    ("gux_taptamux", 32769), ("gux_taptamgux", 65), ("gux_taptamgux", 40000),
                                    ("gux_taptamggux", 1), ("gux_taptamggux", 1000), ("gux_taptamggux", 33000)])
def test_totals_are_the_sum_of_the_helicities(env, proc, n):
    torch, me = env
    print(f"[hel] {proc} n={n}", flush=True)
    mom = tiled(torch, process_points(proc, min(n, 1000), 91), n)
    m = me.MatrixElement(proc)
    me2 = torch.full((n + 64,), -7.0, dtype=torch.float64, device="cuda")
    nhel = m.info()["nhel"]
    qh = torch.full((n + 64, nhel), -7.0, dtype=torch.float64, device="cuda")
    me.me_eval_helicities(m.ctx, mom, n, me2, qh)
    assert bool((me2[n:] == -7.0).all()) and bool((qh[n:] == -7.0).all())
    me2, qh = me2[:n], qh[:n]
    sums = qh.sum(1) / AVERAGE[proc]
    close(me2, sums)
    close(m.eval(mom), sums)
    good = m.good_helicities()
    dropped = [h for h in range(nhel) if h not in good]
    assert (len(dropped) == 0) == (proc.startswith("gg"))
    if dropped:  # nothing but the rounding of amplitudes that cancel
        assert bool((qh[:, dropped].abs() <= 1e-24 * qh.amax(1, keepdim=True)).all())
    m.close()


@pytest.mark.parametrize("proc,few,many,mfma", [("gg_tt", 500, 33000, False), ("gg_ttg", 17, 33000, False),
                                                ("gg_ttgg", 3, 33000, False), ("gg_ttgg", 3, 33000, True),
                                                ("gg_ttggg", 5, 8200, False), ("gg_ttggg", 5, 8200, True),
                                                ("gux_taptamggux", 700, 33000, False)])
def test_lanes_give_the_same_helicities(env, proc, few, many, mfma):
    """Each helicity of an event at many lanes and at one: the same program,
    bit for bit (five gluons: to rounding, its waves add atomically)."""
    torch, me = env
    print(f"[hel] lanes {proc} mfma={mfma}", flush=True)
    base = process_points(proc, few, 92)
    m = me.MatrixElement(proc)
    if mfma:
        m.set_colour_form(me.ME_COLOUR_MFMA)
    a, qa = m.eval_helicities(torch.from_numpy(base).cuda())
    b, qb = m.eval_helicities(tiled(torch, base, many))
    qb, b = qb[:few], b[:few]
    if proc == "gg_ttggg":
        assert bool(((qa - qb).abs() <= 1e-12 * qb.amax(1, keepdim=True)).all())
    else:
        assert torch.equal(qa, qb)
    close(a, b)
    m.close()


@pytest.mark.parametrize("proc", ["gg_tt", "gg_ttg", "gg_ttgg", "gg_ttggg"])
def test_massless_top(env, proc):
    """The filter keeps the spin pairs of opposite helicity alone: me_eval sums
    over those, and the others contribute nothing."""
    torch, me = env
    nf = {"gg_tt": 2, "gg_ttg": 3, "gg_ttgg": 4, "gg_ttggg": 5}[proc]
    mom = torch.from_numpy(rambo(150 if nf < 5 else 12, 13000.0, [0.0] * nf, 93)).cuda()
    m = me.MatrixElement(proc, masses=(91.188, 2.4414, 0.0, 0.0))
    good = m.good_helicities()
    npart = nf + 2
    assert good and all((h >> (npart - 3)) & 1 != (h >> (npart - 4)) & 1 for h in good)
    me2, qh = m.eval_helicities(mom)
    dropped = [h for h in range(1 << npart) if h not in good]
    assert bool((qh[:, dropped].abs() <= 1e-24 * qh.amax(1, keepdim=True)).all())
    sums = qh[:, good].sum(1) / (256 * math.factorial(nf - 2))
    close(m.eval(mom), sums)
    close(me2, sums)
    m.close()
