"""What the mixed form keeps in a context, and when (run on an MI355X)."""
import pytest

from inputs import process_points

pytestmark = pytest.mark.gpu

BIG = 300000  # more events than the mixed form parts over blocks


@pytest.fixture(scope="module")
def env():
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import numpy as np

    import paper_2503_21935_amd as me

    me.lib()
    base = process_points("gg_ttgg", 1000, 95, precise=False)
    return torch, me, torch.from_numpy(np.tile(base, (BIG // 1000, 1, 1))).cuda()


def mixed(me):
    m = me.MatrixElement("gg_ttgg")
    m.set_precision(me.ME_MIXED, 1e-5)
    return m


def free(torch):
    torch.cuda.synchronize()
    return torch.cuda.mem_get_info()[0]


def test_calls_too_large_to_be_parted_keep_the_index_list_alone(env):
    torch, me, mom = env
    out = torch.empty(BIG, dtype=torch.float64, device="cuda")
    small = torch.empty(100, dtype=torch.float64, device="cuda")
    m = mixed(me)
    m.eval_mixed_diag(mom[:64])  # the kernels are loaded
    me.me_eval(m.ctx, mom, 64, out)
    m.close()
    m = mixed(me)
    before = free(torch)
    me.me_eval(m.ctx, mom, BIG, out)
    kept = free(torch)
    assert before - kept < 16 << 20  # four bytes an event
    me.me_eval(m.ctx, mom, 100, small)  # parted: its room comes now
    assert 64 << 20 < kept - free(torch) < 160 << 20
    assert torch.equal(small, out[:100])
    m.close()


def test_first_parted_call_under_capture(env):
    """A context whose index list is long enough: the call may come in a capture,
    and the graph stays valid through later calls of any size up to the list's."""
    torch, me, mom = env
    m = mixed(me)
    ref = m.eval(mom)[:3000].clone()
    n = 3000
    out = torch.empty(n, dtype=torch.float64, device="cuda")
    torch.cuda.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        me.me_eval(m.ctx, mom, n, out)
    for other in (64, 70000, BIG):
        out.fill_(-1.0)
        g.replay()
        torch.cuda.synchronize()
        assert torch.equal(out, ref)
        assert torch.equal(m.eval(mom[:other])[:64], ref[:64])
        torch.cuda.synchronize()
    del g
    m.close()


def test_two_contexts_on_two_streams(env):
    """Overlapping parted calls, each on a context of its own."""
    torch, me, mom = env
    a, b = mixed(me), mixed(me)
    want_a, want_b = a.eval(mom[:20000]), b.eval(mom[500:9000])
    streams = torch.cuda.Stream(), torch.cuda.Stream()
    outs = [(torch.empty_like(want_a), torch.empty_like(want_b)) for _ in range(4)]
    torch.cuda.synchronize()
    for oa, ob in outs:
        a.eval(mom[:20000], oa, stream=streams[0])
        b.eval(mom[500:9000], ob, stream=streams[1])
    torch.cuda.synchronize()
    assert all(torch.equal(oa, want_a) and torch.equal(ob, want_b) for oa, ob in outs)
    a.close(), b.close()
