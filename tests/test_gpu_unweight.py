"""Two-stage unweighting: every form of the network's first stage and of the
exact second one (run on an MI355X)."""
import numpy as np
import pytest

from inputs import process_points, uniforms

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def env():
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2503_21935_amd as me

    me.lib()
    return torch, me


class Sample:
    """n points of a process with thresholds that about a third passes at either stage."""

    def __init__(self, torch, me, proc, n, seed):
        mom, w = process_points(proc, n, seed, return_weight=True)
        self.torch, self.me, self.n = torch, me, n
        self.mom, self.w = torch.from_numpy(mom).cuda(), torch.from_numpy(w).cuda()
        self.u = torch.from_numpy(uniforms(n, 2, seed)).cuda()
        self.idx = torch.empty(n, dtype=torch.int32, device="cuda")
        self.out = torch.empty(n, dtype=torch.float64, device="cuda")
        self.count = torch.zeros(2, dtype=torch.int32, device="cuda")

    def thresholds(self, m, net):
        s = net.forward(self.me.features(self.mom)).double().exp() * self.w
        self.s, self.r = s, m.eval(self.mom) * self.w / s
        self.s_max, self.r_max = float(s.quantile(0.9)), float(self.r.quantile(0.9))

    def run(self, m, net):
        self.me.unweight_two_stage(m.ctx, net.h, self.mom, self.w, self.n, self.u, 0.0, 1.0, self.s_max, self.r_max,
                                   self.idx, self.out, self.count)

    def result(self):
        """(survivors, accepted indices in order, their weights)"""
        self.torch.cuda.synchronize()
        first, k = self.count.tolist()
        order = self.idx[:k].argsort()
        return first, self.idx[:k][order].cpu().numpy(), self.out[:k][order].cpu().numpy()


def test_another_network_under_capture(env):
    """Scratch of a context that has seen a call of this size suffices for any
    network: a layered one, itself warm, after one with a kernel of its own."""
    torch, me = env
    s = Sample(torch, me, "gg_tt", 3000, 81)
    m, one, layered = me.MatrixElement("gg_tt"), me.Surrogate(16, 256, 2, 5), me.Surrogate(16, 128, 2, 6)
    s.thresholds(m, one)
    s.run(m, one)
    s.thresholds(m, layered)  # runs its forward pass
    torch.cuda.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        s.run(m, layered)
    got = []
    for _ in range(3):
        s.count.fill_(-1)
        g.replay()
        got.append(s.result())
        torch.cuda.synchronize()
    s.run(m, layered)
    want = s.result()
    assert 0 < len(want[1]) < want[0] < s.n
    for r in got:
        assert r[0] == want[0] and np.array_equal(r[1], want[1]) and np.array_equal(r[2], want[2])
    del g
    m.close(), one.close(), layered.close()


@pytest.mark.parametrize("proc,n", [("ee_mumu", 1500), ("gg_tt", 3001), ("gg_ttg", 3001), ("gg_ttgg", 2049),
                                    ("gg_ttggg", 500), ("gux_taptamux", 3001), ("gux_taptamgux", 1025),
                                    ("gux_taptamggux", 2000)])
@pytest.mark.parametrize("width,depth", [(256, 4), (256, 6), (128, 2)])
def test_every_process_and_form_of_network(env, proc, n, width, depth):
    """Survivors (a part of the points, so that the exact weights go through a list) and
    their weights, from the network's outputs on the features and me_eval's |M|^2.
    The network gives the same bits from momenta as from features, and the exact
    kernels from a list as from all points; exponential and products may differ by
    rounding, so the weights agree to 1e-12 and no decision lies within 1e-12 of its bound."""
    torch, me = env
    print(f"[uw] {proc} width={width} depth={depth}", flush=True)
    s = Sample(torch, me, proc, n, 83)
    m, net = me.MatrixElement(proc), me.Surrogate(s.mom.shape[1] * 4, width, depth, 7)
    s.thresholds(m, net)
    s.run(m, net)
    first, idx, wt = s.result()
    p1, p2 = (s.s / s.s_max).clamp(max=1.0), (s.r / s.r_max).clamp(max=1.0)
    assert not bool((((s.u[:, 0] / p1 - 1).abs() < 1e-12) | ((s.u[:, 1] / p2 - 1).abs() < 1e-12)).any())
    one = s.u[:, 0] < p1
    both = (one & (s.u[:, 1] < p2)).nonzero()[:, 0]
    assert 0 < len(both) < first < n
    assert first == int(one.sum()) and np.array_equal(idx, both.cpu().numpy())
    want = (s.s / s.s_max).clamp(min=1.0) * (s.r / s.r_max).clamp(min=1.0)
    np.testing.assert_allclose(wt, want[both].cpu().numpy(), rtol=1e-12)
    m.close(), net.close()
