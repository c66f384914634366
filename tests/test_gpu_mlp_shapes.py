"""The one-kernel training step and inference at every depth, and at batches that
give a block several tiles (run on an MI355X).

The kernels are templates of the depth whose buffers alternate with its parity;
they are compared with a float64 reference that rounds to BF16 where they do.
Bounds as for the default network: an output within 2^-6 of the sum of the
magnitudes of its terms in the output layer, a gradient entry within 2^-5 of the sum
of the magnitudes of its terms over the batch (a flipped rounding of an activation moves
it by at most 2^-8 of itself; a wrong row, column or buffer by O(1))."""
import numpy as np
import pytest

from oracle import mlp_ref as R

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def env():
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2503_21935_amd as me

    me.lib()
    return torch, me


def forward(theta, x, n_in, width, depth):
    layers, w_out, b_out = R.unpack(theta, n_in, width, depth)
    zs, hs = [], [R.bf16_round(x)]
    for W, b in layers:
        zs.append(hs[-1] @ R.bf16_round(W).T + b)
        hs.append(R.bf16_round(R.silu(zs[-1])))
    return hs[-1] @ w_out + b_out[0], zs, hs, layers, w_out, b_out[0]


def gradient(theta, x, t, n_in, depth):
    """(gradient, sums of the magnitudes behind it, loss)"""
    y, zs, hs, layers, w_out, _ = forward(theta, x, n_in, 256, depth)
    dy = 2 * (y - t) / len(t)
    g, a = [dy.sum()[None], hs[-1].T @ dy], [np.abs(dy).sum()[None], np.abs(hs[-1]).T @ np.abs(dy)]
    dz = R.bf16_round(np.outer(dy, w_out) * R.silu_prime(zs[-1]))
    for l in range(depth - 1, -1, -1):
        g += [dz.sum(0), (dz.T @ hs[l]).ravel()]
        a += [np.abs(dz).sum(0), (np.abs(dz).T @ np.abs(hs[l])).ravel()]
        if l:
            dz = R.bf16_round((dz @ R.bf16_round(layers[l][0])) * R.silu_prime(zs[l - 1]))
    return np.concatenate(g[::-1]), np.concatenate(a[::-1]), np.mean((y - t) ** 2)


def data(torch, n, n_in, seed):
    rng = np.random.default_rng(seed)
    x = (rng.normal(size=(n, n_in)) * 0.5).astype(np.float32)
    t = rng.normal(size=n).astype(np.float32)
    return x, t, torch.from_numpy(x).cuda(), torch.from_numpy(t).cuda()


# 16 rows a tile, a tile per CU at 4096 rows: one block in two without one, one each, some with two, all with two
@pytest.mark.parametrize("depth", [1, 2, 3, 4])
@pytest.mark.parametrize("n,n_in", [(128, 24), (2048, 5), (4224, 32), (8192, 24)])
def test_gradient_at_every_depth(env, depth, n, n_in):
    torch, me = env
    print(f"[mlp] gradient depth={depth} n={n} n_in={n_in}", flush=True)
    net = me.Surrogate(n_in, 256, depth, seed=31 + depth)
    x, t, xd, td = data(torch, n, n_in, 7)
    g, loss = net.backward(xd, td)
    want, mag, lref = gradient(net.get_params().astype(np.float64), x.astype(np.float64), t.astype(np.float64), n_in,
                               depth)
    g = g.cpu().numpy().astype(np.float64)
    ratio = np.abs(g - want) / np.maximum(mag, 1e-30)
    assert ratio.max() < 2.0 ** -5, (int(ratio.argmax()), ratio.max())
    assert abs(loss.item() / lref - 1) < 1e-2
    net.close()


@pytest.mark.parametrize("depth", [1, 2, 3, 4])
@pytest.mark.parametrize("n,n_in,listed", [(128, 24, True), (4224, 24, False), (8192, 5, True)])
def test_steps_in_one_launch_at_every_depth(env, depth, n, n_in, listed):
    """Against one launch per step: the same sums, the bias corrections on the
    device instead of the host."""
    torch, me = env
    print(f"[mlp] steps depth={depth} n={n} n_in={n_in}", flush=True)
    _, _, x, t = data(torch, 4 * n, n_in, 8)
    lrs = [1e-3, 8e-4, 6e-4, 3e-4]
    idx = None
    if listed:
        idx = torch.from_numpy(np.random.default_rng(9).permutation(4 * n).astype(np.int32)).cuda()
    a, b = me.Surrogate(n_in, 256, depth, seed=41), me.Surrogate(n_in, 256, depth, seed=41)
    la, lb = (torch.zeros(4, dtype=torch.float32, device="cuda") for _ in range(2))
    a.train_steps(x, t, idx, n, torch.tensor(lrs, dtype=torch.float32, device="cuda"), la)
    for s, lr in enumerate(lrs):
        rows = slice(s * n, (s + 1) * n)
        if listed:
            b.train_step(x, t, idx[rows], lr, lb[s:s + 1])
        else:
            b.train_step(x[rows], t[rows], None, lr, lb[s:s + 1])
    torch.cuda.synchronize()
    np.testing.assert_allclose(la.cpu().numpy(), lb.cpu().numpy(), rtol=1e-5)
    assert np.abs(a.get_params().astype(np.float64) - b.get_params()).max() <= 1e-6
    # the copies that other kernels read have followed: the layered gradient and the inference
    y = a.forward(x[:200]).cpu().numpy().astype(np.float64)
    want, _, hs, _, w_out, b_out = forward(a.get_params().astype(np.float64), x[:200].cpu().numpy().astype(np.float64),
                                           n_in, 256, depth)
    assert (np.abs(y - want) / (np.abs(hs[-1]) @ np.abs(w_out) + abs(b_out))).max() < 2.0 ** -6
    gf, _ = a.backward(x[:n], t[:n])
    a.set_fused_step(False)
    gl, _ = a.backward(x[:n], t[:n])
    _, mag, _ = gradient(a.get_params().astype(np.float64), x[:n].cpu().numpy().astype(np.float64),
                         t[:n].cpu().numpy().astype(np.float64), n_in, depth)
    assert (np.abs((gf - gl).cpu().numpy()) / np.maximum(mag, 1e-30)).max() < 2.0 ** -5
    a.close(), b.close()


# weights in fragment order (depth to 4), row by row (5 to 8), and the layered kernels
@pytest.mark.parametrize("width,depth", [(256, 1), (256, 2), (256, 4), (256, 5), (256, 8), (256, 9), (128, 3)])
@pytest.mark.parametrize("n,n_in", [(1, 24), (127, 5), (129, 32), (3000, 16)])
def test_forward_of_every_form(env, width, depth, n, n_in):
    torch, me = env
    net = me.Surrogate(n_in, width, depth, seed=51)
    x, _, xd, _ = data(torch, n, n_in, 10)
    out = torch.full((n + 64,), -7.0, dtype=torch.float32, device="cuda")
    me.mlp_forward(net.h, xd, n, out)
    y = out.cpu().numpy().astype(np.float64)
    assert np.all(y[n:] == -7.0)
    want, _, hs, _, w_out, b_out = forward(net.get_params().astype(np.float64), x.astype(np.float64), n_in, width, depth)
    scale = np.abs(hs[-1]) @ np.abs(w_out) + abs(b_out)
    assert (np.abs(y[:n] - want) / scale).max() < 2.0 ** -6
    net.close()
