"""GPU: the training gradient and the BF16 inference at the edges of their row
tiles and splits."""
import numpy as np
import pytest

import gwsynth

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


@pytest.fixture(scope="module")
def net():
    if not torch.cuda.is_available():
        pytest.skip("no GPU visible")
    import paper_2607_28265_amd as gw
    prob = gwsynth.make_problem(4.0, 20.0, 256.0, psd_scale=1e-47)
    with gw.Context(prob) as ctx:
        m = gw.Mlp(ctx, seed=7)
        m.set_scaling(np.full(11, 0.4), np.linspace(0.2, 0.4, 11), -30.0, 12.0)
        yield m
        m.close()


def _exact(m, x, y):
    """Gradient and loss in FP64."""
    p, at, layers = m.get_params().astype(np.float64), 0, []
    for k, j in ((11, 256), (256, 256), (256, 256), (256, 1)):
        w = torch.from_numpy(p[at:at + k * j].reshape(k, j)).requires_grad_()
        b = torch.from_numpy(p[at + k * j:at + k * j + j]).requires_grad_()
        at += k * j + j
        layers.append((w, b))
    a = (torch.from_numpy(x) - 0.4) / torch.linspace(0.2, 0.4, 11, dtype=torch.float64)
    for i, (w, b) in enumerate(layers):
        a = a @ w + b
        if i < 3:
            a = torch.nn.functional.gelu(a)
    loss = ((a[:, 0] - (torch.from_numpy(y) + 30.0) / 12.0) ** 2).mean()
    loss.backward()
    return np.concatenate([np.concatenate([w.grad.numpy().ravel(), b.grad.numpy()]) for w, b in layers]), float(loss.detach())


@pytest.mark.parametrize("n", [1, 3, 5, 127, 128, 129, 1023, 1025, 4096, 4097, 4111, 9000])
def test_gradient_at_row_tile_edges(net, n):
    rng = np.random.default_rng(n)
    x, y = rng.random((n, 11)), -30.0 + 12.0 * rng.standard_normal(n)
    g, loss = net.grad(torch.from_numpy(x).cuda(), torch.from_numpy(y).cuda())
    g = np.asarray(g, dtype=np.float64)
    ref, lref = _exact(net, x, y)
    # FP32 rounding of six products of 256 terms: 6 sqrt(256) eps / 2 of the scale
    assert np.max(np.abs(g - ref)) < 6e-6 * np.max(np.abs(ref))
    assert abs(float(np.asarray(loss).reshape(-1)[0]) - lref) < 6e-6 * lref


def test_inference_rows_independent_of_launch(net):
    x = torch.from_numpy(np.random.default_rng(1).random((16400, 11))).cuda()
    whole = net.forward(x).clone()
    for n in (1, 31, 33, 64, 8192, 8193, 16384, 16385):
        assert torch.equal(net.forward(x[:n].contiguous()), whole[:n])
