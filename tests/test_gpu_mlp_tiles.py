"""GPU tests of the network kernels (mlp.hip) at the edges of their tiles, through the C-ABI.

* Forward: a row's output does not depend on the call it is in, so calls long enough for the kernel that
  keeps the weights in LDS (with a ragged end) give, bit for bit, what short calls give row by row.
* Gradient: in FP32 mode loss and gradient equal a float64 network's at sizes around the kernels' 16-, 64-
  and 128-row tiles. Sums of n FP32 products err by at most n 2^-24 of the sum of their sizes, and the
  errors of a layer pass through the next ones; the bar is 1e-4 of each parameter block's norm.
"""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")
lib_mod = pytest.importorskip("paper_2001_04890_amd")

if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

DEV = torch.device("cuda:0")


def network(seed):
    r = np.random.default_rng(seed)
    return [r.uniform(-1, 1, s).astype(np.float32) * np.float32(f) for s, f in
            (((16, 256), 0.6), ((256,), 0.05), ((256, 256), 0.15), ((256,), 0.05), ((256,), 0.02), ((1,), 0.01))]


def make(seed):
    parts = network(seed)
    net = lib_mod.Mlp(0, seed=1)
    net.set_params(np.concatenate([p.ravel() for p in parts]))
    return net, [torch.as_tensor(p, device=DEV).double() for p in parts]


@pytest.mark.parametrize("n", [18001, 32768, 65541, 131072 + 77])
def test_forward_rows_do_not_depend_on_the_call(n):
    net, _ = make(3)
    feat = torch.randn(n, 16, device=DEV, generator=torch.Generator(DEV).manual_seed(n))
    out = torch.empty(n, device=DEV)
    net.forward(feat, out)
    for a, b in ((0, 1), (0, 4099), (n - 65, n), (n // 2 - 8, n // 2 + 9)):
        part = torch.empty(b - a, device=DEV)
        net.forward(feat[a:b].contiguous(), part)
        assert torch.equal(part, out[a:b]), (a, b)


@pytest.mark.parametrize("n", [1, 3, 15, 17, 63, 65, 127, 128, 129, 513, 1000])
def test_gradient_at_tile_edges(n):
    net, (w1, b1, w2, b2, w3, b3) = make(5)
    net.set_fp32(True)
    gen = torch.Generator(DEV).manual_seed(n)
    feat, pairs = torch.randn(n, 16, device=DEV, generator=gen), torch.randn(n, 3, device=DEV, generator=gen)
    grad, loss = torch.full((lib_mod.MLP_PARAMS,), float("nan"), device=DEV), torch.empty(1, device=DEV)
    net.grad(feat, pairs, grad, loss)
    f, (a, b, w) = feat.double(), pairs.double().unbind(1)
    h1 = torch.relu(f @ w1 + b1)
    h2 = torch.relu(h1 @ w2 + b2)
    e = a * (1 + h2 @ w3 + b3) - b
    g = 2 * w * a * e / n
    d2 = g[:, None] * w3 * (h2 > 0)
    d1 = (d2 @ w2.T) * (h1 > 0)
    at = 0
    for ref in (f.T @ d1, d1.sum(0), h1.T @ d2, d2.sum(0), h2.T @ g, g.sum()[None]):
        got = grad[at:at + ref.numel()].double().view(ref.shape)
        at += ref.numel()
        assert (got - ref).norm() <= 1e-4 * max(float(ref.norm()), 1e-30)
    assert abs(float(loss) - float((w * e * e).mean())) <= 1e-4 * float((w * e * e).abs().mean())
