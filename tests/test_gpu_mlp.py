"""BF16-MFMA corrector network kernels against the FP64 reference MLP:
forward outputs, loss and gradients within BF16 tolerance, and training."""
import numpy as np
import pytest

from oracle import mlp as omlp
from tests.gpu_util import say

pytestmark = pytest.mark.gpu

WIDTHS = [1120, 256, 256, 256, 160]


def _net(B, seed=3):
    import torch
    from paper_1607_05535_amd import thor
    net = thor.MLP(WIDTHS, B, seed=seed)
    rs = np.random.default_rng(seed)
    x32 = rs.normal(size=(B, WIDTHS[0])).astype(np.float32)
    x = torch.from_numpy(x32).to("cuda:0").to(torch.bfloat16)
    xr = x.float().cpu().numpy().astype(np.float64)   # what the kernels see
    t32 = (0.5 * rs.normal(size=(B, WIDTHS[-1]))).astype(np.float32)
    t = torch.from_numpy(t32).to("cuda:0")
    return net, x, xr, t, t32.astype(np.float64)


def _ref_params(net):
    return [(W.astype(np.float64), b.astype(np.float64)) for W, b in net.unpack(net.get_params())]


def test_forward_matches_reference():
    import torch
    B = 100    # ragged against the 64-row GEMM tiles and the 48-row fused tiles
    say(f"[mlp] forward widths={WIDTHS} B={B}")
    net, x, xr, t, tr = _net(B)
    y = torch.empty(B, WIDTHS[-1], dtype=torch.float32, device="cuda:0")
    net.forward(x, y)
    got = y.cpu().numpy().astype(np.float64)
    ref, _ = omlp.forward(_ref_params(net), xr)
    rel = np.linalg.norm(got - ref) / np.linalg.norm(ref)
    say(f"      forward rel err {rel:.3e}")
    assert rel < 2e-2


@pytest.mark.parametrize("B", [1, 100, 10242])
def test_fused_inference_equals_layer_by_layer(B):
    """The fused 4-layer inference kernel (one workgroup per 48-row tile,
    inputs and hidden activations in LDS, weights in fragment order) against
    the layer-by-layer GEMMs: the same products in the same order, so the
    same outputs, at a single row, a ragged tile and the g5 corrector's
    10242 columns."""
    import torch
    net, x, xr, t, tr = _net(B, seed=7)
    y1 = torch.empty(B, WIDTHS[-1], dtype=torch.float32, device="cuda:0")
    y2 = torch.empty_like(y1)
    net.set_fused(False)
    net.forward(x, y1)
    net.set_fused(True)
    net.forward(x, y2)
    net.set_fused(False)
    a, b = y1.cpu().numpy(), y2.cpu().numpy()
    say(f"[mlp] fused vs layered B={B}: max |diff| {np.abs(a - b).max():.3e}, bitwise {np.array_equal(a, b)}")
    assert np.abs(a - b).max() <= 1e-6 * np.abs(a).max()


def test_gradients_match_reference():
    B = 128
    net, x, xr, t, tr = _net(B, seed=5)
    loss, g = net.loss_grad(x, t)
    params = _ref_params(net)
    ref_loss = omlp.loss(params, xr, tr)
    assert abs(loss / ref_loss - 1) < 2e-2
    ref = omlp.backward(params, xr, tr)
    got = net.unpack(g.astype(np.float64))
    for li, ((gW, gb), (rW, rb)) in enumerate(zip(got, ref)):
        for name, a, r in (("W", gW, rW), ("b", gb, rb)):
            rel = np.linalg.norm(a - r) / np.linalg.norm(r)
            cos = float(np.sum(a * r) / (np.linalg.norm(a) * np.linalg.norm(r)))
            say(f"      layer {li} d{name}: rel {rel:.3e} cos {cos:.6f}")
            assert rel < 2e-2 and cos > 0.999, (li, name, rel, cos)


def test_training_reduces_loss():
    B = 256
    net, x, xr, t, tr = _net(B, seed=7)
    l0, _ = net.loss_grad(x, t, want_grad=False)
    for _ in range(200):
        net.train_step(x, t, 1e-3)
    l1, _ = net.loss_grad(x, t, want_grad=False)
    say(f"      loss {l0:.4f} -> {l1:.4f}")
    assert l1 < 0.1 * l0


def test_argument_errors():
    from paper_1607_05535_amd import thor
    net, x, xr, t, tr = _net(64)
    with pytest.raises(thor.ThorError):
        net.loss_grad(x[:40], t[:40])          # batch not a multiple of 32
    with pytest.raises(thor.ThorError):
        thor.MLP([100, 64], 32)                # width not a multiple of 32


def test_split_batch_gradients_match_reference_and_repeat_bitwise():
    """A batch of 2048 rows reduces the weight gradients over 8 chunks and
    the bias gradients over 32: still the reference gradients, and the same
    bits on a second call (fixed summation order)."""
    import torch
    B = 2048
    net, x, xr, t, tr = _net(B, seed=9)
    loss, g = net.loss_grad(x, t)
    loss2, g2 = net.loss_grad(x, t)
    assert loss == loss2 and np.array_equal(g, g2)
    params = _ref_params(net)
    ref = omlp.backward(params, xr, tr)
    got = net.unpack(g.astype(np.float64))
    for li, ((gW, gb), (rW, rb)) in enumerate(zip(got, ref)):
        for name, a, r in (("W", gW, rW), ("b", gb, rb)):
            rel = np.linalg.norm(a - r) / np.linalg.norm(r)
            cos = float(np.sum(a * r) / (np.linalg.norm(a) * np.linalg.norm(r)))
            assert rel < 2e-2 and cos > 0.999, (li, name, rel, cos)
    # the inference path (no stored pre-activations) gives the same outputs
    y = torch.empty(B, WIDTHS[-1], dtype=torch.float32, device="cuda:0")
    net.forward(x, y)
    d = y.cpu().numpy().astype(np.float64) - tr
    assert abs(np.mean(d * d) / loss - 1) < 1e-6


@pytest.mark.parametrize("widths,B", [([32, 32], 32), ([96, 160, 32], 96), ([64, 256, 96, 160], 1056),
                                      ([1120, 256, 256, 256, 160], 320)])
def test_gradients_and_adam_at_ragged_tiles(widths, B):
    """Batches and widths that leave part of the 64 x 64 tiles over, one layer
    to four: gradients against the reference, one Adam step against the same
    formula in FP32 on the returned gradient, and the two inference paths on
    the updated weights against each other."""
    import torch
    from paper_1607_05535_amd import thor
    net = thor.MLP(widths, B, seed=2)
    rs = np.random.default_rng(4)
    x = torch.from_numpy(rs.normal(size=(B, widths[0])).astype(np.float32)).to("cuda:0").to(torch.bfloat16)
    t32 = rs.normal(size=(B, widths[-1])).astype(np.float32)
    t = torch.from_numpy(t32).to("cuda:0")
    p0 = net.get_params()
    loss, g = net.loss_grad(x, t)
    params, xr = _ref_params(net), x.float().cpu().numpy().astype(np.float64)
    assert abs(loss / omlp.loss(params, xr, t32.astype(np.float64)) - 1) < 2e-2
    for (gW, gb), (rW, rb) in zip(net.unpack(g.astype(np.float64)),
                                  omlp.backward(params, xr, t32.astype(np.float64))):
        for a, r in ((gW, rW), (gb, rb)):
            assert np.linalg.norm(a - r) < 2e-2 * np.linalg.norm(r)
    net.train_step(x, t, 1e-2)
    f = np.float32
    m, v = f(0.1) * g, f(1) * (f(1) - f(0.999)) * g * g
    ref = p0 - f(1e-2) * (m / (f(1) - f(0.9))) / (np.sqrt(v / (f(1) - f(0.999))) + f(1e-8))
    # a few FP32 roundings of the parameter and of a step of at most 1e-2
    assert np.abs(net.get_params() - ref).max() <= 8 * 2.0 ** -24 * (np.abs(p0).max() + 1e-2)
    y = [torch.empty(B, widths[-1], device="cuda:0") for _ in range(2)]
    net.forward(x, y[0])
    net.set_fused(False)
    net.forward(x, y[1])
    assert torch.equal(y[0], y[1])


@pytest.mark.parametrize("w_in,w_out,B", [(32, 32, 32), (1152, 256, 96), (1120, 160, 4096), (1120, 160, 4128),
                                          (64, 224, 8192)])
def test_fused_training_equals_layer_by_layer(w_in, w_out, B):
    """Forward and backward in one launch (16-row workgroups up to 4096 rows,
    32-row above) against the layer-by-layer products: the same products in
    the same order, so the same gradients and, over three Adam steps (whose
    update also writes the transposed weights the pass reads), the same
    parameters bit for bit.  The loss adds up to 4096 squares per partial sum
    in FP32 in another order, at most 32 additions deep: 32 x 2^-24 on each
    side."""
    import torch
    from paper_1607_05535_amd import thor
    say(f"[mlp] fused training {w_in} -> {w_out}, B={B}")
    widths = [w_in, 256, 256, 256, w_out]
    rs = np.random.default_rng(B)
    x = torch.from_numpy(rs.normal(size=(B, w_in)).astype(np.float32)).to("cuda:0").to(torch.bfloat16)
    t = torch.from_numpy(rs.normal(size=(B, w_out)).astype(np.float32)).to("cuda:0")
    res = []
    for fused in (False, True):
        net = thor.MLP(widths, B, seed=11)
        net.set_fused(fused)
        loss, g = net.loss_grad(x, t)
        for _ in range(3):
            net.train_step(x, t, 1e-3)
        loss3, g3 = net.loss_grad(x, t)
        res.append((loss, loss3, g, g3, net.get_params()))
    a, b = res
    for k in (0, 1):
        assert abs(a[k] - b[k]) <= 64 * 2.0 ** -24 * a[k]
    for k in (2, 3, 4):
        assert np.array_equal(a[k], b[k])


@pytest.mark.parametrize("widths,B", [([32, 32], 32), ([64, 96, 160], 160), ([64, 256, 256, 256, 256], 64),
                                      ([64, 256, 256, 256, 160], 96), ([64, 256, 256, 256, 256], 4128)])
@pytest.mark.parametrize("c", [3667 / 2048, 2049 / 2048])
def test_loss_adds_squares_without_losing_digits(widths, B, c):
    """Zero parameters and equal targets: every squared error is the same
    24-bit number, whose FP32 sums one after the other all round the same way
    (3.7 and 2 units over the 16 and 8 squares of a lane).  A partial sum may
    round once: 2^-24."""
    import torch
    from paper_1607_05535_amd import thor
    net = thor.MLP(widths, B)
    net.set_params(np.zeros(net.n_params, np.float32))
    x = torch.zeros(B, widths[0], dtype=torch.bfloat16, device="cuda:0")
    t = torch.full((B, widths[-1]), c, device="cuda:0")
    for fused in (True, False):
        net.set_fused(fused)
        assert abs(net.loss_grad(x, t, want_grad=False)[0] / c ** 2 - 1) <= 2.0 ** -24


@pytest.mark.parametrize("widths,B", [([2048, 4096, 512, 32], 64), ([32, 4096, 2304, 64], 1056)])
def test_gradients_of_networks_that_share_their_partial_sums(widths, B):
    """Layers whose partial sums pass 256 MiB together take several gradient
    launches in turn: two of one and two layers, and three of one."""
    test_gradients_and_adam_at_ragged_tiles(widths, B)


@pytest.mark.parametrize("K", [32, 64, 96, 128, 192, 224, 256, 288, 320, 384, 448])
def test_products_of_few_tiles(K):
    """One to seven 64-k tiles, whole and half ones: a layer of whole numbers
    (exact in BF16 and in FP32 sums) over K inputs, and its weight gradient over
    K rows from the gradient of the outputs as the kernels round it (its FP32
    sum of K terms: K 2^-24 of their absolute sum)."""
    import torch
    from paper_1607_05535_amd import thor
    say(f"[mlp] {K} inputs and rows")
    rs = np.random.default_rng(K)
    net = thor.MLP([K, 96], K)
    net.set_params(rs.integers(-4, 5, net.n_params).astype(np.float32))
    (W, b), = net.unpack(net.get_params())
    x = rs.integers(-4, 5, (K, K)).astype(np.float32)
    t = rs.integers(-4, 5, (K, 96)).astype(np.float32)
    xd, td = torch.from_numpy(x).to("cuda:0").to(torch.bfloat16), torch.from_numpy(t).to("cuda:0")
    y = torch.empty(K, 96, device="cuda:0")
    net.forward(xd, y)
    ref = x @ W.T + b
    assert np.array_equal(y.cpu().numpy(), ref)
    loss, g = net.loss_grad(xd, td)
    d = torch.from_numpy(2 * (ref - t) / np.float32(K * 96)).to(torch.bfloat16).double().numpy()
    (gW, _), = net.unpack(g)
    assert np.all(np.abs(gW - d.T @ x) <= K * 2.0 ** -24 * (np.abs(d).T @ np.abs(x)))
    assert abs(loss / np.mean((ref - t).astype(np.float64) ** 2) - 1) <= 2.0 ** -24
