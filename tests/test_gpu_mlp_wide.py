"""Networks so wide that the rows of a product's tile span more than the 4 GiB a
32-bit byte offset reaches, against plain 64-bit torch on the device.  Products
of 2e7 FP32 terms in chains of 32 carry under 2e-5 normwise, BF16 operands 3e-2."""
import pytest

pytestmark = pytest.mark.gpu

WIDE = (1 << 24) + (1 << 22)  # 64 rows of it: 5.4e9 bytes
CHUNK = 1 << 20


@pytest.fixture(scope="module")
def qg():
    from paper_2310_06650_amd import qg as _qg
    return _qg


def layer(net, flat, i, a, b):
    wo, bo = net.offsets(i)
    return flat[wo:wo + a * b].view(a, b), flat[bo:bo + b]


def close(got, ref, tol):
    return float((got.double() - ref).abs().max()) <= tol * float(ref.abs().max())


def test_wide_output_layer(qg):
    """A training step of 8 -> 64 -> 2e7: the activation gradient reads 64 rows of
    the weights (dW_1 shows it), the weight gradient updates 64 rows of parameters
    and moments."""
    import torch
    B, W, lr = 2, 64, 1e-3
    gen = torch.Generator(device="cuda").manual_seed(5)
    net = qg.MLP(8, W, 1, WIDE, max_batch=B)
    net.params.normal_(0, 0.3, generator=gen)
    net.m.normal_(0, 1e-8, generator=gen)
    net.v.copy_(net.m)
    net.v.square_()
    before = [a.clone() for a in (net.params, net.m, net.v)]
    x = torch.randn(B, 8, generator=gen, device="cuda")
    t = torch.randn(B, WIDE, generator=gen, device="cuda")
    loss = net.train_step(x, t, lr)
    grad = net.grad
    (W1, b1), (W2, b2) = layer(net, before[0], 0, 8, W), layer(net, before[0], 1, W, WIDE)
    z = (x.double() @ W1.double() + b1.double())
    z.requires_grad_(True)
    h = torch.nn.functional.gelu(z)
    hd = h.detach()
    dh = torch.zeros_like(hd)
    total = 0.0
    new = {k: layer(net, a, 1, W, WIDE)[0]
           for k, a in (("p", net.params), ("m", net.m), ("v", net.v), ("g", grad))}
    old = {k: layer(net, a, 1, W, WIDE)[0] for k, a in zip("pmv", before)}
    for c in range(0, WIDE, CHUNK):
        s = slice(c, min(c + CHUNK, WIDE))
        w = W2[:, s].double()
        d = hd @ w + b2[s].double() - t[:, s].double()
        total += float((d * d).sum())
        dy = 2.0 * d / (B * WIDE)
        dh += dy @ w.T.contiguous()
        g = hd.T.contiguous() @ dy
        assert close(new["g"][:, s], g, 2e-5), c
        m = 0.9 * old["m"][:, s].double() + 0.1 * g
        v = 0.999 * old["v"][:, s].double() + 0.001 * g * g
        assert close(new["m"][:, s], m, 2e-5) and close(new["v"][:, s], v, 4e-5), c
        # the update from the moments as stored: a few FP32 roundings
        m, v = new["m"][:, s].double(), new["v"][:, s].double()
        p = old["p"][:, s].double() - lr * (m / 0.1) / ((v / 0.001).sqrt() + 1e-8)
        assert close(new["p"][:, s], p, 1e-6), c
    assert abs(float(loss) - total / (B * WIDE)) <= 2e-5 * total / (B * WIDE)
    h.backward(dh)
    assert close(layer(net, grad, 0, 8, W)[0], x.double().T.contiguous() @ z.grad, 2e-5)


def test_wide_input_layer(qg):
    """Forward passes of 2e7 -> 1 -> 1 on 64 rows, in both precisions."""
    import torch
    B = 64
    gen = torch.Generator(device="cuda").manual_seed(6)
    net = qg.MLP(WIDE, 1, 1, 1, max_batch=B)
    net.params.normal_(0, 1.0, generator=gen)
    net.params[:WIDE] *= WIDE ** -0.5
    net.to_bf16()
    x = torch.randn(B, WIDE, generator=gen, device="cuda")
    y, y16 = net.forward(x), net.forward_bf16(x)
    for got, cast, tol in ((y, lambda a: a.double(), 2e-5),
                           (y16, lambda a: a.bfloat16().double(), 3e-2)):
        z = torch.zeros(B, 1, dtype=torch.float64, device="cuda")
        (W1, b1), (W2, b2) = layer(net, net.params, 0, WIDE, 1), layer(net, net.params, 1, 1, 1)
        for c in range(0, WIDE, CHUNK):
            s = slice(c, min(c + CHUNK, WIDE))
            z += cast(x[:, s]) @ cast(W1[s])
        ref = torch.nn.functional.gelu(z + cast(b1)) @ cast(W2) + cast(b2)
        assert close(got, ref, tol)
