"""Order and rounding of the network's sums: in FP32 no more than 32 terms are added
one after another before a sum joins others like it; in BF16 an output's sum has
one order however the product is launched."""
import math

import numpy as np
import pytest

from oracle import mlp as omlp
from tests.test_gpu_mlp import make

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def qg():
    from paper_2310_06650_amd import qg as _qg
    return _qg


def rms(a, ref):
    return np.linalg.norm(a - ref) / np.linalg.norm(ref)


def product32(a, b):
    """a @ b in FP32: fused multiply-adds in chains of 32, the chains in sums of
    eight, those one after another."""
    total = np.zeros((a.shape[0], b.shape[1]), np.float32)
    for k8 in range(0, a.shape[1], 256):
        eight = np.zeros_like(total)
        for k32 in range(k8, min(k8 + 256, a.shape[1]), 32):
            acc = np.zeros_like(total)
            for k in range(k32, min(k32 + 32, a.shape[1])):
                acc = (acc.astype(np.float64) + np.outer(a[:, k].astype(np.float64), b[k])
                       ).astype(np.float32)
            eight += acc
        total += eight
    return total


@pytest.mark.parametrize("batch", [64, 1024])
def test_error_is_that_of_chains_of_32(qg, batch):
    """Outputs and the output layer's weight gradient of 512 -> 512 -> 512 are no
    further from 64 bits than a model with chains of 32: independent rounding
    errors of chains of 64 under eight sums would be sqrt((64 + 8) / (32 + 2 + 8))
    = 1.31 times as large, half of that excess is allowed."""
    import torch
    net, params, x, t, xd, td = make(qg, 512, 512, 1, 512, batch, seed=batch)
    y = net.forward(xd).cpu().numpy()
    g = net.grad_and_loss(xd, td)[0].cpu().numpy()
    torch.cuda.synchronize()
    (W1, b1), (W2, b2) = params
    f32 = np.float32
    h = omlp.gelu(product32(x.astype(f32), W1.astype(f32)) + b1.astype(f32)).astype(f32)
    ym = product32(h, W2.astype(f32)) + b2.astype(f32)
    dy = f32(2.0) * (ym - t.astype(f32)) * f32(1.0 / t.size)
    dwm = product32(np.ascontiguousarray(h.T), dy)
    y_ref = omlp.forward(params, x)
    dw_ref = omlp.loss_and_grad(params, x, t)[1][1][0]
    wo = net.offsets(1)[0]
    assert rms(y, y_ref) <= 1.15 * rms(ym, y_ref)
    assert rms(g[wo:wo + dw_ref.size].reshape(dw_ref.shape), dw_ref) <= 1.15 * rms(dwm, dw_ref)


def test_long_batch(qg):
    """A weight gradient of 65,536 rows whose terms are mostly of one sign, so that
    every partial sum matters: sums of 32, 8, 8, 8 and 4 terms have errors of at most
    2^-24 / sqrt(3) sqrt(32 / (3 2048) + 8 / (3 256) + 8 / (3 32) + 8 / (3 4) + 4 / 3) = 5e-8
    in the mean square; twice that is allowed.  All divisors are powers of two."""
    import torch
    net, params, x, _, xd, td = make(qg, 32, 32, 1, 32, 65536, seed=7)
    t = np.full(td.shape, -3.0)
    td.fill_(-3.0)
    g = net.grad_and_loss(xd, td)[0].cpu().numpy()
    torch.cuda.synchronize()
    dw_ref = omlp.loss_and_grad(params, x, t)[1][1][0]
    wo = net.offsets(1)[0]
    bound = 2.0 ** -24 / math.sqrt(3) * math.sqrt(32 / 6144 + 8 / 768 + 8 / 96 + 8 / 12 + 4 / 3)
    assert rms(g[wo:wo + dw_ref.size].reshape(dw_ref.shape), dw_ref) <= 2 * bound


@pytest.mark.parametrize("width", [64, 97, 128, 200, 301, 512, 1000])
def test_bf16_outputs_do_not_depend_on_how_many_there_are(qg, width):
    """An output's sum has one order whether the output layer takes one launch
    (64 tiles and more) or slices (fewer), bit for bit: 4,096 outputs and the
    first 2,048 of them."""
    import torch
    wide, params, x, _, xd, _ = make(qg, 8, width, 1, 4096, 50, seed=width)
    few = qg.MLP(8, width, 1, 2048, max_batch=50)
    flat = np.zeros(few.n_params, dtype=np.float32)
    for i, (W, b) in enumerate(params):
        W, b = (W, b) if i == 0 else (W[:, :2048], b[:2048])
        wo, bo = few.offsets(i)
        flat[wo:wo + W.size], flat[bo:bo + b.size] = W.reshape(-1), b
    few.set_params(flat)
    for net in (wide, few):
        net.to_bf16()
    a = wide.forward_bf16(xd).cpu().numpy()
    b = few.forward_bf16(xd).cpu().numpy()
    torch.cuda.synchronize()
    assert np.array_equal(a[:, :2048], b)
