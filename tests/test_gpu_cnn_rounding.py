"""The gradient at the third layer is rounded to BF16 from the dense head's FP32 values: their order of additions decides
where it falls, so it is one order, whatever the tiles are: the pixels of a channel one after the other, then the hidden
units.

The convolutions of this network are products with one weight each, so the activations are known exactly; the head is
repeated here operation by operation in FP32, and the weight gradients follow in 64 bits from the rounded values.  Their
sums of n^2 batch FP32 products hold to 64 u of the sum of the products' sizes (partial sums of at most 32 at a time);
one other rounding of a sample's gradient moves them by 2^-9 of its share of 1 / batch."""
import numpy as np
import pytest

from oracle import cnn as ref

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

import paper_2311_08872_amd as dk  # noqa: E402

F = np.float32


def bf16(v):
    return torch.from_numpy(np.ascontiguousarray(v, dtype=F)).to(torch.bfloat16).to(torch.float32).numpy()


def fma(a, b, c):
    return F(a.astype(np.float64) * b.astype(np.float64) + c.astype(np.float64))


def head(q, a3, y):
    """FP32, in the kernels' order: the gradient at the third layer's output [batch][16], and the pooled means."""
    batch, nn = a3.shape[0], a3.shape[2]
    g = np.cumsum(a3, axis=2, dtype=F)[:, :, -1] / F(nn)
    h = np.repeat(q["c1"][None], batch, 0)
    for c in range(16):
        h = fma(np.broadcast_to(q["U1"][:, c], h.shape), g[:, c:c + 1], h)
    r = np.full(batch, q["c2"][0], F)
    for k in range(64):
        r = fma(np.broadcast_to(q["U2"][0, k], r.shape), np.maximum(h[:, k], 0), r)
    dr = F(2) * (r - y) / F(batch)
    dh = np.where(h > 0, dr[:, None] * q["U2"], F(0))
    dg = np.zeros((batch, 16), F)
    for k in range(64):
        dg = fma(np.broadcast_to(q["U1"][k], dg.shape), dh[:, k:k + 1], dg)
    return bf16(dg / F(nn))


@pytest.mark.parametrize("n,batch,calls", [(4, 8, 20), (16, 3, 20), (20, 8, 20), (64, 8, 150)])
def test_gradient_is_rounded_where_the_order_of_the_head_puts_it(n, batch, calls):
    print(f"[gpu] cnn gradient rounding n={n} batch={batch}", flush=True)
    rng = np.random.default_rng(n)
    for _ in range(calls):
        p = dk.cnn_init(int(rng.integers(1 << 30))).astype(F)
        p[:4800] = 0
        w1 = rng.uniform(0.5, 2.0, 16).astype(F) * rng.choice([-1, 1], 16).astype(F)
        p[4:144:9] = w1
        for off in (160, 2480):
            p[off:off + 2304].reshape(16, 16, 9)[np.arange(16), np.arange(16), 4] = 1
        p[5824:5888] = 0.1 * rng.standard_normal(64)
        x = rng.standard_normal((batch, n, n)).astype(F)
        y = rng.standard_normal(batch).astype(F)
        q = {k: v.astype(F) for k, v in ref.unflatten(p.astype(np.float64)).items()}
        a = bf16(np.maximum(x.reshape(batch, 1, -1) * w1[None, :, None], 0))
        dz = (head(q, a, y)[:, :, None] * (a > 0)).astype(np.float64)
        _, g = dk.cnn_loss_grad(p, torch.from_numpy(x).cuda(), torch.from_numpy(y).cuda())
        got = ref.unflatten(g.astype(np.float64))["W3"][:, :, 1, 1]
        want, size = np.einsum("bop,bcp->oc", dz, a), np.einsum("bop,bcp->oc", np.abs(dz), a)
        assert np.all(np.abs(got - want) <= 64 * 6e-8 * size)
