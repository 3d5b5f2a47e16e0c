"""The control variate's tiled kernels at the edges of their tiles: partial and several tiles per
sample, several samples per block, batches that do not fill a block, and a batch of one.

The reference is the FP64 network with BF16 rounding at the points where the kernels round (operands
and outputs of the 16->16 layers, and the gradients there): a batch of one has few units, and one ReLU
that the rounding of a layer's input switches moves its whole gradient.

Tolerances as for the other sizes: 1e-2 of the output's RMS, 3e-2 of a gradient block's norm."""
import numpy as np
import pytest

from oracle import cnn as ref

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

import paper_2311_08872_amd as dk  # noqa: E402


def bf16(v):
    return torch.from_numpy(np.ascontiguousarray(v, dtype=np.float32)).to(torch.bfloat16).to(torch.float64).numpy()


def rounded_network(p, x, y):
    """Outputs, loss and gradient of the network with the kernels' BF16 rounding points."""
    a1 = bf16(np.maximum(ref.conv(x[:, None], p["W1"], p["b1"]), 0))
    w2, w3 = bf16(p["W2"]), bf16(p["W3"])
    a2 = bf16(np.maximum(ref.conv(a1, w2, p["b2"]), 0))
    a3 = bf16(np.maximum(ref.conv(a2, w3, p["b3"]), 0))
    g = a3.mean(axis=(2, 3))
    h = g @ p["U1"].T + p["c1"]
    r = np.maximum(h, 0) @ p["U2"][0] + p["c2"][0]
    dr = 2.0 * (r - y) / len(y)
    dh = dr[:, None] * p["U2"] * (h > 0)
    dz3 = bf16((dh @ p["U1"])[:, :, None, None] / x[0].size) * (a3 > 0)
    d2, dW3, db3 = ref.conv_backward(a2, w3, dz3)
    dz2 = bf16(d2 * (a2 > 0))
    d1, dW2, db2 = ref.conv_backward(a1, w2, dz2)
    _, dW1, db1 = ref.conv_backward(x[:, None], p["W1"], bf16(d1 * (a1 > 0)))
    grad = {"W1": dW1, "b1": db1, "W2": dW2, "b2": db2, "W3": dW3, "b3": db3, "U1": dh.T @ g, "c1": dh.sum(0),
            "U2": (dr @ np.maximum(h, 0))[None], "c2": np.array([dr.sum()])}
    return r, float(np.mean((r - y) ** 2)), grad


# n = 4 .. 16: several samples per block; 20: two tiles of rows, 4 of 8 pixels idle; 36: 2 x 3 tiles with a
# partial last column; 64: 2 x 4 full tiles; 132: 5 x 9 tiles, partial in both directions
@pytest.mark.parametrize("n,batch", [(4, 1), (4, 1500), (8, 3001), (12, 1200), (16, 5), (20, 7), (36, 6), (64, 3), (132, 2)])
def test_forward_and_gradient_at_tile_edges(n, batch):
    print(f"[gpu] cnn tiles n={n} batch={batch}", flush=True)
    rng = np.random.default_rng(n)
    p = dk.cnn_init(n).astype(np.float32)
    for off, cnt in [(144, 16), (2464, 16), (4784, 16), (5824, 64), (5952, 1)]:
        p[off:off + cnt] = 0.1 * rng.standard_normal(cnt)
    x = rng.standard_normal((batch, n, n)).astype(np.float32)
    y = rng.standard_normal(batch).astype(np.float32)
    xd, yd = torch.from_numpy(x).cuda(), torch.from_numpy(y).cuda()
    r = dk.cnn_forward(p, xd).cpu().numpy()
    loss, g = dk.cnn_loss_grad(p, xd, yd)
    prm = ref.unflatten(p.astype(np.float64))
    rr, lr, gr = rounded_network(prm, x.astype(np.float64), y.astype(np.float64))
    assert np.max(np.abs(r - rr)) <= 1e-2 * np.sqrt(np.mean(rr ** 2))
    assert abs(loss - lr) <= 1e-2 * lr
    gd = ref.unflatten(g.astype(np.float64))
    for k in ref.ORDER:
        assert np.linalg.norm(gd[k] - gr[k]) <= 3e-2 * np.linalg.norm(gr[k]) + 1e-7, k
    # a second call on the same buffers gives the same bits
    loss2, g2 = dk.cnn_loss_grad(p, xd, yd)
    assert loss2 == loss and np.array_equal(g2, g)
    assert np.array_equal(dk.cnn_forward(p, xd).cpu().numpy(), r)


@pytest.mark.parametrize("n,batch", [(4, 1500), (8, 3001), (16, 2000)])
def test_samples_of_a_block_do_not_mix(n, batch):
    """An input that is not finite changes its own output only (several samples share a block's image)."""
    print(f"[gpu] cnn one infinite input of {batch}, n={n}", flush=True)
    p = dk.cnn_init(n).astype(np.float32)
    x = torch.from_numpy(np.random.default_rng(n).standard_normal((batch, n, n)).astype(np.float32)).cuda()
    want = dk.cnn_forward(p, x)
    bad = x.clone()
    bad[7] = float("inf")
    got = dk.cnn_forward(p, bad)
    keep = torch.arange(batch, device="cuda") != 7
    assert torch.equal(got[keep], want[keep])
