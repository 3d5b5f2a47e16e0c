"""A forward pass of any batch keeps at most 2^17 tiles' sums and as many samples' means, 64 B each, beside its fixed
buffers; inputs on both sides of a launch's end have their own outputs."""
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

import paper_2311_08872_amd as dk  # noqa: E402


@pytest.mark.parametrize("n,batch", [(4, 900000), (8, 300000), (36, 22000), (64, 16390)])
def test_forward_memory_is_bounded(n, batch):
    print(f"[gpu] cnn memory n={n} batch={batch}", flush=True)
    p = dk.cnn_init(1)
    x = torch.randn((batch, n, n), device="cuda", generator=torch.Generator("cuda").manual_seed(n))
    ctx = dk.Context(0)
    r = dk.cnn_forward(p, x[:8].contiguous(), ctx=ctx)
    torch.cuda.synchronize()
    free = torch.cuda.mem_get_info()[0]
    got = dk.cnn_forward(p, x, ctx=ctx)
    torch.cuda.synchronize()
    used = free - torch.cuda.mem_get_info()[0]
    assert used <= 2 * (1 << 17) * 64 + (20 << 20) + 4 * batch          # allocation granularity; the output itself
    for at in ((1 << 17) // (1 if n < 20 else 6 if n == 36 else 8), batch - 5, 0):
        some = dk.cnn_forward(p, x[max(0, at - 3):at + 3].contiguous(), ctx=ctx)
        assert torch.allclose(got[max(0, at - 3):at + 3], some, rtol=0, atol=4e-6 * float(got.abs().max()))
    assert torch.allclose(got[:8], r, rtol=0, atol=4e-6 * float(got.abs().max()))
    ctx.close()
