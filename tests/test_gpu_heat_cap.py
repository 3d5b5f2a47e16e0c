"""The launch cap bounds the steps of one launch of the noise-free scheme, as it bounds a level's; fields are the same."""
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

import paper_2311_08872_amd as dk  # noqa: E402


@pytest.mark.parametrize("n,batch,steps", [(256, 4, 50), (100, 7, 301), (64, 1000, 9), (8, 20000, 5)])
def test_capped_launches_give_the_same_fields(n, batch, steps):
    print(f"[gpu] heat cap n={n} steps={steps}", flush=True)
    x = torch.rand((batch, n, n), device="cuda", generator=torch.Generator("cuda").manual_seed(n))
    y = x.clone()
    ctx = dk.Context(0)
    dk.heat_steps(x, steps, 0.2, ctx=ctx)
    ctx.set_launch_cap(1e6)                        # one to sixteen steps a launch
    dk.heat_steps(y, steps, 0.2, ctx=ctx)
    ctx.close()
    assert torch.equal(x, y)
