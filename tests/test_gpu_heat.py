"""dk_heat_steps over every layout: several fields per wavefront, a field per block, windows with halos,
row groups that do not divide the field, odd and even step counts, batches that leave lanes idle.

Each FP32 step rounds its five operations: the update a * lap (|a lap| <= 4 a max|rho| <= max|rho|) and
the sum carry at most 3 u max|rho| of new error (u = 2^-24), and the scheme does not amplify errors in
the maximum norm for mu <= 1/4 (convex combination); bound 4 u steps max|rho|."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

import paper_2311_08872_amd as dk  # noqa: E402


@pytest.mark.parametrize("n,batch", [(4, 70), (8, 3), (12, 200), (32, 2300), (36, 9), (60, 5), (64, 7), (68, 4), (100, 3),
                                     (128, 5), (132, 2), (252, 2), (256, 3), (260, 2), (512, 2), (700, 1), (1024, 1)])
@pytest.mark.parametrize("steps,mu", [(0, 0.1), (1, 0.25), (2, 0.1), (17, 0.25), (64, 0.1)])
def test_heat_layouts(n, batch, steps, mu):
    print(f"[gpu] heat n={n} batch={batch} steps={steps}", flush=True)
    g = torch.Generator(device="cuda").manual_seed(n + steps)
    rho = torch.rand((batch + 1, n, n), device="cuda", generator=g) + 0.5
    guard = rho[batch].clone()                    # the field behind the batch stays untouched
    x = rho[:batch].double()
    dk.heat_steps(rho[:batch], steps, mu)
    for _ in range(steps):
        x = x + 0.5 * mu * (x.roll(1, 1) + x.roll(-1, 1) + x.roll(1, 2) + x.roll(-1, 2) - 4.0 * x)
    torch.cuda.synchronize()
    assert torch.equal(rho[batch], guard)
    err = (rho[:batch].double() - x).abs().max().item()
    assert err <= 4 * 2.0 ** -24 * steps * 1.5, err
