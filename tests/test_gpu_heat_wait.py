"""dk_heat_steps returns with the fields written, also where a single step ends in a copy: another stream that reads them
at once, and writes the scratch, waits for nothing."""
import ctypes as C

import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

import paper_2311_08872_amd as dk  # noqa: E402


@pytest.mark.parametrize("n,batch,steps", [(512, 1024, 1), (512, 1024, 2), (260, 2000, 1), (256, 1000, 1)])
def test_fields_are_written_on_return(n, batch, steps):
    print(f"[gpu] heat wait n={n} steps={steps}", flush=True)
    rho = torch.rand((batch, n, n), device="cuda")
    want = rho.clone()
    for _ in range(steps):
        lap = want.roll(1, 1) + want.roll(-1, 1) + want.roll(1, 2) + want.roll(-1, 2) - 4.0 * want
        want = want + 0.05 * lap
    work = torch.empty_like(rho)
    ctx, mine, other = dk.Context(0), torch.cuda.Stream(), torch.cuda.Stream()
    torch.cuda.synchronize()
    assert ctx.lib.dk_heat_steps(ctx.h, n, batch, steps, C.c_double(0.1), C.c_void_p(rho.data_ptr()), C.c_void_p(work.data_ptr()),
                                 None, C.c_void_p(mine.cuda_stream)) == 0
    with torch.cuda.stream(other):
        work.zero_()
        got = rho.clone()
    other.synchronize()
    assert float((got - want).abs().max()) <= steps * 1e-6
    torch.cuda.synchronize()
    ctx.close()
