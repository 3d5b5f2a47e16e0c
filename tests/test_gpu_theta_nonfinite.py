"""b0 > 0 on grids that share a matrix tile: a sample whose state overflows changes no other sample's values.  At these
particle numbers and densities the noise drives the state to the edge of its type's range, past it on some paths and not on others;
every sample of a batch has to be what it is alone."""
import ctypes as C

import pytest

import dk_workloads as W

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

import paper_2311_08872_amd as dk  # noqa: E402
from paper_2311_08872_amd import _lib as L  # noqa: E402


def values(ctx, p, level, coupled, first, count):
    """Per-sample values whatever the status is: a batch with a value that is not finite is reported as an error."""
    out = torch.full((count, 1, 2), -1.0, dtype=torch.float64, device="cuda")
    cp = dk._cp(p)
    sums = (L.dk_moments * 1)()
    ptr, n = C.c_void_p(out.data_ptr()), C.c_uint64(count)
    if coupled:
        ctx.lib.dk_mlmc_level_pair(ctx.h, cp.ref, level, C.c_uint64(first), n, 0, sums, ptr, ctx.stream())
    else:
        ctx.lib.dk_mc_level(ctx.h, cp.ref, level, C.c_uint64(first), n, sums, ptr, ctx.stream())
    torch.cuda.synchronize()
    return out


@pytest.mark.parametrize("prec,c0,N", [(W.PREC_F64, 1e306, 1e-308), (W.PREC_F32, 1e36, 1e-38)])
@pytest.mark.parametrize("n,coupled", [(4, False), (8, False), (8, True), (16, True)])
def test_samples_of_a_tile_do_not_mix(prec, c0, N, n, coupled):
    print(f"[gpu] b0 > 0 overflowing samples n={n} coupled={coupled} prec={prec}", flush=True)
    n0, level = (n // 2, 1) if coupled else (n, 0)
    obs = [W.Obs(W.Field(W.FIELD_MODES, 0.0, [W.cos_mode(1, 0, 1e-8)]), False, False, W.PSI_ID)]
    p = W.Problem(box=1.0, n0=n0, levels=level + 1, mu=0.1, T=0.1 * 4 / n0 ** 2, N=1.0, b0=0.5, seed=3, obs=obs, precision=prec,
                  rho0=W.Field(W.FIELD_MODES, c0, []))
    ctx = dk.Context(0)
    mixed = 0
    for scale in 10.0 ** (0.25 * torch.arange(13).double()):
        q = p.with_(N=N * float(scale))
        got = values(ctx, q, level, coupled, 0, 70)
        alone = torch.cat([values(ctx, q, level, coupled, i, 1) for i in range(70)])
        assert torch.equal(torch.nan_to_num(got, nan=7.0), torch.nan_to_num(alone, nan=7.0)), float(scale)
        ok = torch.isfinite(got).all(dim=(1, 2)).sum()
        mixed += int(0 < ok < 70)
    ctx.close()
    assert mixed, "no batch with both kinds of samples"
