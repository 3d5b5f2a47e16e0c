"""An observable whose sum leaves the range of FP64 is infinite, as a plain sum of its terms is, in the kernels whose sums
carry their rounding errors."""
import ctypes as C

import numpy as np
import pytest

import dk_workloads as W

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

import paper_2311_08872_amd as dk  # noqa: E402
from paper_2311_08872_amd import _lib as L  # noqa: E402


def problem(n, sign, **kw):
    h = 1.0 / n
    return W.Problem(box=1.0, n0=n, levels=1, mu=0.1, T=2 * 0.1 * h * h, N=1e9, rho0=W.Field(W.FIELD_MODES, 1.0, []), seed=1,
                     obs=[W.Obs(W.Field(W.FIELD_MODES, sign * 1e308, []), False, False, W.PSI_ID)], **kw)


@pytest.mark.parametrize("sign", [1.0, -1.0])
@pytest.mark.parametrize("kind", ["fourier", "theta", "stream"])
def test_overflowing_sum_is_infinite(kind, sign):
    print(f"[gpu] overflowing observable {kind} {sign}", flush=True)
    ctx = dk.Context(0)
    if kind == "fourier":
        p = problem(8, sign, coupling=W.COUPLING_FOURIER, precision=W.PREC_F64)
    elif kind == "theta":
        p = problem(8, sign, b0=0.5, precision=W.PREC_F64)
    else:
        p = problem(64, sign)
        ctx.set_streaming(True)
    out = torch.zeros((3, 1, 2), dtype=torch.float64, device="cuda")
    sums = (L.dk_moments * 1)()
    # the batch is reported as not finite; its values are written all the same
    assert ctx.lib.dk_mc_level(ctx.h, dk._cp(p).ref, 0, C.c_uint64(0), C.c_uint64(3), sums, C.c_void_p(out.data_ptr()),
                               ctx.stream()) == -4
    torch.cuda.synchronize()
    ctx.close()
    assert np.array_equal(out[:, 0, 0].cpu().numpy(), np.full(3, sign * np.inf))
