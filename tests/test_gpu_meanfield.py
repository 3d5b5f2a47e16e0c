"""The discrete mean field of every kind of grid against numpy's FFT of the same scheme: rho^M has the
Fourier coefficients g^M rho^0, g = 1 - 2 mu (sin^2(pi kx/n) + sin^2(pi ky/n)).

Tolerance: the transform forms sums of n products twice each way with factors of size sqrt(2); with
u = 1.1e-16 the error of a cell is at most 4 * 2 n u * max |rho| in the worst case and grows like
sqrt(n) u in practice, and g^M carries a few u of its own; bound 64 sqrt(n) u max |rho|.  Stepping (few
steps) adds steps * 8 u."""
import math

import numpy as np
import pytest

import dk_workloads as W

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

import paper_2311_08872_amd as dk  # noqa: E402


# one block up to 64, several launches beyond; 12, 36, 108: grids of the Fourier coupling (not a multiple of
# 16); 6, 22, 70: sizes that are only even; 1 step and 3 steps: stepping; mu = 0.5: g down to -1
@pytest.mark.parametrize("n", [4, 6, 8, 12, 16, 22, 32, 36, 64, 70, 108, 128, 256, 320, 1024])
@pytest.mark.parametrize("steps,mu", [(1, 0.1), (3, 0.5), (40, 0.25), (1001, 0.5), (60000, 0.1)])
def test_meanfield_against_fft(n, steps, mu):
    print(f"[gpu] mean field n={n} steps={steps} mu={mu}", flush=True)
    h = 1.0 / n
    modes = W.random_modes(6, n, amp_max=0.2, kmax=max(2, n // 2)) + [W.cos_mode(1, 0, 0.3), W.cos_mode(n // 2, n // 2, 0.2)]
    phi = W.Field(W.FIELD_MODES, 0.5, [W.cos_mode(1, 0), W.sin_mode(0, 1)])
    p = W.Problem(box=1.0, n0=n, levels=1, mu=mu, T=steps * mu * h * h, N=1e4, steps_policy=W.STEPS_ROUND_T,
                  rho0=W.Field(W.FIELD_MODES, 1.0, modes), obs=[W.Obs(phi, True, False, W.PSI_ID)] * 3, seed=0)
    ctx = dk.Context(0)
    centre, rho = dk.meanfield(p, 0, want_field=True, ctx=ctx)
    ctx.close()
    c = np.arange(n) / n
    grid = lambda f: f.c0 + sum(m.amp * np.cos(2 * math.pi * (m.kx * c[None, :] + m.ky * c[:, None]) + m.phase)
                                for m in f.modes)   # noqa: E731
    s = np.sin(math.pi * c) ** 2
    lam = 2 * mu * (s[:, None] + s[None, :])
    with np.errstate(divide="ignore"):
        g = np.where(lam <= 1, np.exp(steps * np.log1p(-np.minimum(lam, 1.0))),
                     (-1.0) ** steps * np.exp(steps * np.log1p(np.maximum(lam, 1.0) - 2.0)))
    ref = np.real(np.fft.ifft2(np.fft.fft2(grid(p.rho0)) * g))
    top = np.max(np.abs(grid(p.rho0)))
    bound = (64 * math.sqrt(n) + (8 * steps if steps <= 64 else 0)) * 1.1e-16 * top
    assert np.max(np.abs(rho.cpu().numpy() - ref)) <= bound
    want = float(np.sum(ref * grid(phi))) * h * h
    assert np.allclose(centre, want, rtol=0, atol=2 * bound)
