"""Centring constants that vanish in exact arithmetic: the value is the rounding of the scheme's own steps, in their
order of operations.  The paper's datum has half the period of its observable, so (rho^M, I_h phi)_h = 0 there.

The steps and the sums are repeated here operation by operation on the library's own rho^0 and phi (a run whose
mu = 1e-300 leaves a field as it is), so the comparison is exact."""
from fractions import Fraction

import numpy as np
import pytest

import dk_workloads as W

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

import paper_2311_08872_amd as dk  # noqa: E402


def fma(a, b, c):
    return float(Fraction(a) * Fraction(b) + Fraction(c))


def device_field(p, f, level):
    h = p.h(level)
    q = W.Problem(box=p.box, n0=p.n(level), levels=1, mu=1e-300, T=1e-300 * h * h, N=p.N, steps_policy=W.STEPS_ROUND_T,
                  rho0=f, obs=p.obs, precision=W.PREC_F64)
    return dk.meanfield(q, 0, want_field=True)[1].cpu().numpy()


def stepped(rho, a, steps, resident):
    for _ in range(steps):
        s = (np.roll(rho, 1, 1) + np.roll(rho, -1, 1)) + (np.roll(rho, 1, 0) + np.roll(rho, -1, 0))
        lap = s - 4.0 * rho                              # 4 rho is exact: one rounding, as in the kernels
        if resident:
            rho = rho + a * lap
        else:
            rho = np.array([fma(a, l, c) for l, c in zip(lap.ravel(), rho.ravel())]).reshape(rho.shape)
    return rho


def product(rho, phi, h2, resident):
    n = len(rho)
    if not resident:                                     # 256 strided sums, then halves
        r, f = rho.ravel(), phi.ravel()
        v = np.zeros(256)
        for t in range(256):
            for i in range(t, n * n, 256):
                v[t] = fma(r[i], f[i], v[t])
        w = 128
        while w:
            v[:w] += v[w:2 * w]
            w //= 2
        return h2 * v[0]
    rows, lanes = (4 if n == 4 else 16 if n == 128 else 8), n // 2
    v = np.zeros((n // rows) * lanes)
    for t in range(len(v)):
        g, c = t // lanes, t % lanes
        for i in range(rows):
            for k in range(2):
                v[t] = fma(rho[rows * g + i, 2 * c + k], phi[rows * g + i, 2 * c + k], v[t])
    total = 0.0
    for w in v.reshape(-1, min(len(v), 64)):             # a wavefront's lanes: halves; then in order
        while len(w) > 1:
            w = w[:len(w) // 2] + w[len(w) // 2:]
        total = total + w[0]
    return h2 * total


@pytest.mark.parametrize("name,level", [(k, l) for k in ("paper_reg", "paper_irreg") for l in range(6)] +
                         [("paper_fourier", 1), ("paper_fourier", 2)])
def test_vanishing_centre_is_that_of_the_steps(name, level):
    p = getattr(W, name)()
    n = p.n(level)
    print(f"[gpu] vanishing centre {name} n={n}", flush=True)
    resident = n in (4, 8, 16, 32, 64, 128)
    centre, rho = dk.meanfield(p, level, want_field=True)
    want = stepped(device_field(p, p.rho0, level), 0.5 * p.mu, p.steps(level), resident)
    assert np.array_equal(rho.cpu().numpy(), want)
    assert centre[0] == product(want, device_field(p, p.obs[0].phi, level), p.h(level) ** 2, resident)
    assert abs(centre[0]) <= 1e-14


@pytest.mark.parametrize("n", [64, 128, 256, 320])
def test_a_uniform_field_stays_uniform(n):
    """The product with a wave cancels, so the field comes from the steps, which keep 1 exactly."""
    print(f"[gpu] uniform field n={n}", flush=True)
    h = 1.0 / n
    p = W.Problem(box=1.0, n0=n, levels=1, mu=0.1, T=4096 * 0.1 * h * h, N=1e4, steps_policy=W.STEPS_ROUND_T,
                  rho0=W.Field(W.FIELD_MODES, 1.0, []), obs=[W.Obs(W.Field(W.FIELD_MODES, 0.0, [W.cos_mode(1, 0)]), True, True,
                                                                   W.PSI_ID)])
    centre, rho = dk.meanfield(p, 0, want_field=True)
    assert torch.equal(rho, torch.ones_like(rho))
    assert abs(centre[0]) <= 1e-14
