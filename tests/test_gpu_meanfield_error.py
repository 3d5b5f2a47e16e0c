"""The mean field formed in the scheme's eigenbasis is no further from the exact field than the scheme's steps are: both
against the basis products in extended precision, the steps repeated here in FP64 from the library's own rho^0."""
import numpy as np
import pytest

import dk_workloads as W

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

import paper_2311_08872_amd as dk  # noqa: E402

X = np.longdouble


def exact(rho0, mu, steps):
    n = len(rho0)
    k = np.arange(n)
    t = 2 * X("3.14159265358979323846264338327950288") / n
    c = np.cos(t * (np.outer(k, k) % n)) + np.sin(t * (np.outer(k, k) % n))
    s = np.sin(t * k / 2) ** 2
    g = np.exp(steps * np.log1p(-2 * X(mu) * (s[:, None] + s[None, :])))
    return (c @ ((c @ rho0.astype(X) @ c) * g) @ c) / (X(n) * n)


def stepped(rho, a, steps):
    for _ in range(steps):
        rho = rho + a * (((np.roll(rho, 1, 1) + np.roll(rho, -1, 1)) + (np.roll(rho, 1, 0) + np.roll(rho, -1, 0))) - 4.0 * rho)
    return rho


@pytest.mark.parametrize("name,level", [("config2", 1), ("config2", 2), ("config5", 1), ("config5", 2)])
@pytest.mark.parametrize("seed", [0, 1, 2])
def test_error_is_no_larger_than_that_of_the_steps(name, level, seed):
    p = getattr(W, name)()
    phase = np.random.default_rng(seed).uniform(0, 3, 2)
    long_waves = [W.Mode(0.2, 1, 0, float(phase[0])), W.Mode(0.2, 1, 1, float(phase[1]))]
    p = p.with_(rho0=W.Field(W.FIELD_MODES, 1.0, W.random_modes(6, seed) + long_waves), obs=[
        W.Obs(W.Field(W.FIELD_MODES, 0.0, [W.Mode(1.0, 1, 0, float(phase[0]))]), True, True, W.PSI_ID)])
    n, h = p.n(level), p.h(level)
    print(f"[gpu] mean field error {name} n={n} seed={seed}", flush=True)
    still = W.Problem(box=p.box, n0=n, levels=1, mu=1e-300, T=1e-300 * h * h, N=p.N, steps_policy=W.STEPS_ROUND_T, rho0=p.rho0,
                      obs=p.obs)
    rho0 = dk.meanfield(still, 0, want_field=True)[1].cpu().numpy()
    want = exact(rho0, p.mu, p.steps(level))
    err = lambda f: float(np.linalg.norm((f.astype(X) - want).astype(np.float64)))     # noqa: E731
    centre, rho = dk.meanfield(p, level, want_field=True)
    assert abs(centre[0]) > 1e-3                       # not a product that cancels: the eigenbasis is used
    assert err(rho.cpu().numpy()) <= err(stepped(rho0, 0.5 * p.mu, p.steps(level)))
