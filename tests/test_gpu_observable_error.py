"""Observables of FP64 states keep the rounding errors of their sums: a product with a wave that cancels most of the field is
the exact one's rounding, whatever the tile shape.

Reference: the exact sum of the returned field's products (rational arithmetic), phi from a run whose mu = 1e-300 leaves a
field as it is.  Bound: u = 1.1e-16; the sum of the errors is itself rounded, n^2 u^2 of the terms' size, and the value four
times (the sum, h^2, its product, the errors' addition)."""
from fractions import Fraction

import numpy as np
import pytest

import dk_workloads as W

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

import paper_2311_08872_amd as dk  # noqa: E402


@pytest.mark.parametrize("n,shapes", [(4, [0]), (8, [0, 1, 2, 4]), (16, [0, 1, 2, 4]), (32, [0, 1, 4]), (64, [0, 3, 4]), (128, [0, 1])])
@pytest.mark.parametrize("coupled", [False, True])
def test_observable_is_the_exact_sums_rounding(n, shapes, coupled):
    if coupled and n == 4:
        pytest.skip("no coarser level")
    print(f"[gpu] observable error n={n} coupled={coupled}", flush=True)
    h = 1.0 / n
    phi = W.Field(W.FIELD_MODES, 0.0, [W.cos_mode(1, 0), W.sin_mode(0, 1)])
    p = W.Problem(box=1.0, n0=n // 2 if coupled else n, levels=2 if coupled else 1, mu=0.1, T=8 * 0.1 * h * h, N=1e12,
                  steps_policy=W.STEPS_ROUND_T, rho0=W.Field(W.FIELD_MODES, 1.0, [W.cos_mode(2, 1, 0.3)]), seed=n,
                  obs=[W.Obs(phi, False, False, W.PSI_ID)], precision=W.PREC_F64)
    count, level = 3, int(coupled)
    grids = [n, n // 2] if coupled else [n]
    waves = []
    for m in grids:
        still = p.with_(n0=m, levels=1, mu=1e-300, T=1e-300 / m ** 2, rho0=phi)
        waves.append(dk.meanfield(still, 0, want_field=True)[1].cpu().numpy())
    ctx = dk.Context(0)
    for v in shapes:
        ctx.set_shape(n, v)
        got, *fields = dk.level_fields(p, level, coupled, 0, count, ctx=ctx)
        got = got.cpu().numpy()[:, 0]
        for k, m in enumerate(grids):
            for i, rho in enumerate(fields[k].cpu().numpy()):
                terms = [Fraction(a) * Fraction(b) for a, b in zip(rho.ravel().tolist(), waves[k].ravel().tolist())]
                want, size = sum(terms) / m ** 2, float(sum(map(abs, terms))) / m ** 2
                assert abs(Fraction(float(got[i, k])) - want) <= 4 * 1.1e-16 * abs(float(want)) + m * m * 1.3e-32 * size, (v, m, i)
    ctx.close()
