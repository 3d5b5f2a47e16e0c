"""Batches of every size take the tile shape of that size; a sample's values do not depend on it: each
batch equals, bit for bit, the same samples of a batch that runs the default shape."""
import pytest

import dk_workloads as W

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

import paper_2311_08872_amd as dk  # noqa: E402


# counts on both sides of the lines where the rows per lane change (1, 2, 4, 8), a single sample among them
@pytest.mark.parametrize("n,prec,counts", [
    (8, W.PREC_F32, [1, 6000, 6001, 24000, 24001, 80001]), (16, W.PREC_F32, [1, 1200, 1201, 20000, 20001]),
    (32, W.PREC_F32, [1, 2500, 2501, 6000, 6001]), (64, W.PREC_F32, [1, 256, 257, 400, 401]),
    (8, W.PREC_F64, [1, 3000, 3001, 8193, 20001]), (16, W.PREC_F64, [1, 800, 801, 3001, 10001]),
    (32, W.PREC_F64, [1, 600, 601, 6001]), (64, W.PREC_F64, [1, 300, 301, 769, 1025]), (128, W.PREC_F64, [1, 3]),
])
@pytest.mark.parametrize("pair", [True, False])
def test_values_do_not_depend_on_the_batch(n, prec, counts, pair):
    print(f"[gpu] batches n={n} prec={prec} pair={pair}", flush=True)
    steps = 8 if n < 128 else 4
    p = W.Problem(box=1.0, n0=n // 2 if pair else n, levels=2 if pair else 1, mu=0.1, T=steps * 0.1 / n ** 2, N=1e4,
                  steps_policy=W.STEPS_ROUND_T, rho0=W.Field(W.FIELD_MODES, 1.0, [W.cos_mode(1, 1, 0.25)]),
                  obs=W.config2_obs(), seed=n, precision=prec)
    run = (lambda c, ctx: dk.level_pair(p, 1, 5, c, per_sample=True, ctx=ctx)) if pair else \
        (lambda c, ctx: dk.mc_level(p, 0, 5, c, per_sample=True, ctx=ctx))
    base = dk.Context(0)
    base.set_shape(n, 0)
    want = run(max(counts), base)[1]
    ctx = dk.Context(0)
    for c in counts:
        ms, ps = run(c, ctx)
        assert torch.equal(ps, want[:c]), c
        y = ps[:, 0, 0] - ps[:, 0, 1]
        assert abs(float(y.sum()) - ms[0].sums[0]) <= 1e-12 * float(y.abs().sum()) and ms[0].count == c
    ctx.close()
    base.close()
