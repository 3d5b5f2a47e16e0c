"""A choice that was timed, or loaded as JSON, is one of launches that fill the chip: small batches of the same grid keep the
shape (the streaming depth) of their size, and the rows that are reported are the ones that ran."""
import json

import pytest

import dk_workloads as W

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

import paper_2311_08872_amd as dk  # noqa: E402


def problem(n, pair, steps, prec=W.PREC_F32):
    return W.Problem(box=1.0, n0=n // 2 if pair else n, levels=2 if pair else 1, mu=0.1, T=steps * 0.1 / n ** 2, N=1e4,
                     steps_policy=W.STEPS_ROUND_T, rho0=W.Field(W.FIELD_MODES, 1.0, [W.cos_mode(1, 1, 0.25)]),
                     obs=W.config2_obs(), seed=n, precision=prec)


def rows(ctx, p, pair, count):
    ctx.reset()
    (dk.level_pair if pair else dk.mc_level)(p, int(pair), 0, count, ctx=ctx)
    return [s["rows"] for s in ctx.stats() if s["level"] == int(pair)][0]


def loaded(*entries):
    ctx = dk.Context(0)
    doc = json.loads(ctx.tuning_json())
    doc["shapes"] = [dict(e) for e in entries]
    ctx.load_tuning_json(json.dumps(doc))
    return ctx


# small: rows of the size; large: above the sizes at which a chip fills, the loaded choice
@pytest.mark.parametrize("n,pair,choice,small,small_rows,large", [
    (8, False, 4, 1000, 1, 90000), (8, True, 4, 1000, 2, 90000), (16, False, 4, 1000, 1, 30000), (16, True, 8, 1000, 2, 30000),
    (32, True, 16, 1000, 2, 6001), (32, False, 16, 1000, 2, 6001), (64, True, 16, 200, 2, 257), (128, True, 16, None, None, 3)])
def test_loaded_shape(n, pair, choice, small, small_rows, large):
    print(f"[gpu] loaded shape n={n} pair={pair}", flush=True)
    p = problem(n, pair, 8)
    ctx = loaded({"n": n, "pair": int(pair), "flux": 0, "rows": choice})
    assert rows(ctx, p, pair, large) == choice
    if small:
        assert rows(ctx, p, pair, small) == small_rows
    ctx.close()


def test_timed_shape():
    p = problem(16, True, 4096)
    print("[gpu] timed shape n=16", flush=True)
    ctx = dk.Context(0)
    assert rows(ctx, p, True, 100000) == 8            # 1.1e11 cell updates: timed, among the shapes of full chips
    assert [s["n"] for s in json.loads(ctx.tuning_json())["shapes"]] == [16]
    assert rows(ctx, p, True, 1000) == 2
    ctx.close()


@pytest.mark.parametrize("count,depth", [(1, 4), (12, 4), (24, 4), (26, 2), (30, 2)])
def test_loaded_depth(count, depth):
    print(f"[gpu] loaded depth, {count} pairs", flush=True)
    ctx = loaded({"n": 256, "pair": 1, "flux": 0, "depth": 2})
    assert rows(ctx, problem(256, True, 8), True, count) == -depth
    ctx.close()


def test_reported_rows_are_those_that_ran():
    print("[gpu] reported rows", flush=True)
    for n in (8, 16):                                  # one-row shapes are of single paths
        ctx = dk.Context(0)
        ctx.set_shape(n, 4)
        assert rows(ctx, problem(n, True, 8), True, 10) == 2
        assert rows(ctx, problem(n, False, 8), False, 10) == 1
        ctx.close()
        ctx = loaded({"n": n, "pair": 1, "flux": 0, "rows": 1})
        assert [s["rows"] for s in json.loads(ctx.tuning_json())["shapes"]] == [2]
        ctx.close()
    for n, v, ran in ((32, 2, 8), (32, 3, 8), (64, 1, 8), (64, 3, 4), (128, 1, 16)):    # shapes of FP64 states
        ctx = dk.Context(0)
        ctx.set_shape(n, v)
        assert rows(ctx, problem(n, True, 4, W.PREC_F64), True, 3) == ran
        ctx.close()
