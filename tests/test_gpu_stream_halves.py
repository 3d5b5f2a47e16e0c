"""Streamed batches that advance as two halves on two streams (more than 256 tiles of 64 x 64): every sample's
values are those of a batch that runs on one stream, bit for bit, at every depth."""
import pytest

import dk_workloads as W

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

import paper_2311_08872_amd as dk  # noqa: E402


@pytest.mark.parametrize("depth", [4, 1, 2, 8])
@pytest.mark.parametrize("coupled", [True, False])
@pytest.mark.parametrize("flux", [W.FLUX_CENTRAL, W.FLUX_STAGGERED])
def test_halves_match_one_stream(depth, coupled, flux):
    p = W.config2(N=3e3).with_(flux=flux, n0=128, levels=2)
    p = p.with_(T=p.tau(1) * 16)
    print(f"[gpu] stream halves depth={depth} coupled={coupled} flux={flux}", flush=True)
    run = dk.level_pair if coupled else dk.mc_level
    ctx = dk.Context(0)
    ctx.set_stream_depth(depth)
    whole = run(p, 1, 3, 35, per_sample=True, ctx=ctx)[1]       # 560 tiles, 17 and 18 samples
    for first, count in ((0, 17), (17, 2)):                     # 272 tiles: two streams; 32: one
        part = run(p, 1, 3 + first, count, per_sample=True, ctx=ctx)[1]
        assert torch.equal(part, whole[first:first + count]), (first, count)
    one = torch.cat([run(p, 1, 3 + b, min(16, 35 - b), per_sample=True, ctx=ctx)[1] for b in range(0, 35, 16)])
    assert torch.equal(one, whole)                              # 256 tiles and fewer: one stream
    side = torch.cuda.Stream()
    with torch.cuda.stream(side):
        again = run(p, 1, 3, 35, per_sample=True, ctx=ctx)[1]
    assert torch.equal(again, whole)
    ctx.close()


@pytest.mark.parametrize("coupled", [True, False])
@pytest.mark.parametrize("flux", [W.FLUX_CENTRAL, W.FLUX_STAGGERED])
def test_small_tiles_match_large(coupled, flux):
    """Depth 4 in 32 x 32 tiles (up to 192 tiles of 64 x 64 a launch) and in 64 x 64 tiles; 13 steps of single
    paths end on a partial launch."""
    level = 1 if coupled else 0
    p = W.config2(N=3e3).with_(flux=flux, n0=320 >> level, levels=level + 1)
    p = p.with_(T=p.tau(level) * (12 if coupled else 13), steps_policy=W.STEPS_EXACT)
    print(f"[gpu] stream tile sizes coupled={coupled} flux={flux}", flush=True)
    run = dk.level_pair if coupled else dk.mc_level
    ctx = dk.Context(0)
    ctx.set_stream_depth(4)
    large = run(p, level, 0, 8, per_sample=True, ctx=ctx)[1]         # 320 x 320: 200 tiles
    for first, count in ((0, 7), (7, 1)):
        assert torch.equal(run(p, level, first, count, per_sample=True, ctx=ctx)[1], large[first:first + count])
    ctx.close()
