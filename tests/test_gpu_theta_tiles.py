"""The general-weight kernel's layouts: several samples per tile with the last block partly empty, and single
paths on every grid in both state types (against the oracle; FP64 1e-9 and FP32 1e-5 of the batch's RMS, the
bounds of the FP64 plain-MC paths and of the FP32 pairs)."""
import numpy as np
import pytest

import dk_workloads as W
from oracle import theta

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

import paper_2311_08872_amd as dk  # noqa: E402


def problem(prec):
    return W.config2(N=1e4).with_(b0=0.5, levels=5, n0=4, precision=prec, T=0.1 / 16)


@pytest.mark.parametrize("level", [0, 1, 2, 3, 4])
@pytest.mark.parametrize("prec", [W.PREC_F32, W.PREC_F64])
def test_partial_blocks(level, prec):
    p = problem(prec)
    print(f"[gpu] b0 > 0 partial blocks n={p.n(level)} prec={prec}", flush=True)
    whole = dk.level_pair(p, level, 7, 261, per_sample=True)[1]
    for c in (1, 3, 4, 5, 15, 16, 17, 64, 65, 256, 257):
        assert torch.equal(dk.level_pair(p, level, 7, c, per_sample=True)[1], whole[:c]), c


@pytest.mark.parametrize("level,count", [(0, 70), (1, 20), (2, 6), (3, 3), (4, 2)])
@pytest.mark.parametrize("coupled", [False, True])
@pytest.mark.parametrize("prec,tol", [(W.PREC_F32, 1e-5), (W.PREC_F64, 1e-9)])
def test_every_grid(level, count, coupled, prec, tol):
    if coupled and level == 0:
        pytest.skip("no coarser level")
    p = problem(prec)
    print(f"[gpu] b0 > 0 n={p.n(level)} coupled={coupled} prec={prec}", flush=True)
    run = dk.level_pair if coupled else dk.mc_level
    gpu = run(p, level, 5, count, per_sample=True)[1].cpu().numpy()
    ref = theta.run_range(p, level, 5, count, tag=W.TAG_MLMC if coupled else W.TAG_MC, coupled=coupled)
    rms = np.sqrt(np.mean(ref ** 2, axis=0, keepdims=True))
    assert np.max(np.abs(gpu - ref) / np.maximum(np.abs(ref), rms + 1e-300)) <= tol
