"""The Fourier kernel's lane layouts: several samples per wavefront with the last block partly empty, and
the FP64 state on the grids 8, 24, 72 (against the oracle; 1e-9 of the batch's RMS, as for the FP64
plain-MC paths: the uncentred sums here cancel nothing beyond the increments themselves)."""
import numpy as np
import pytest

import dk_workloads as W
from oracle import fourier as F

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

import paper_2311_08872_amd as dk  # noqa: E402


@pytest.mark.parametrize("n0", [4, 8])
@pytest.mark.parametrize("level", [0, 1, 2])
@pytest.mark.parametrize("prec", [W.PREC_F32, W.PREC_F64])
def test_partial_blocks(n0, level, prec):
    p = W.config2(N=1e4).with_(coupling=W.COUPLING_FOURIER, levels=3, n0=n0, precision=prec, T=0.1 / n0 ** 2)
    print(f"[gpu] Fourier partial blocks n={p.n(level)} prec={prec}", flush=True)
    whole = dk.level_pair(p, level, 7, 131, per_sample=True)[1]
    for c in (1, 2, 3, 12, 13, 128, 129):
        assert torch.equal(dk.level_pair(p, level, 7, c, per_sample=True)[1], whole[:c]), c


@pytest.mark.parametrize("level,count", [(0, 40), (1, 9), (2, 2)])
def test_unit_box_fp64(level, count):
    p = W.config2(N=1e4).with_(coupling=W.COUPLING_FOURIER, levels=3, precision=W.PREC_F64)
    print(f"[gpu] Fourier FP64 n={p.n(level)}", flush=True)
    gpu = dk.level_pair(p, level, 5, count, per_sample=True)[1].cpu().numpy()
    ref = F.run_range(p, level, 5, count)
    rms = np.sqrt(np.mean(ref ** 2, axis=0, keepdims=True))
    assert np.max(np.abs(gpu - ref) / np.maximum(np.abs(ref), rms + 1e-300)) <= 1e-9
