"""GPU parity of the many-row GEMMs on outputs of few tiles, where smaller tiles are chosen: sizes around the borders of
the choice and of the tiles (ragged rows and columns, one K step, an odd number of them, both weight layouts, both output
types).  W4: 2e-6 of the oracle, the bar of the other W4 tests (fp32 sums of exact block products in another order); BF16
outputs one rounding more (2^-9 = 2e-3).  W8: 1e-6 (exact integer sums, four fp32 roundings)."""
import numpy as np
import pytest
import torch

import oracle
from paper_2605_13915_amd import synth
from gpu_util import bf16_to_dev, to_dev, rel_l2

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def msd():
    from paper_2605_13915_amd import binding
    binding.lib()
    return binding


def _both(msd, canonical, packed, y_ref, tol):
    for fn in (canonical, packed):
        if fn is None:
            continue
        for dt, t in ((torch.float32, tol), (torch.bfloat16, 2e-3)):
            y = fn(dt)
            torch.cuda.synchronize()
            assert rel_l2(y.float().cpu().numpy(), y_ref) <= t


@pytest.mark.parametrize("M,K,N", [(40, 192, 70), (129, 64, 65), (129, 320, 100), (191, 512, 33), (257, 1024, 640),
                                   (700, 512, 1500), (1000, 128, 3000), (1025, 512, 2700), (2049, 64, 1025)])
def test_w4(msd, M, K, N):
    seed = synth.seed_for(3, M + 7 * N)
    x = synth.activations(seed, M, K, outliers=K >= 1024)
    codes, exps = synth.mxfp4_weights(seed, N, K)
    y_ref = oracle.gemm_w4a16(x, codes, exps)
    xd, cd, ed = bf16_to_dev(x), to_dev(codes), to_dev(exps)
    packed = None
    if K % 512 == 0:
        p = msd.msd_pack_weights_w4(cd, ed)
        packed = lambda dt: msd.msd_gemm_w4a16_packed(xd, *p, N, out_dtype=dt)
    _both(msd, lambda dt: msd.msd_gemm_w4a16(xd, cd, ed, out_dtype=dt), packed, y_ref, 2e-6)


@pytest.mark.parametrize("M,K,N", [(65, 128, 16500), (129, 64, 12000), (129, 192, 8192), (200, 256, 11000), (777, 128, 4100),
                                   (1024, 64, 4096), (1025, 192, 3900), (672, 64, 8192), (193, 192, 28700), (1151, 64, 8100), (2048, 128, 2048), (2049, 64, 2049)])
def test_w8(msd, M, K, N):
    seed = synth.seed_for(1, M + 7 * N)
    x = synth.activations(seed, M, K, outliers=False)
    W, s = synth.int8_weights(seed, N, K)
    y_ref = oracle.gemm_w8a16(x, W, s)
    xd, Wd, sd = bf16_to_dev(x), to_dev(W), to_dev(s)
    p = msd.msd_pack_weights_w8(Wd)
    _both(msd, lambda dt: msd.msd_gemm_w8a16(xd, Wd, sd, out_dtype=dt), lambda dt: msd.msd_gemm_w8a16_packed(xd, p, sd, out_dtype=dt), y_ref, 1e-6)
