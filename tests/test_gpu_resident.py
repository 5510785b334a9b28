"""Resident-weight convolutions whose output rows are no whole 16-byte pieces: the register epilogue
stores four channels at a time and the rest by element."""
import numpy as np
import pytest
import torch

from gpu_util import RTOL, bits, empty, f32_dev, gpu_available, rand, rel_err, to_f64

pytestmark = [pytest.mark.gpu,
              pytest.mark.skipif(not gpu_available(), reason="needs an MI355X")]

# (N, H, W, C, K, ks, stride, act): widths of no, one and several whole groups of four channels, rows
# at every alignment, the last n tile with one channel, and C = 64 (staged epilogue) beside it
CASES = [
    (1, 9, 35, 24, 63, 1, 1, "relu6"),
    (2, 7, 33, 16, 20, 3, 1, "relu"),
    (1, 13, 40, 8, 30, 3, 2, "none"),
    (1, 5, 32, 32, 65, 1, 1, "gelu"),
    (1, 6, 31, 32, 3, 3, 1, "relu"),
    (1, 9, 37, 64, 33, 3, 1, "relu"),
    (1, 8, 36, 64, 600, 1, 1, "relu"),  # parameters of one n tile at a time
]


@pytest.mark.parametrize("dtype", ["f16", "bf16"])
@pytest.mark.parametrize("case", CASES)
def test_resident_odd_widths_match_oracle_and_are_elastic(orc, dtype, case):
    from paper_2307_04339_amd import _lib as L, ops
    N, H, W, C, K, ks, st, act = case
    p = ks // 2
    x, x64 = rand((N, H, W, C), dtype, seed=K)
    w, w64 = rand((K, ks, ks, C), dtype, seed=K + 1, lo=-0.2, hi=0.2)
    Ho, Wo = (H + 2 * p - ks) // st + 1, (W + 2 * p - ks) // st + 1
    b64 = np.random.default_rng(K + 2).uniform(-1, 1, K).astype(np.float32).astype(np.float64)
    res, r64 = rand((N, Ho, Wo, K), dtype, seed=K + 3)
    y = empty((N, Ho, Wo, K), dtype)
    op = ops.conv2d(x, w, y, stride=st, pad=p, bias=f32_dev(b64), residual=res, act=act, tile=8)
    assert op.info.path == L.PATH_RESIDENT
    op.run()
    torch.cuda.synchronize()
    ref = orc.conv2d(x64, w64, stride=st, pad=p, bias=b64, bn=None, residual=r64, act=act)
    assert rel_err(to_f64(y), ref) <= RTOL[dtype]
    ref_bits = bits(y)
    for block in [64, 128, 256]:
        y.fill_(float("nan"))
        for b, l in reversed(orc.balanced_split(op.T, min(3, op.T))):
            op.launch(b, l, 2, block)
        torch.cuda.synchronize()
        assert bits(y) == ref_bits, block
