"""Softmax element by element against float64 where the scaled scores are large beside their spread: the
exponent's argument must come from one rounding of scale v - max, not from the difference of two rounded
products, and the terms and quotients must be good to an fp32 rounding or two."""
import numpy as np
import pytest
import torch

from gpu_util import empty, gpu_available, rand, to_f64

pytestmark = [pytest.mark.gpu,
              pytest.mark.skipif(not gpu_available(), reason="needs an MI355X")]

BITS = {"f32": (23, -126), "f16": (10, -14), "bf16": (7, -126)}  # mantissa bits, exponent of the smallest normal value


@pytest.mark.parametrize("n", [40, 96, 129, 512, 1000, 4104])
@pytest.mark.parametrize("dtype", ["f32", "f16", "bf16"])
def test_softmax_of_large_scores_is_exact_to_rounding(dtype, n):
    from paper_2307_04339_amd import ops
    rows, scale = 24, 0.3
    x, x64 = rand((rows, n), dtype, seed=n, lo=300, hi=350)
    y = empty((rows, n), dtype)
    ops.softmax(x, y, rows, n, scale=scale).run()
    torch.cuda.synchronize()
    z = x64 * np.float64(np.float32(scale))
    e = np.exp(z - z.max(axis=1, keepdims=True))
    ref = e / e.sum(axis=1, keepdims=True)
    mant, low = BITS[dtype]
    ulp = 2.0 ** (np.maximum(np.floor(np.log2(ref)), low) - mant)
    err = (np.abs(to_f64(y) - ref) / ulp).max()
    # before the rounding to the output: half an ulp of an argument below 16, one of the exponential, two of
    # the sum (terms of one sign, added in a tree) and one of the quotient, relative to the value
    before = 2.0 ** -21 + 4 * 2.0 ** -24
    print(f"softmax {dtype} n={n}: {err:.4f} ulp")
    assert err <= 0.5 + before * 2.0 ** (mant + 1)
