"""GELU of 16-bit outputs, element by element against float64: the fp32 value before the rounding must be
as good as v / 2 (1 + erff(v / sqrt 2)) at every argument, also in the negative tail, where a bound
relative to the tensor's rms says nothing."""
import numpy as np
import pytest
import torch

from gpu_util import TORCH, empty, gpu_available, to_f64

pytestmark = [pytest.mark.gpu,
              pytest.mark.skipif(not gpu_available(), reason="needs an MI355X")]

BITS = {"f16": (10, -14), "bf16": (7, -126)}  # mantissa bits, exponent of the smallest normal value
EDGES = [-12.5, -9, -6, -4, -3, -2, -1.25, -0.5, -0.01, 0, 0.01, 0.5, 1.25, 2, 4, 8]


def _ulp(v, dtype):
    mant, low = BITS[dtype]
    return 2.0 ** (np.maximum(np.floor(np.log2(np.maximum(np.abs(v), 1e-300))), low) - mant)


def _gelu(ops, v, dtype, m):
    """GELU of the fp32 values v, handed over as the bias of a product of zeros with m rows: up to 16
    rows the small-batch kernel computes erff, beyond the contraction kernels the form under test."""
    n = v.numel()
    x = torch.zeros((m, 128), dtype=TORCH[dtype], device="cuda")
    w = torch.zeros((n, 128), dtype=TORCH[dtype], device="cuda")
    y = empty((m, n), dtype)
    op = ops.gemm(x, w, y, bias=v, act="gelu")
    op.run()
    torch.cuda.synchronize()
    return to_f64(y[-1]), op


@pytest.mark.parametrize("dtype", ["f16", "bf16"])
def test_gelu_is_as_exact_as_erff_at_every_argument(dtype):
    from paper_2307_04339_amd import _lib as L, ops
    for k, (a, b) in enumerate(zip(EDGES, EDGES[1:])):
        v = torch.from_numpy(np.random.default_rng(k).uniform(a, b, 1 << 16).astype(np.float32)).cuda()
        v64 = v.double().cpu()
        ref = (0.5 * v64 * torch.special.erfc(-v64 / 2.0 ** 0.5)).numpy()
        got, op = _gelu(ops, v, dtype, 32)
        old, ref_op = _gelu(ops, v, dtype, 16)
        assert op.info.path != L.PATH_SKINNY and ref_op.info.path == L.PATH_SKINNY
        err, was = (np.abs(y - ref) / _ulp(ref, dtype) for y in (got, old))
        print(f"gelu {dtype} [{a}, {b}]: {err.max():.5f} ulp, rms {np.sqrt((err ** 2).mean()):.6f}; "
              f"erff {was.max():.5f}, {np.sqrt((was ** 2).mean()):.6f}")
        # half an ulp for the rounding and 5e-6 of the value, at most 2^(mantissa bits + 1) ulps, before it
        assert err.max() <= 0.5 + 5e-6 * 2.0 ** (BITS[dtype][0] + 1)
        # no larger than erff's but for the few values of 65536 that lie at a tie
        assert np.sqrt((err ** 2).mean()) <= np.sqrt((was ** 2).mean()) * (1 + 1e-5)


@pytest.mark.parametrize("dtype", ["f16", "bf16"])
def test_gelu_of_infinities_nan_and_zeros(dtype):
    from paper_2307_04339_amd import ops
    v = torch.tensor([float("inf"), float("-inf"), float("nan"), 0.0, 1e30, -1e30, -30.0, 6e4], dtype=torch.float32,
                     device="cuda")
    got, _ = _gelu(ops, v.repeat(8), dtype, 32)
    old, _ = _gelu(ops, v.repeat(8), dtype, 16)
    assert np.array_equal(got, old, equal_nan=True), (got[:8], old[:8])
