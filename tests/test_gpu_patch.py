"""GPU parity and elastic invariance of the 3x3 stride-1 patch convolution (the tile's input pixels
in LDS, 256 consecutive output pixels per tile) at the sizes where its tile, run and channel edges
lie, through the library's own choice of kernel."""
import numpy as np
import pytest
import torch

from gpu_util import bits, empty, f32_dev, gpu_available, ints, patch_lds, rand, rel_err, to_f64

pytestmark = [pytest.mark.gpu,
              pytest.mark.skipif(not gpu_available(), reason="needs an MI355X")]

# one rounding to the output type (half an ulp: 2^-11 and 2^-8 of the value) plus fp32 sums of
# at most a few thousand products (below 1e-4 of the rms here)
TOL = {"f16": 2.0 ** -11 + 1e-4, "bf16": 2.0 ** -8 + 1e-4}

# N, H, W, C, K, pad, act, bias, bn, residual, tile_n
CASES = [
    (1, 56, 56, 32, 256, 1, "relu", True, False, False, 64),    # one chunk of channels, last tile 64 pixels
    (3, 33, 21, 96, 328, 1, "relu6", False, True, True, 64),    # tiles across images, last n tile 8 channels
    (2, 64, 64, 32, 128, 1, "gelu", True, False, False, 64),    # run too long across images: tiles per image
    (1, 20, 150, 32, 256, 1, "none", True, True, False, 64),    # wide image: the larger patch buffer
    (4, 30, 30, 64, 512, 0, "relu", True, False, True, 64),     # no padding, two chunks
    (70, 7, 7, 32, 264, 2, "none", False, False, False, 64),    # small images, wider padding
    (11, 56, 56, 32, 256, 1, "relu", True, False, False, 128),  # 128-channel tiles, two rounds per workgroup
]


@pytest.fixture(scope="module")
def ops():
    from paper_2307_04339_amd import ops as o
    return o


def _is_patch(op, tile_n):
    from paper_2307_04339_amd import _lib as L
    return ((op.info.path, op.info.tile_m, op.info.tile_n, op.info.ksplit) == (L.PATH_DMA_UNIFORM, 256, tile_n, 1)
            and op.info.lds_bytes in (patch_lds(tile_n, 512), patch_lds(tile_n, 768)))


@pytest.mark.parametrize("case", CASES)
@pytest.mark.parametrize("dtype", ["f16", "bf16"])
def test_patch_conv_matches_oracle_and_is_elastic(ops, orc, dtype, case):
    N, H, W, C, K, pad, act, has_bias, has_bn, has_res, tile_n = case
    x, x64 = rand((N, H, W, C), dtype, seed=1)
    w, w64 = rand((K, 3, 3, C), dtype, seed=2, lo=-0.2, hi=0.2)
    Ho, Wo = H + 2 * pad - 2, W + 2 * pad - 2
    rng = np.random.default_rng(3)
    b64 = rng.uniform(-1, 1, K).astype(np.float32).astype(np.float64) if has_bias else None
    bn64 = np.stack([rng.uniform(0.8, 1.2, K), rng.uniform(-0.1, 0.1, K), rng.uniform(-0.1, 0.1, K),
                     rng.uniform(0.8, 1.2, K)]).astype(np.float32).astype(np.float64) if has_bn else None
    res, r64 = rand((N, Ho, Wo, K), dtype, seed=4) if has_res else (None, None)
    y = empty((N, Ho, Wo, K), dtype)
    op = ops.conv2d(x, w, y, stride=1, pad=pad, bias=f32_dev(b64) if has_bias else None,
                    bn=f32_dev(bn64) if has_bn else None, residual=res, act=act)
    assert _is_patch(op, tile_n), (op.info.path, op.info.tile_m, op.info.tile_n)
    op.run()
    torch.cuda.synchronize()
    ref = orc.conv2d(x64, w64, stride=1, pad=pad, bias=b64, bn=None if bn64 is None else tuple(bn64),
                     residual=r64, act=act)
    err = rel_err(to_f64(y), ref)
    print(f"patch {dtype} {case}: T={op.T} rel={err:.3e}")
    assert err <= TOL[dtype], err
    ref_bits = bits(y)
    for n, block in [(1, 256), (3, 256), (2, 128), (5, 64)]:
        y.fill_(float("nan"))
        for j, (b, l) in enumerate(reversed(orc.balanced_split(op.T, n))):
            op.launch(b, l, [l, 7, l + 3][j % 3], block)
        torch.cuda.synchronize()
        assert bits(y) == ref_bits, (n, block)


def test_patch_conv_integer_inputs_exact(ops, orc):
    # operands in {-1, 0, 1}: partial sums of at most 288 terms are exact in fp32 and fp16
    x, x64 = ints((3, 40, 40, 32), "f16", seed=5, lo=-1, hi=1)
    w, w64 = ints((192, 3, 3, 32), "f16", seed=6, lo=-1, hi=1)
    y = empty((3, 40, 40, 192), "f16")
    op = ops.conv2d(x, w, y, stride=1, pad=1)
    assert _is_patch(op, 64)
    op.run()
    torch.cuda.synchronize()
    assert np.array_equal(to_f64(y), orc.conv2d(x64, w64, stride=1, pad=1))


def test_patch_conv_tile_map_matches_oracle(ops, orc):
    x, _ = rand((3, 40, 40, 32), "bf16", seed=8)
    w, _ = rand((192, 3, 3, 32), "bf16", seed=9, lo=-0.1, hi=0.1)
    y = empty((3, 40, 40, 192), "bf16")
    op = ops.conv2d(x, w, y, stride=1, pad=1)
    T = op.T
    assert _is_patch(op, 64) and T == 19 * 3
    for n, grids, block in [(1, [T], 256), (4, [5, 64, 1, 3], 128), (3, [7, 7, 7], 64), (2, [4, 2], 256)]:
        plan = orc.balanced_split(T, n)
        ow, oi = (torch.full((T,), -1, dtype=torch.int32, device="cuda") for _ in range(2))
        cnt = torch.zeros((T,), dtype=torch.int32, device="cuda")
        wp, ws = (torch.full((4 * T,), -1, dtype=torch.int32, device="cuda") for _ in range(2))
        for (b, l), g in zip(plan, grids):
            op.launch_traced(b, l, g, block, ow, oi, cnt, wave_phys=wp, wave_slot=ws)
        torch.cuda.synchronize()
        _, wg_ref, it_ref, cnt_ref = orc.owner_map(T, plan, grids)
        assert np.array_equal(cnt.cpu().numpy(), cnt_ref)
        assert np.array_equal(ow.cpu().numpy(), wg_ref)
        assert np.array_equal(oi.cpu().numpy(), it_ref)
        exp = np.array([orc.wave_map(4, block // 64, lam) for lam in range(4)], dtype=np.int32)
        assert np.array_equal(wp.cpu().numpy().reshape(T, 4), np.tile(exp[:, 0], (T, 1)))
        assert np.array_equal(ws.cpu().numpy().reshape(T, 4), np.tile(exp[:, 1], (T, 1)))
