"""GPU parity and elastic invariance of the register-tile pipelined contraction at the edges of its
tiles (rows, columns, K chunks, batches, filter taps), through the library's own choice of tile."""
import numpy as np
import pytest
import torch

from gpu_util import bits, empty, f32_dev, gpu_available, pipe_lds, rand, rel_err, to_f64

pytestmark = [pytest.mark.gpu,
              pytest.mark.skipif(not gpu_available(), reason="needs an MI355X")]

# one rounding to the output type (half an ulp: 2^-11 and 2^-8 of the value) plus fp32 sums of at
# most a few thousand products (below 1e-4 of the rms here) and, for GELU, an erf of 1.5e-7
TOL = {"f16": 2.0 ** -11 + 1e-4, "bf16": 2.0 ** -8 + 1e-4}


@pytest.fixture(scope="module")
def ops():
    from paper_2307_04339_amd import ops as o
    return o


def _is_pipe(op, tile):
    from paper_2307_04339_amd import _lib as L
    return (op.info.path in (L.PATH_DMA, L.PATH_DMA_UNIFORM)
            and (op.info.tile_m, op.info.tile_n, op.info.ksplit) == (*tile, 1) and op.info.lds_bytes == pipe_lds(*tile))


def _elastic(op, y, orc):
    ref = bits(y)
    for n, block in [(1, 256), (3, 256), (2, 128), (5, 64)]:
        y.fill_(float("nan"))
        for j, (b, l) in enumerate(reversed(orc.balanced_split(op.T, n))):
            op.launch(b, l, [l, 7, l + 3][j % 3], block)
        torch.cuda.synchronize()
        assert bits(y) == ref, (n, block)


# M, N, K, act, residual, row strides padded by 8, tile
GEMMS = [
    (500, 520, 200, "gelu", True, True, (64, 64)),       # K tail of 8, last column tile 8 wide
    (1027, 264, 40, "none", False, False, (64, 64)),     # a single partial chunk
    (2000, 520, 72, "relu", False, True, (128, 64)),
    (2000, 1032, 136, "relu6", True, False, (128, 128)),
    (4104, 1032, 64, "none", False, False, (256, 128)),
    (4000, 3064, 128, "gelu", False, False, (256, 192)),
]


@pytest.mark.parametrize("case", GEMMS)
@pytest.mark.parametrize("dtype", ["f16", "bf16"])
def test_pipe_gemm_matches_oracle_and_is_elastic(ops, orc, dtype, case):
    M, N, K, act, has_res, padded, tile = case
    ld = K + 8 if padded else K
    x, x64 = rand((M, ld), dtype, seed=1)
    w, w64 = rand((N, ld), dtype, seed=2, lo=-0.2, hi=0.2)
    x[:, K:] = float("nan")  # past the row's K values: never used
    w[:, K:] = float("nan")
    b64 = np.random.default_rng(3).uniform(-1, 1, N).astype(np.float32).astype(np.float64)
    res, r64 = rand((M, N), dtype, seed=4) if has_res else (None, None)
    y = empty((M, N), dtype)
    op = ops.gemm(x, w, y, bias=f32_dev(b64), residual=res, act=act, ldx=ld, ldw=ld, k=K)
    assert _is_pipe(op, tile), (op.info.path, op.info.tile_m, op.info.tile_n, op.info.lds_bytes)
    op.run()
    torch.cuda.synchronize()
    ref = orc.linear(np.ascontiguousarray(x64[:, :K]), np.ascontiguousarray(w64[:, :K]), bias=b64, residual=r64, act=act)
    err = rel_err(to_f64(y), ref)
    print(f"pipe {dtype} {case}: T={op.T} rel={err:.3e}")
    assert err <= TOL[dtype], err
    _elastic(op, y, orc)


# N, H, W, C, K, ks, stride, pad, act, bn, residual, tile
CONVS = [
    # two images: the 225 32x32 tiles fit the CUs one each, and the four-stage kernel has it; with five the pipeline
    (2, 40, 40, 64, 264, 3, 2, 1, "relu", True, False, (32, 32)),
    (5, 40, 40, 64, 264, 3, 2, 1, "relu", True, False, (64, 64)),
    (9, 21, 23, 144, 24, 1, 1, 0, "none", True, True, (64, 64)),     # one tap, K tail of 16, narrow output
    (9, 41, 23, 40, 72, 1, 2, 0, "relu6", False, False, (64, 64)),   # one tap, stride 2, K below a chunk
    (15, 40, 40, 64, 136, 3, 2, 1, "relu", False, True, (128, 64)),
    (15, 40, 40, 64, 392, 2, 2, 0, "none", True, False, (128, 128)),
    (15, 40, 40, 64, 776, 2, 2, 0, "relu", False, False, (256, 128)),
]


@pytest.mark.parametrize("case", CONVS)
def test_pipe_conv_matches_oracle_and_is_elastic(ops, orc, case):
    N, H, W, C, K, ks, st, pad, act, has_bn, has_res, tile = case
    dtype = "bf16" if has_bn else "f16"
    x, x64 = rand((N, H, W, C), dtype, seed=1)
    w, w64 = rand((K, ks, ks, C), dtype, seed=2, lo=-0.2, hi=0.2)
    Ho, Wo = (H + 2 * pad - ks) // st + 1, (W + 2 * pad - ks) // st + 1
    rng = np.random.default_rng(3)
    bn64 = np.stack([rng.uniform(0.8, 1.2, K), rng.uniform(-0.1, 0.1, K), rng.uniform(-0.1, 0.1, K),
                     rng.uniform(0.8, 1.2, K)]).astype(np.float32).astype(np.float64) if has_bn else None
    res, r64 = rand((N, Ho, Wo, K), dtype, seed=4) if has_res else (None, None)
    y = empty((N, Ho, Wo, K), dtype)
    op = ops.conv2d(x, w, y, stride=st, pad=pad, bn=f32_dev(bn64) if has_bn else None, residual=res, act=act)
    assert _is_pipe(op, tile) if tile != (32, 32) else (op.info.tile_m, op.info.tile_n) == tile, (
        op.info.path, op.info.tile_m, op.info.tile_n, op.info.lds_bytes)
    op.run()
    torch.cuda.synchronize()
    ref = orc.conv2d(x64, w64, stride=st, pad=pad, bn=None if bn64 is None else tuple(bn64), residual=r64, act=act)
    err = rel_err(to_f64(y), ref)
    print(f"pipe {dtype} {case}: T={op.T} rel={err:.3e}")
    assert err <= TOL[dtype], err
    _elastic(op, y, orc)


@pytest.mark.parametrize("B,H,S,tile", [(4, 6, 136, (64, 64)), (2, 12, 264, (128, 128)), (3, 12, 264, (256, 128))])
def test_pipe_batched_scores_match_oracle(ops, orc, B, H, S, tile):
    D = 64
    qkv, q64 = rand((B * S, 3 * H * D), "bf16", seed=5)
    y = empty((B * H, S, S), "bf16")
    op = ops.bgemm(qkv, qkv[:, H * D:], y, m=S, n=S, k=D, batch=B * H, batch_div=H, ldx=3 * H * D, ldw=3 * H * D, ldy=S,
                   sx=(S * 3 * H * D, D), sw=(S * 3 * H * D, D), sy=(H * S * S, S * S))
    assert _is_pipe(op, tile), (op.info.path, op.info.tile_m, op.info.tile_n, op.info.lds_bytes)
    op.run()
    torch.cuda.synchronize()
    q = q64.reshape(B, S, 3, H, D)
    ref = np.einsum("bihd,bjhd->bhij", q[:, :, 0], q[:, :, 1]).reshape(B * H, S, S)
    assert rel_err(to_f64(y), ref) <= TOL["bf16"]
    _elastic(op, y, orc)


# attention's probabilities times values ([k][n] right operand); odd lengths go through the
# register-staged kernel, which reads the probabilities' rows in unaligned 16-byte pieces
@pytest.mark.parametrize("B,H,S,tile", [(4, 8, 136, (64, 64)), (13, 12, 128, (128, 64)), (12, 12, 256, (256, 64)),
                                        (3, 4, 131, None), (2, 3, 9, None)])
@pytest.mark.parametrize("dtype", ["f16", "bf16"])
def test_batched_context_matches_oracle_and_is_elastic(ops, orc, dtype, B, H, S, tile):
    from paper_2307_04339_amd import _lib as L
    D = 64
    p, p64 = rand((B * H, S, S), dtype, seed=6, lo=0.0, hi=1.0)
    qkv, q64 = rand((B * S, 3 * H * D), dtype, seed=7)
    y = empty((B * S, H * D), dtype)
    op = ops.bgemm(p, qkv[:, 2 * H * D:], y, m=S, n=D, k=S, batch=B * H, batch_div=H, ldx=S, ldw=3 * H * D, ldy=H * D,
                   sx=(H * S * S, S * S), sw=(S * 3 * H * D, D), sy=(S * H * D, D), b_nmajor=True)
    if tile:
        assert _is_pipe(op, tile), (op.info.path, op.info.tile_m, op.info.tile_n, op.info.lds_bytes)
    else:
        assert op.info.path == L.PATH_STAGED
    op.run()
    torch.cuda.synchronize()
    v = q64.reshape(B, S, 3, H, D)[:, :, 2]
    ref = np.einsum("bhij,bjhd->bihd", p64.reshape(B, H, S, S), v).reshape(B * S, H * D)
    err = rel_err(to_f64(y), ref)
    print(f"context {dtype} {B}x{H}x{S}: T={op.T} rel={err:.3e}")
    assert err <= TOL[dtype], err
    _elastic(op, y, orc)


# a single K chunk: the epilogue's parameters have one meeting between their writer and their readers.
# M, N, K, 1x1 convolution stride (None: product), tile
ONE_CHUNK = [
    (4000, 120, 64, None, (64, 64)),
    (4000, 120, 40, 2, (64, 64)),
    (16000, 120, 64, None, (128, 64)),
    (16000, 120, 40, 1, (128, 64)),
]


@pytest.mark.parametrize("case", ONE_CHUNK)
@pytest.mark.parametrize("dtype", ["f16", "bf16"])
def test_pipe_single_chunk_parameters(ops, orc, dtype, case):
    M, N, K, stride, tile = case
    rng = np.random.default_rng(12)
    # parameters far apart from channel to channel: another channel's, or none, would show
    b64 = (rng.uniform(-1, 1, N) + np.arange(N) % 7).astype(np.float32).astype(np.float64)
    w, w64 = rand((N, K), dtype, seed=13, lo=-0.2, hi=0.2)
    if stride is None:
        x, x64 = rand((M, K), dtype, seed=14)
        y = empty((M, N), dtype)
        op = ops.gemm(x, w, y, bias=f32_dev(b64), act="none")
        ref = orc.linear(x64, w64, bias=b64)
    else:
        x, x64 = rand((M // 400, 20 * stride, 20 * stride, K), dtype, seed=14)
        y = empty((M // 400, 20, 20, N), dtype)
        bn64 = np.stack([rng.uniform(0.5, 2, N), rng.uniform(-3, 3, N), rng.uniform(-1, 1, N),
                         rng.uniform(0.5, 2, N)]).astype(np.float32).astype(np.float64)
        op = ops.conv2d(x, w.reshape(N, 1, 1, K), y, stride=stride, pad=0, bias=f32_dev(b64), bn=f32_dev(bn64))
        ref = orc.conv2d(x64, w64.reshape(N, 1, 1, K), stride=stride, pad=0, bias=b64, bn=tuple(bn64))
    assert _is_pipe(op, tile), (op.info.path, op.info.tile_m, op.info.tile_n, op.info.lds_bytes)
    op.run()
    torch.cuda.synchronize()
    assert rel_err(to_f64(y), ref) <= TOL[dtype]
    _elastic(op, y, orc)


@pytest.mark.parametrize("S", [40, 64])
def test_context_of_a_single_chunk_matches_oracle(ops, orc, S):
    B, H, D = 16, 12, 64
    p, p64 = rand((B * H, S, S), "bf16", seed=15, lo=0.0, hi=1.0)
    qkv, q64 = rand((B * S, 3 * H * D), "bf16", seed=16)
    y = empty((B * S, H * D), "bf16")
    op = ops.bgemm(p, qkv[:, 2 * H * D:], y, m=S, n=D, k=S, batch=B * H, batch_div=H, ldx=S, ldw=3 * H * D, ldy=H * D,
                   sx=(H * S * S, S * S), sw=(S * 3 * H * D, D), sy=(S * H * D, D), b_nmajor=True)
    assert _is_pipe(op, (64, 64)), (op.info.path, op.info.tile_m, op.info.tile_n, op.info.lds_bytes)
    op.run()
    torch.cuda.synchronize()
    v = q64.reshape(B, S, 3, H, D)[:, :, 2]
    ref = np.einsum("bhij,bjhd->bihd", p64.reshape(B, H, S, S), v).reshape(B * S, H * D)
    assert rel_err(to_f64(y), ref) <= TOL["bf16"]
    _elastic(op, y, orc)


@pytest.mark.parametrize("n", [1, 3, 8, 77, 333, 512, 520, 2047, 2056])
@pytest.mark.parametrize("dtype", ["f32", "f16", "bf16"])
def test_rows_of_any_length_match_oracle(ops, orc, dtype, n):
    tol = {"f32": 1e-5, **TOL}[dtype]
    rows = 13
    x, x64 = rand((rows, n + 3), dtype, seed=8, lo=-3, hi=3)
    x[5, :] = torch.finfo(x.dtype).min  # a fully masked row: uniform probabilities
    x64 = to_f64(x)
    y = empty((rows, n + 5), dtype)
    ops.softmax(x, y, rows, n, scale=1.0, ldx=n + 3, ldy=n + 5).run()
    torch.cuda.synchronize()
    got = to_f64(y)
    assert np.isnan(got[:, n:]).all()  # nothing past the rows' ends
    assert rel_err(got[:, :n], orc.softmax_rows(np.ascontiguousarray(x64[:, :n]), 1.0)) <= tol
    z, z64 = rand((rows, n), dtype, seed=9, lo=-2, hi=2)
    r, r64 = rand((rows, n), dtype, seed=10)
    rng = np.random.default_rng(11)
    g, b = (rng.uniform(0.5, 1.5, n).astype(np.float32).astype(np.float64) for _ in range(2))
    o = empty((rows, n), dtype)
    ops.layernorm(z, f32_dev(g), f32_dev(b), o, rows, n, residual=r, eps=1e-2).run()
    torch.cuda.synchronize()
    # values near +-3 on parameters near 1.5: a few fp32 ulps more than the output's rounding
    assert rel_err(to_f64(o), orc.layernorm_rows(z64 + r64, g, b, 1e-2)) <= tol + 1e-5
