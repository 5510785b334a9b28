"""The library's choice of contraction kernel away from the sizes it was first measured at: layers whose
shape would leave the newer kernels' tiles nearly empty, or short of rounds, stay on the implicit GEMM."""
import ctypes

import pytest

from gpu_util import patch_lds, pipe_lds
from paper_2307_04339_amd import _lib as L

FAKE = 0x10000


def tile_of(**fields):
    lib = L.load()
    d, h, info = L.OpDesc(), ctypes.c_void_p(), L.OpInfo()
    for k, v in dict(x=FAKE, wt=FAKE, y=FAKE, **fields).items():
        setattr(d, k, v)
    assert lib.miriam_op_create(ctypes.byref(d), ctypes.byref(h)) == 0, lib.miriam_last_error()
    assert lib.miriam_op_query(h, ctypes.byref(info)) == 0
    lib.miriam_op_destroy(h)
    return (info.tile_m, info.tile_n, info.lds_bytes)


def conv(n, h, w, c, k, ks, stride=1):
    return tile_of(kind=L.OP_CONV2D, dtype=L.F16, n=n, h=h, w=w, c=c, k=k, kh=ks, kw=ks, stride=stride, pad=ks // 2)


# the patch kernel takes 256 pixels of one image where a tile over several would need too many padded ones
@pytest.mark.parametrize("n,h,w,c,k,patch", [
    (128, 1, 1, 512, 512, False), (128, 4, 4, 512, 512, False), (64, 5, 5, 256, 256, False), (128, 1, 64, 256, 256, False),
    (128, 2, 32, 512, 512, False), (128, 2, 70, 256, 256, True), (128, 3, 100, 64, 512, False), (128, 7, 75, 64, 512, False),
    (64, 7, 160, 64, 512, False), (16, 7, 160, 64, 512, False), (4, 7, 160, 64, 512, True), (128, 6, 6, 512, 512, True),
    (8, 56, 56, 256, 256, True), (8, 120, 120, 64, 512, True),
])
def test_patch_kernel_needs_full_tiles(n, h, w, c, k, patch):
    tm, _, lds = conv(n, h, w, c, k, 3)
    assert (tm == 256 and lds in (patch_lds(64, 512), patch_lds(128, 512), patch_lds(64, 768))) == patch


def is_pipe(tm, tn, lds):
    return lds == pipe_lds(tm, tn)


@pytest.mark.parametrize("m,n,k,pipe", [
    (500, 512, 512, False), (200, 1024, 256, False), (1000, 512, 3072, False), (10000, 24, 2048, False),
    (2000, 256, 1024, False), (2000, 256, 512, True), (128, 2304, 768, False), (128, 2304, 512, True), (10000, 160, 3072, True),
    (50000, 64, 192, False), (40000, 64, 3072, False), (25000, 64, 3072, True), (50000, 64, 144, True),
    (110000, 64, 144, False), (4096, 2304, 768, True),
])
def test_pipeline_needs_rounds_for_products(m, n, k, pipe):
    assert is_pipe(*tile_of(kind=L.OP_GEMM, dtype=L.BF16, m=m, nn=n, kk=k)) == pipe


@pytest.mark.parametrize("n,h,w,c,k,ks,stride,pipe", [
    (1, 76, 76, 64, 160, 3, 2, False), (1, 96, 114, 320, 160, 3, 2, False), (13, 28, 111, 192, 24, 5, 1, False),
    (14, 100, 100, 64, 24, 3, 2, False), (11, 100, 100, 64, 24, 3, 2, True), (8, 56, 56, 128, 256, 3, 2, True),
    (44, 50, 50, 320, 24, 1, 1, False), (32, 50, 50, 144, 24, 1, 1, True),
])
def test_pipeline_needs_rounds_for_convolutions(n, h, w, c, k, ks, stride, pipe):
    assert is_pipe(*conv(n, h, w, c, k, ks, stride)) == pipe


def test_pipeline_leaves_single_chunk_scores_of_many_tiles():
    scores = dict(kind=L.OP_BGEMM, dtype=L.BF16, kk=64, batch_div=12, ldx=2304, ldw=2304, sx0=64, sw0=64)
    assert not is_pipe(*tile_of(m=512, nn=512, batch=96, ldy=512, sy0=512 * 512, **scores))
    assert is_pipe(*tile_of(m=256, nn=256, batch=48, ldy=256, sy0=256 * 256, **scores))
