// Direct convolution with the weights resident in registers and the epilogue from registers, for
// 3x3 stride 2 on 8-channel images (at most 64 output channels) and 1x1 stride 1 (any number) (fp16 / bf16).
// Tile, wave split, patch stream, weights, K order and elastic blocks are in conv_rw_tile.h.  With one n
// tile a workgroup loads its weights once; with several (1x1) the next tile's load with its patch.
//
// With the weights as the MFMA's row operand a lane ends up with four adjacent output channels of one
// pixel, so the tile is finished and stored from registers.  Staged through LDS these layers spent two
// barriers and a pass over LDS on a tile of 1 to 5 K steps and had LDS for two workgroups per CU instead
// of three (1x1 of 16x56x56x24 to 144 channels 12.4 to 9.6 us, 3x3 stride 2 of 16x224x224x8 to 32
// channels 16.5 to 10.6).  3x3 stride 1 stays staged: at C = 64 the 144 weight registers leave none for
// this epilogue (conv1_2 of VGG-16 b8 44.8 against 42.4 us), and from memory the whole 128-byte rows
// matter more than the barriers (conv1_1 to pool1 of VGG-16 b8 on buffers in turn 71.2 against 70.3 us).
#pragma once

#include "conv_rw_tile.h"
#include "tile_regs.h"

namespace miriam {

template <class T, int C, int P, int KS, int ST>
struct RwRegsKernel : RwTile<T, C, P, KS, ST> {
    static_assert((KS == 3 && ST == 2) || (KS == 1 && ST == 1), "3x3 stride 2, 1x1 stride 1");
    using RwTile<T, C, P, KS, ST>::PATCH;
    static constexpr int AFFN = 512;                       // channels whose affine parameters LDS keeps for the launch
    static constexpr int AFF0 = 2 * PATCH;
    static constexpr int LDS_BYTES = AFF0 + 2 * AFFN * 4;
    static constexpr int NST = 4;                          // output stores per wave and tile (P = 4)
    static constexpr int WAVES_PER_SIMD = (P == 4 && 2 * (LDS_BYTES + 16) <= 160 * 1024) ? 2 : 1;
};

template <class T, int C, int P, int KS, int ST>
__global__ __launch_bounds__(kWave * P, (RwRegsKernel<T, C, P, KS, ST>::WAVES_PER_SIMD)) void rw_regs_kernel(IgemmArgs a,
                                                                                                     Shard sh) {
    typedef RwRegsKernel<T, C, P, KS, ST> K_;
    typedef typename K_::MF MF;
    typedef typename K_::op_t op_t;
    typedef typename K_::acc_t acc_t;
    constexpr int TW = K_::TW, NT = K_::NT, NS = K_::NS, SL = K_::SL, ROUNDS = K_::ROUNDS, BUF = K_::PATCH;

    __shared__ __attribute__((aligned(1024))) char smem_[K_::LDS_BYTES];
    const uint32_t lds0 = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) char *)smem_;

    const int tid = threadIdx.x;
    const int pw = __builtin_amdgcn_readfirstlane(tid / kWave);
    const int lane = tid % kWave;
    const int hx = lane >> 5, xl = lane & 31;  // MFMA operand half, pixel column / channel
    T *__restrict__ Y = static_cast<T *>(a.y);
    const T *__restrict__ R = static_cast<const T *>(a.res);
    const int64_t G = gridDim.x;
    const int64_t rank = wg_rank(blockIdx.x, G);
    const int64_t end = sh.begin + sh.len;
    const int32_t Ho32 = (int32_t)a.Ho, Wo32 = (int32_t)a.Wo;
    const uint32_t nT32 = (uint32_t)a.nT;
    const __amdgpu_buffer_rsrc_t ry = __builtin_amdgcn_make_buffer_rsrc(Y, (short)0, (int)a.y_bytes, 0x00020000);
    const __amdgpu_buffer_rsrc_t rr = __builtin_amdgcn_make_buffer_rsrc(const_cast<T *>(R), (short)0, (int)a.y_bytes, 0x00020000);

    const bool has_res = (a.epi.flags & EPI_RES) != 0;

    int64_t t = sh.begin + rank;
    if (t >= end) return;

    // P = 4: logical wave pw; P = 2: channel half pw, both row halves; P = 1: both, in rounds
    const int wn_mine = P == 4 ? (pw & 1) : (P == 2 ? pw : 0);

    const bool one_nt = nT32 == 1;
    // per-channel affine part of the epilogue folded into one multiply-add, v = acc * sc + sh (bias,
    // then batch norm), in LDS: once for all channels, or for one n tile at a time beyond AFFN
    const bool all_aff = nT32 * 64u <= (uint32_t)K_::AFFN;
    auto load_affine = [&](uint32_t c0, uint32_t count) {
        float *const aff = reinterpret_cast<float *>(smem_ + K_::AFF0);
        for (uint32_t i = tid; i < count; i += NT) {
            const int64_t c = c0 + i;
            float sc, shf;
            chan_affine(a.epi, c < a.Nc ? c : 0, sc, shf);
            aff[i] = sc;
            aff[K_::AFFN + i] = shf;
        }
    };

    const RwWalk walk(a, (uint32_t)G);
    const RwPatch<K_> stream(pw, lane);
    RwCursor cu = walk.at((uint32_t)t);
    // one n tile: weights and per-channel constants once for the workgroup's lifetime; several (1x1 only):
    // for each tile, the next tile's weights load with its patch
    op_t bw[NS], bw_next[KS == 1 ? NS : 1];
    if constexpr (P != 1) rw_load_weights<K_>(a, bw, cu.nt, wn_mine, lane);
    if (all_aff) load_affine(0u, nT32 * 64u);
    stream.issue(a, cu, lds0, pw);
    int iter = 0;
    for (; t < end; t += G, ++iter) {
        trace_tile(sh, t, iter);
        const int cur = iter & 1;
        // the patch of this tile (and, on the first tile, the weights) has landed, its loads all
        // older than the previous tile's stores; every wave is done with the other buffer
        if (P == 4 && iter > 0 && a.y_bytes != 0u) wait_and_meet<K_::NST>();
        else wait_and_meet<0>();
        const RwCursor nx = walk.advance(cu);
        if constexpr (KS == 1 && P != 1) {
            if (!one_nt && iter > 0) {
                // the weights loaded with this tile's patch (complete: waited above)
#pragma unroll
                for (int s = 0; s < NS; ++s) bw[s] = bw_next[s];
            }
        }
        if (t + G < end) {
            stream.issue(a, nx, lds0 + (uint32_t)((cur ^ 1) * BUF), pw);
            if constexpr (KS == 1 && P != 1)
                if (!one_nt) rw_load_weights<K_>(a, bw_next, nx.nt, wn_mine, lane);
        }

        const uint32_t tx = cu.tx, ty = cu.ty, img = cu.img, ntile = cu.nt;
        if (!all_aff) {
            load_affine(64u * ntile, 64u);
            __syncthreads();
        }
        cu = nx;
        const int32_t oy0 = (int32_t)ty * K_::TH, ox0 = (int32_t)tx * TW;
        const char *patch = smem_ + cur * BUF;
#pragma unroll
        for (int rd = 0; rd < ROUNDS; ++rd) {
            acc_t acc[SL][2];
            // logical wave lambda = (rd SL + sl) P + pw owns tile rows 2 wm, 2 wm + 1 and channel
            // half wn, with wm = lambda div 2 and wn = lambda mod 2
            const int wn = P == 1 ? (rd & 1) : wn_mine;
            if constexpr (P == 1) rw_load_weights<K_>(a, bw, ntile, wn, lane);
            const RwOperands<K_> pixels(patch, pw, rd, hx, xl);
            constexpr int LA = kRwAhead<K_>;
            op_t opnd[LA + 1][SL][2];
#pragma unroll
            for (int s = 0; s < LA && s < NS; ++s) pixels.fetch(s, opnd[s]);
#pragma unroll
            for (int s = 0; s < NS; ++s) {
                if (s + LA < NS) pixels.fetch(s + LA, opnd[(s + LA) % (LA + 1)]);
#pragma unroll
                for (int sl = 0; sl < SL; ++sl)
#pragma unroll
                    for (int i = 0; i < 2; ++i)
                        acc[sl][i] = MF::run(bw[s], opnd[s % (LA + 1)][sl][i], s == 0 ? acc_t{} : acc[sl][i]);
                __builtin_amdgcn_sched_barrier(0);
            }
            // ---- epilogue from registers: MFMA rows are channels and columns the tile row's pixels
#pragma unroll
            for (int sl = 0; sl < SL; ++sl) {
                const int wm = K_::row_half(pw, rd, sl);
                trace_wave(sh, t, 2 * wm + wn, pw, rd * SL + sl);
                acc_t out[2][1] = {{acc[sl][0]}, {acc[sl][1]}};
                const int nl = all_aff ? 64 * (int)ntile + 32 * wn : 32 * wn;
                const uint32_t n0 = all_aff ? 0u : 64u * ntile;
                auto row_of = [&](int b, int x, uint32_t &row) {
                    const int32_t oy = oy0 + 2 * wm + b, ox = ox0 + x;
                    row = (((uint32_t)img * (uint32_t)Ho32 + (uint32_t)oy) * (uint32_t)Wo32 + (uint32_t)ox) * (uint32_t)a.ldy;
                    return oy < Ho32 && ox < Wo32;
                };
                if (a.y_bytes != 0u) {
                    finish_tile<T, false>(a.epi, smem_ + K_::AFF0, K_::AFFN, nl, n0, (uint32_t)a.Nc, ry, rr, out, row_of);
                    continue;
                }
                // output rows that 16-byte pieces with 32-bit offsets do not cover: a lane's four channels
                // at a time, eight bytes at an element's alignment (1x1 of 16x112x112x24 to 63 channels
                // 29.2 us staged, 52.4 by element, 23.6 so)
                typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
                struct __attribute__((packed, aligned(2))) Loose8 { u32x2 u; };
                struct Quad { T e[4]; };
                const float *const aff = reinterpret_cast<const float *>(smem_ + K_::AFF0) + nl + 4 * hx;
                if (64 * (int64_t)ntile + 32 * wn >= a.Nc) continue;
                with_act(a.epi.act, [&](auto actc) {
                    constexpr int ACT = decltype(actc)::value;
#pragma unroll
                    for (int b = 0; b < 2; ++b) {
                        const int32_t oy = oy0 + 2 * wm + b, ox = ox0 + xl;
                        if (oy >= Ho32 || ox >= Wo32) continue;
                        const int64_t row = (((int64_t)img * a.Ho + oy) * a.Wo + ox) * a.ldy;
#pragma unroll
                        for (int q = 0; q < MF::NACC / 4; ++q) {
                            const int64_t n = 64 * (int64_t)ntile + 32 * wn + 4 * hx + 8 * q;
                            if (n >= a.Nc) break;
                            const int64_t off = row + n;
                            const bool whole = n + 4 <= a.Nc;
                            Quad o, r = {};
                            if (has_res) {
                                if (whole) r = __builtin_bit_cast(Quad, reinterpret_cast<const Loose8 *>(R + off)->u);
                                else
#pragma unroll
                                    for (int e = 0; e < 3; ++e)
                                        if (n + e < a.Nc) r.e[e] = R[off + e];
                            }
#pragma unroll
                            for (int e = 0; e < 4; ++e) {
                                const float v = out[b][0][4 * q + e] * aff[8 * q + e] + aff[K_::AFFN + 8 * q + e];
                                o.e[e] = TypeOps<T>::from_f(act_t<T, ACT>(has_res ? v + TypeOps<T>::to_f(r.e[e]) : v));
                            }
                            if (whole) reinterpret_cast<Loose8 *>(Y + off)->u = __builtin_bit_cast(u32x2, o);
                            else
#pragma unroll
                                for (int e = 0; e < 3; ++e)
                                    if (n + e < a.Nc) Y[off + e] = o.e[e];
                        }
                    }
                });
            }
        }
    }
    wait_vmcnt<0>();  // no load into LDS outlives the workgroup
}

template <class T, int C, int KS, int ST>
inline int rw_regs_table(const void *out[3], int *lds) {
    out[0] = reinterpret_cast<const void *>(&rw_regs_kernel<T, C, 1, KS, ST>);
    out[1] = reinterpret_cast<const void *>(&rw_regs_kernel<T, C, 2, KS, ST>);
    out[2] = reinterpret_cast<const void *>(&rw_regs_kernel<T, C, 4, KS, ST>);
    *lds = RwRegsKernel<T, C, 4, KS, ST>::LDS_BYTES;
    return 0;
}

// 3x3 stride 2 with C = 8, 1x1 with C in {16, 24, 32, 64}; -1 otherwise.
template <class T>
inline int rw_regs_table_c(int64_t ks, int64_t st, int64_t c, const void *out[3], int *lds) {
    if (ks == 3 && st == 2 && c == 8) return rw_regs_table<T, 8, 3, 2>(out, lds);
    if (ks != 1 || st != 1) return -1;
    switch (c) {
    case 16: return rw_regs_table<T, 16, 1, 1>(out, lds);
    case 24: return rw_regs_table<T, 24, 1, 1>(out, lds);
    case 32: return rw_regs_table<T, 32, 1, 1>(out, lds);
    case 64: return rw_regs_table<T, 64, 1, 1>(out, lds);
    default: return -1;
    }
}

}  // namespace miriam
