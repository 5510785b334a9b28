// Direct convolution with the weights resident in registers and the epilogue from registers, for
// 3x3 stride 2 on 8-channel images and 1x1 stride 1 (fp16 / bf16).  Tile, wave split, patch stream,
// weights, K order and elastic blocks are those of conv_rw.h.
//
// With the weights as the MFMA's row operand a lane ends up with four adjacent output channels of one
// pixel, so the tile is finished and stored from registers.  Staged through LDS these layers spent two
// barriers and a pass over LDS on a tile of 1 to 5 K steps and had LDS for two workgroups per CU instead
// of three (1x1 of 16x56x56x24 to 144 channels 12.4 to 9.6 us, 3x3 stride 2 of 16x224x224x8 to 32
// channels 16.5 to 10.6).  3x3 stride 1 stays staged: at C = 64 the 144 weight registers leave none for
// this epilogue (conv1_2 of VGG-16 b8 44.8 against 42.4 us), and from memory the whole 128-byte rows
// matter more than the barriers (conv1_1 to pool1 of VGG-16 b8 on buffers in turn 71.2 against 70.3 us).
#pragma once

#include "conv_rw.h"
#include "tile_regs.h"

namespace miriam {

template <class T, int C, int P, int KS, int ST>
struct RwRegsKernel {
    typedef Mfma<T, 32> MF;
    static_assert(sizeof(T) == 2, "16-bit operands only");
    static_assert(C % 8 == 0 && C >= 8 && C <= 64, "C must be a multiple of 8 up to 64");
    // two MFMA operand halves share one tap unless one tap holds a single half (C = 8)
    static_assert(KS == 1 || C == 8 || C % 16 == 0, "3x3 needs C = 8 or a multiple of 16");
    static_assert((KS == 3 && ST == 2) || (KS == 1 && ST == 1), "3x3 stride 2, 1x1 stride 1");
    static constexpr int TH = 4, TW = 32, TM = TH * TW, TN = 64;
    static constexpr int NT = kWave * P;
    static constexpr int VEC = 8;                         // 16-bit elements per 16 bytes
    static constexpr int NP = C / 8;                      // 16-byte pieces of a pixel
    static constexpr int SP = NP % 2 == 1 ? NP : NP + 1;  // LDS slots per pixel (odd stride)
    static constexpr int PS = SP * 16;                    // LDS bytes per patch pixel
    static constexpr int PH = (TH - 1) * ST + KS, PW = (TW - 1) * ST + KS, PPIX = PH * PW;
    static constexpr int NSLOT = PPIX * SP;
    static constexpr int NINS = (NSLOT + kWave - 1) / kWave;  // DMA instructions per patch
    static constexpr int NJ = (NINS + P - 1) / P;             // per wave (the last may be idle)
    static constexpr int PATCH = NINS * kWave * 16;
    static constexpr int KTOT = KS * KS * C;
    static constexpr int NS = (KTOT + 15) / 16;            // MFMA k-steps of 16
    static constexpr int LW = kLogicalWaves / P;
    static constexpr int SL = P == 2 ? 2 : 1;              // logical waves held at once
    static constexpr int ROUNDS = LW / SL;
    static constexpr int AFFN = 512;                       // channels whose affine parameters LDS keeps for the launch
    static constexpr int AFF0 = 2 * PATCH;
    static constexpr int LDS_BYTES = AFF0 + 2 * AFFN * 4;
    static constexpr int NST = 4;                          // output stores per wave and tile (P = 4)
    static constexpr int WAVES_PER_SIMD = (P == 4 && 2 * (LDS_BYTES + 16) <= 160 * 1024) ? 2 : 1;
    static_assert(LW % SL == 0, "slots");
};

template <class T, int C, int P, int KS, int ST>
__global__ __launch_bounds__(kWave * P, (RwRegsKernel<T, C, P, KS, ST>::WAVES_PER_SIMD)) void rw_regs_kernel(IgemmArgs a,
                                                                                                     Shard sh) {
    typedef RwRegsKernel<T, C, P, KS, ST> K_;
    typedef typename K_::MF MF;
    typedef typename MF::op_t op_t;
    typedef typename MF::acc_t acc_t;
    constexpr int TW = K_::TW, TN = K_::TN, PW = K_::PW, PS = K_::PS, SP = K_::SP, NP = K_::NP;
    constexpr int NT = K_::NT, VEC = K_::VEC, NS = K_::NS, SL = K_::SL, ROUNDS = K_::ROUNDS;
    constexpr int KTOT = K_::KTOT, NJ = K_::NJ, NINS = K_::NINS, BUF = K_::PATCH;

    __shared__ __attribute__((aligned(1024))) char smem_[K_::LDS_BYTES];
    const uint32_t lds0 = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) char *)smem_;

    const int tid = threadIdx.x;
    const int pw = __builtin_amdgcn_readfirstlane(tid / kWave);
    const int lane = tid % kWave;
    const int hx = lane >> 5, xl = lane & 31;  // MFMA operand half, pixel column / channel
    const T *__restrict__ X = static_cast<const T *>(a.x);
    const T *__restrict__ Wt = static_cast<const T *>(a.w);
    T *__restrict__ Y = static_cast<T *>(a.y);
    const T *__restrict__ R = static_cast<const T *>(a.res);
    const int64_t G = gridDim.x;
    const int64_t rank = wg_rank(blockIdx.x, G);
    const int64_t end = sh.begin + sh.len;
    const int32_t H32 = (int32_t)a.H, W32 = (int32_t)a.W, Ho32 = (int32_t)a.Ho, Wo32 = (int32_t)a.Wo;
    const int32_t ldx32 = (int32_t)a.ldx;
    const uint32_t tX32 = (uint32_t)a.tX, tY32 = (uint32_t)a.tY, nT32 = (uint32_t)a.nT;
    const __amdgpu_buffer_rsrc_t ry = __builtin_amdgcn_make_buffer_rsrc(Y, (short)0, (int)a.y_bytes, 0x00020000);
    const __amdgpu_buffer_rsrc_t rr = __builtin_amdgcn_make_buffer_rsrc(const_cast<T *>(R), (short)0, (int)a.y_bytes, 0x00020000);

    const bool has_res = (a.epi.flags & EPI_RES) != 0;

    int64_t t = sh.begin + rank;
    if (t >= end) return;

    // weights of n tile nt, channel half wn: step s holds k = 16s + 8hx .. +7 of output
    // channel 64 nt + 32 wn + xl
    op_t bw[NS];
    auto load_weights = [&](op_t *dst, uint32_t nt, int wn) {
        const int64_t n = 64 * (int64_t)nt + 32 * wn + xl;
#pragma unroll
        for (int s = 0; s < NS; ++s) {
            const int k = 16 * s + 8 * hx;
            op_t v = op_t{};
            if (n < a.Nc && k < KTOT) v = *reinterpret_cast<const op_t *>(Wt + n * a.ldw + k);
            dst[s] = v;
        }
    };
    // P = 4: logical wave pw; P = 2: channel half pw, both row halves; P = 1: both, in rounds
    const int wn_mine = P == 4 ? (pw & 1) : (P == 2 ? pw : 0);

    // tile id = ((image * tY + tile row) * tX + tile column) * nT + n tile, kept as mixed-radix
    // digits that advance by the grid (no division per tile)
    struct Cursor {
        uint32_t img, ty, tx, nt;
    };
    const uint32_t g0 = (uint32_t)G;
    const uint32_t gn = g0 % nT32, g1 = g0 / nT32;
    const uint32_t gx = g1 % tX32, g2 = g1 / tX32;
    const uint32_t gy = g2 % tY32, gi = g2 / tY32;
    auto advance = [&](Cursor c) {
        c.nt += gn;
        const uint32_t cn = c.nt >= nT32 ? 1u : 0u;
        c.nt -= cn * nT32;
        c.tx += gx + cn;
        const uint32_t cx = c.tx >= tX32 ? 1u : 0u;
        c.tx -= cx * tX32;
        c.ty += gy + cx;
        const uint32_t cy = c.ty >= tY32 ? 1u : 0u;
        c.ty -= cy * tY32;
        c.img += gi + cy;
        return c;
    };
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

    // DMA of the patch of tile `c` into buffer `buf`: instruction j writes slots 64j .. 64j+63.
    // The slot a lane fills is the same in every tile, so its decode (patch row and column,
    // 16-byte piece, whether the slot holds data) is done once and kept packed in one register
    // per instruction: bits [0, 7) column, [7, 11) row, [11, 15) piece, bit 15 set for a data
    // slot.  Per tile a lane then only adds the tile's origin, checks the image bounds and
    // forms a 32-bit byte offset into the image (the library admits the kernel only for images
    // of less than 2^31 bytes); pixels outside the image and padding slots take an offset past
    // the buffer, which reads zeros.
    static_assert(K_::PW < 128 && K_::PH <= 16 && SP <= 16, "packed patch geometry");
    uint32_t geo[NJ];
#pragma unroll
    for (int jj = 0; jj < NJ; ++jj) {
        const int j = jj * P + pw;
        const int q = j * kWave + lane;
        const int pr = q / SP, sl = q - (q / SP) * SP;
        const int prow = pr / PW, pcol = pr - (pr / PW) * PW;
        const bool ok = j < NINS && pr < K_::PPIX && sl < NP;
        geo[jj] = ok ? ((uint32_t)pcol | ((uint32_t)prow << 7) | ((uint32_t)sl << 11) | (1u << 15)) : 0u;
    }
    const uint32_t img_bytes = (uint32_t)(a.img_x * (int64_t)sizeof(T));
    auto issue_patch = [&](Cursor c, int buf) {
        const uint32_t tx = c.tx, ty = c.ty, img = c.img;
        const int32_t iy0 = (int32_t)ty * K_::TH * ST - a.pad, ix0 = (int32_t)tx * TW * ST - a.pad;
        const rsrc_t rs = make_rsrc(X + (int64_t)img * a.img_x, img_bytes);
        const uint32_t base = lds0 + (uint32_t)(buf * BUF);
#pragma unroll
        for (int jj = 0; jj < NJ; ++jj) {
            const int j = jj * P + pw;
            if (j < NINS) {
                uint32_t g = geo[jj];
                asm volatile("" : "+v"(g));  // unpacked here: hoisted out of the loop, the fields spilled
                const int32_t iy = iy0 + (int32_t)((g >> 7) & 15u), ix = ix0 + (int32_t)(g & 127u);
                const bool ok = (g >> 15) != 0u && (uint32_t)iy < (uint32_t)H32 && (uint32_t)ix < (uint32_t)W32;
                const uint32_t off = (uint32_t)((iy * W32 + ix) * ldx32 + (int32_t)((g >> 11) & 15u) * VEC) * (uint32_t)sizeof(T);
                buf_dma16(ok ? off : kOutOfRange, rs, 0u, base + (uint32_t)(j * kWave * 16));
            }
        }
    };

    Cursor cu;
    {
        const uint32_t t32 = (uint32_t)t, r1 = t32 / nT32, r2 = r1 / tX32;
        cu = Cursor{r2 / tY32, r2 % tY32, r1 % tX32, t32 % nT32};
    }
    // one n tile: weights and per-channel constants once for the workgroup's lifetime;
    // several (1x1 only): for each tile, the next tile's weights load with its patch
    op_t bw_next[KS == 1 ? NS : 1];
    if constexpr (P != 1) load_weights(bw, cu.nt, wn_mine);
    if (all_aff) load_affine(0u, nT32 * 64u);
    issue_patch(cu, 0);
    int iter = 0;
    for (; t < end; t += G, ++iter) {
        trace_tile(sh, t, iter);
        const int cur = iter & 1;
        // the patch of this tile (and, on the first tile, the weights) has landed, its loads all
        // older than the previous tile's stores; every wave is done with the other buffer
        if (P == 4 && iter > 0 && a.y_bytes != 0u) wait_and_meet<K_::NST>();
        else wait_and_meet<0>();
        const Cursor nx = advance(cu);
        if constexpr (KS == 1 && P != 1) {
            if (!one_nt && iter > 0) {
                // the weights loaded with this tile's patch (complete: waited above)
#pragma unroll
                for (int s = 0; s < NS; ++s) bw[s] = bw_next[s];
            }
        }
        if (t + G < end) {
            issue_patch(nx, cur ^ 1);
            if constexpr (KS == 1 && P != 1)
                if (!one_nt) load_weights(bw_next, nx.nt, wn_mine);
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
            if constexpr (P == 1) load_weights(bw, ntile, wn);
            // operand base of block i of slot sl: patch pixel (tile row y, column xl) + this lane's half
            const char *abase[SL][2];
#pragma unroll
            for (int sl = 0; sl < SL; ++sl) {
                const int wm = P == 4 ? (pw >> 1) : (P == 2 ? sl : (rd >> 1));
#pragma unroll
                for (int i = 0; i < 2; ++i) {
                    const int y = 2 * wm + i;
                    abase[sl][i] = patch + (y * ST * PW + xl * ST) * PS + (NP == 1 ? 0 : hx * 16);
                }
            }
            // operands of k-step s for every block; one 8-channel tap per operand half (C = 8,
            // 3x3): halves take taps 2s and 2s+1
            auto fetch = [&](int s, op_t (&av)[SL][2]) {
#pragma unroll
                for (int sl = 0; sl < SL; ++sl)
#pragma unroll
                    for (int i = 0; i < 2; ++i) {
                        if constexpr (NP == 1 && KS == 3) {
                            const int t0 = 2 * s, t1 = 2 * s + 1;
                            const int off0 = rw_toff<PW, KS>(t0) * PS;
                            const int d1 = t1 < 9 ? (rw_toff<PW, KS>(t1) - rw_toff<PW, KS>(t0)) * PS : PS;
                            op_t v = *reinterpret_cast<const op_t *>(abase[sl][i] + off0 + hx * d1);
                            if (16 * s + 8 * hx >= KTOT) v = op_t{};
                            av[sl][i] = v;
                        } else {
                            // both halves in one tap (channels c0 .. c0 + 15); 1x1: the one tap
                            const int k0 = 16 * s, tap = KS == 1 ? 0 : k0 / C, c0 = KS == 1 ? k0 : k0 % C;
                            const int off = rw_toff<PW, KS>(tap) * PS + (c0 / 8) * 16;
                            op_t v = *reinterpret_cast<const op_t *>(abase[sl][i] + off);
                            if (KTOT % 16 != 0 && 16 * s + 8 * hx >= KTOT) v = op_t{};
                            av[sl][i] = v;
                        }
                    }
            };
            // Software pipeline in program order: the operand reads of step s + LA are issued
            // before the MFMAs of step s, and a scheduling fence after each step keeps the
            // compiler from sinking the reads next to their use (it otherwise waited on every
            // read and ran each block's MFMAs as one dependent chain).  Within a step the
            // blocks' MFMAs are independent.
            constexpr int LA = SL == 1 ? 2 : 1;
            op_t opnd[LA + 1][SL][2];
#pragma unroll
            for (int s = 0; s < LA && s < NS; ++s) fetch(s, opnd[s]);
#pragma unroll
            for (int s = 0; s < NS; ++s) {
                if (s + LA < NS) fetch(s + LA, opnd[(s + LA) % (LA + 1)]);
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
                const int wm = P == 4 ? (pw >> 1) : (P == 2 ? sl : (rd >> 1));
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
