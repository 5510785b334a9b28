// Direct 3x3 stride-1 convolution with the weights resident in registers, for narrow layers (fp16 / bf16,
// C in {8, 16, 32, 64}, at most 64 output channels).  3x3 stride 2 on 8-channel images and 1x1 are in
// conv_rw_regs.h; tile, patch stream, weights, K order and elastic blocks of both in conv_rw_tile.h.
//
// There is one n tile, so a workgroup loads its weights once and keeps them across every tile it runs.
// The finished tile is staged through LDS, over the patch buffer it has been read from where one round
// suffices, and stored in whole pixel rows.
#pragma once

#include "conv_rw_tile.h"

namespace miriam {

template <class T, int C, int P>
struct RwKernel : RwTile<T, C, P, 3, 1> {
    typedef RwTile<T, C, P, 3, 1> Tile;
    using Tile::TM;
    using Tile::TN;
    using Tile::PATCH;
    using Tile::ROUNDS;
    static constexpr int LDC = TN + 4;                     // staged fp32 row (residual epilogue)
    static constexpr int LDY = TN + 8;                     // staged output row in elements
    static constexpr int CS = TM * LDC * 4;
    // single round: the staged tile overlays the patch buffer the tile has finished with
    static constexpr bool OVERLAY = ROUNDS == 1;
    static constexpr int BUF = OVERLAY ? (PATCH > CS ? PATCH : CS) : PATCH;
    static constexpr int LDS_BYTES = 2 * BUF + (OVERLAY ? 0 : CS);
    static constexpr int WAVES_PER_SIMD = (P == 4 && 2 * (LDS_BYTES + 16) <= 160 * 1024) ? 2 : 1;
    static_assert(TM * LDY * 2 <= CS, "staged output fits the staging area");
};

template <class T, int C, int P>
__global__ __launch_bounds__(kWave * P, (RwKernel<T, C, P>::WAVES_PER_SIMD)) void rw_conv_kernel(IgemmArgs a, Shard sh) {
    typedef RwKernel<T, C, P> K_;
    typedef typename K_::MF MF;
    typedef typename K_::op_t op_t;
    typedef typename K_::acc_t acc_t;
    constexpr int TW = K_::TW, TM = K_::TM, TN = K_::TN, NT = K_::NT, VEC = K_::VEC, NS = K_::NS, SL = K_::SL, ROUNDS = K_::ROUNDS;
    constexpr int LDC = K_::LDC, LDY = K_::LDY, BUF = K_::BUF;

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
    const bool has_res = (a.epi.flags & EPI_RES) != 0;

    int64_t t = sh.begin + rank;
    if (t >= end) return;

    // P = 4: logical wave pw; P = 2: channel half pw, both row halves; P = 1: both, in rounds
    const int wn_mine = P == 4 ? (pw & 1) : (P == 2 ? pw : 0);

    // per-channel affine part of the epilogue folded into one multiply-add, v = acc * sc + sh,
    // for this lane's channel in each round (bias, then batch norm)
    float esc[ROUNDS], esh[ROUNDS];
    auto load_affine = [&](uint32_t nt) {
#pragma unroll
        for (int rd = 0; rd < ROUNDS; ++rd) {
            const int wn = P == 1 ? (rd & 1) : wn_mine;
            const int64_t col = 64 * (int64_t)nt + 32 * wn + xl;
            chan_affine(a.epi, col < a.Nc ? col : 0, esc[rd], esh[rd]);
        }
    };

    const RwWalk walk(a, (uint32_t)G);
    const RwPatch<K_> stream(pw, lane);
    RwCursor cu = walk.at((uint32_t)t);
    // weights and per-channel constants once for the workgroup's lifetime
    op_t bw[NS];
    if constexpr (P != 1) rw_load_weights<K_>(a, bw, cu.nt, wn_mine, lane);
    load_affine(cu.nt);
    stream.issue(a, cu, lds0, pw);
    int iter = 0;
    for (; t < end; t += G, ++iter) {
        trace_tile(sh, t, iter);
        const int cur = iter & 1;
        // the patch of this tile (and, on the first tile, the weights) has landed; every wave
        // is done with the other buffer (the previous tile's staged outputs)
        wait_vmcnt<0>();
        __syncthreads();
        const RwCursor nx = walk.advance(cu);
        if (t + G < end) stream.issue(a, nx, lds0 + (uint32_t)((cur ^ 1) * BUF), pw);

        const uint32_t tx = cu.tx, ty = cu.ty, img = cu.img, ntile = cu.nt;
        cu = nx;
        const int32_t oy0 = (int32_t)ty * K_::TH, ox0 = (int32_t)tx * TW;
        const char *patch = smem_ + cur * BUF;
        char *const stage = smem_ + (K_::OVERLAY ? cur * BUF : 2 * BUF);
        float *const Cs = reinterpret_cast<float *>(stage);
        T *const Ys = reinterpret_cast<T *>(stage);

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
                        acc[sl][i] = MF::run(opnd[s % (LA + 1)][sl][i], bw[s], s == 0 ? acc_t{} : acc[sl][i]);
                __builtin_amdgcn_sched_barrier(0);
            }
            // ---- epilogue, stage 1: v = acc * sc + sh per channel; without a residual the
            // activation and the one rounding happen here and the tile is staged in the output
            // type, otherwise it is staged as fp32 (tile row y, column x -> staged row y * TW + x)
            if constexpr (K_::OVERLAY) __syncthreads();  // every wave is done reading this patch
            const int col = 32 * wn + xl;
#pragma unroll
            for (int sl = 0; sl < SL; ++sl)
                trace_wave(sh, t, 2 * K_::row_half(pw, rd, sl) + wn, pw, rd * SL + sl);
            auto stage1 = [&](auto actc) {
                constexpr int ACT = decltype(actc)::value;
#pragma unroll
                for (int sl = 0; sl < SL; ++sl) {
                    const int wm = K_::row_half(pw, rd, sl);
#pragma unroll
                    for (int i = 0; i < 2; ++i) {
                        // element e of the block sits at tile column x = 8 (e / 4) + 4 hx + e % 4
                        const int row0 = (2 * wm + i) * TW + hx * 4;
                        float *const cb = Cs + row0 * LDC + col;
                        T *const yb = Ys + row0 * LDY + col;
#pragma unroll
                        for (int e = 0; e < MF::NACC; ++e) {
                            const int dx = (e / 4) * 8 + (e % 4);
                            const float v = acc[sl][i][e] * esc[rd] + esh[rd];
                            if constexpr (ACT < 0) cb[dx * LDC] = v;
                            else yb[dx * LDY] = TypeOps<T>::from_f(act_t<T, ACT>(v));
                        }
                    }
                }
            };
            if (has_res) stage1(ActTag<-1>{});
            else with_act(a.epi.act, stage1);
        }
        __syncthreads();
        // ---- stage 2: 16-byte stores of whole pixel rows (with a residual: + residual,
        // activation and the rounding first)
        constexpr int RV = TN / VEC;
        auto stage2_res = [&](auto actc) {
            constexpr int ACT = decltype(actc)::value;
#pragma unroll 1
            for (int idx = tid; idx < TM * RV; idx += NT) {
                const int row = idx / RV, cv = idx - (idx / RV) * RV;
                const int32_t oy = oy0 + row / TW, ox = ox0 + row % TW;
                const int64_t n = 64 * (int64_t)ntile + (int64_t)cv * VEC;
                if (oy >= Ho32 || ox >= Wo32 || n >= a.Nc) continue;
                const int64_t off = (((int64_t)img * a.Ho + oy) * a.Wo + ox) * a.ldy + n;
                const float *cr = Cs + row * LDC + cv * VEC;
                if (a.vec_store && n + VEC <= a.Nc) {
                    const Vec16<T> rv = ld_vec(R + off);
                    Vec16<T> o;
#pragma unroll
                    for (int e = 0; e < VEC; ++e) o.e[e] = TypeOps<T>::from_f(act_t<T, ACT>(cr[e] + TypeOps<T>::to_f(rv.e[e])));
                    st_vec(Y + off, o);
                } else {
#pragma unroll
                    for (int e = 0; e < VEC; ++e)
                        if (n + e < a.Nc) st_f(Y + off + e, act_t<T, ACT>(cr[e] + ld_f(R + off + e)));
                }
            }
        };
        if (has_res) {
            with_act(a.epi.act, stage2_res);
            continue;
        }
        if (a.y_bytes != 0u) {
            // whole 16-byte pieces and an output of less than 2^31 bytes: buffer stores with
            // 32-bit offsets, pieces outside the output written to an offset past the buffer
            // (dropped), no branch per piece
            static_assert((TM * RV) % NT == 0 && RV == 8 && TW == 32, "stage 2 piece decode");
            const __amdgpu_buffer_rsrc_t ry = __builtin_amdgcn_make_buffer_rsrc(Y, (short)0, (int)a.y_bytes, 0x00020000);
            // (unsigned arithmetic: the offset of a piece outside the output may wrap; it is
            // replaced before use)
            const uint32_t orow0 = ((uint32_t)img * (uint32_t)Ho32 + (uint32_t)oy0) * (uint32_t)Wo32 + (uint32_t)ox0;
            const uint32_t ldyb = (uint32_t)a.ldy * (uint32_t)sizeof(T);
#pragma unroll
            for (int it = 0; it < TM * RV / NT; ++it) {
                const int idx = tid + it * NT;
                const int row = idx >> 3, cv = idx & 7;
                const int32_t oy = oy0 + (row >> 5), ox = ox0 + (row & 31);
                const uint32_t n = 64u * ntile + (uint32_t)(cv * VEC);
                const bool ok = oy < Ho32 && ox < Wo32 && n < (uint32_t)a.Nc;
                const uint32_t off = (orow0 + (uint32_t)(row >> 5) * (uint32_t)Wo32 + (uint32_t)(row & 31)) * ldyb +
                                     n * (uint32_t)sizeof(T);
                const u32x4 v = *reinterpret_cast<const u32x4 *>(Ys + row * LDY + cv * VEC);
                __builtin_amdgcn_raw_buffer_store_b128(v, ry, (int)(ok ? off : kOutOfRange), 0, 0);
            }
            continue;
        }
#pragma unroll 1
        for (int idx = tid; idx < TM * RV; idx += NT) {
            const int row = idx / RV, cv = idx - (idx / RV) * RV;
            const int32_t oy = oy0 + row / TW, ox = ox0 + row % TW;
            const int64_t n = 64 * (int64_t)ntile + (int64_t)cv * VEC;
            if (oy >= Ho32 || ox >= Wo32 || n >= a.Nc) continue;
            const int64_t off = (((int64_t)img * a.Ho + oy) * a.Wo + ox) * a.ldy + n;
            Vec16<T> o;
            {
                o.u = *reinterpret_cast<const u32x4 *>(Ys + row * LDY + cv * VEC);
                if (a.vec_store && n + VEC <= a.Nc) {
                    st_vec(Y + off, o);
                } else {
#pragma unroll
                    for (int e = 0; e < VEC; ++e)
                        if (n + e < a.Nc) Y[off + e] = o.e[e];
                }
            }
        }
    }
}

template <class T, int C>
inline int rw_table(const void *out[3], int *lds) {
    out[0] = reinterpret_cast<const void *>(&rw_conv_kernel<T, C, 1>);
    out[1] = reinterpret_cast<const void *>(&rw_conv_kernel<T, C, 2>);
    out[2] = reinterpret_cast<const void *>(&rw_conv_kernel<T, C, 4>);
    *lds = RwKernel<T, C, 4>::LDS_BYTES;
    return 0;
}

// Kernel table for 3x3 stride 1 with C in {8, 16, 32, 64}; -1 otherwise.
template <class T>
inline int rw_table_c(int64_t c, const void *out[3], int *lds) {
    switch (c) {
    case 8: return rw_table<T, 8>(out, lds);
    case 16: return rw_table<T, 16>(out, lds);
    case 32: return rw_table<T, 32>(out, lds);
    case 64: return rw_table<T, 64>(out, lds);
    default: return -1;
    }
}

}  // namespace miriam
