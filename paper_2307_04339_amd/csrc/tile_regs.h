// Building blocks of the contraction kernels that keep the whole tile in registers (one wave per
// SIMD): compile-time loops, the barrier that orders their LDS-DMA pipelines, and an epilogue that
// stores straight from the accumulators.
#pragma once

#include <utility>

#include "igemm_dma.h"

namespace miriam {

typedef float f32x2 __attribute__((ext_vector_type(2)));

// f(0), f(1), ..., f(N - 1) with compile-time indices (ActTag<i>).
template <class F, int... I>
__device__ __attribute__((always_inline)) inline void static_for_(F &&f, std::integer_sequence<int, I...>) {
    (f(ActTag<I>{}), ...);
}
template <int N, class F>
__device__ __attribute__((always_inline)) inline void static_for(F &&f) {
    static_for_(f, std::make_integer_sequence<int, N>{});
}

// One 4-byte-per-lane buffer -> LDS load (lane i writes LDS bytes [lds + 4 i, + 4)), ordered like lds_dma16.
__device__ __forceinline__ void buf_dma4(uint32_t voff, rsrc_t rsrc, uint32_t lds_addr) {
    const uint32_t lds = __builtin_amdgcn_readfirstlane(lds_addr);
    asm volatile("s_mov_b32 m0, %2\n\ts_nop 0\n\tbuffer_load_dword %0, %1, 0 offen lds"
                 :
                 : "v"(voff), "s"(rsrc), "s"(lds)
                 : "memory", "m0");
}

// Wait until at most N vector-memory operations and no LDS reads of this wave are outstanding,
// then meet the workgroup.
template <int N>
__device__ __forceinline__ void wait_and_meet() {
    asm volatile("" ::: "memory");
    __builtin_amdgcn_s_waitcnt((N & 15) | ((N >> 4) << 14) | (7 << 4) | (0 << 8));
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
}

// The same without waiting for this wave's LDS reads.
template <int N>
__device__ __forceinline__ void wait_and_meet_loads() {
    asm volatile("" ::: "memory");
    wait_vmcnt<N>();
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
}

// Wait for this wave's LDS operations.
__device__ __forceinline__ void wait_lds() {
    asm volatile("" ::: "memory");
    __builtin_amdgcn_s_waitcnt((63 & 15) | ((63 >> 4) << 14) | (7 << 4) | (0 << 8));
    asm volatile("" ::: "memory");
}

// Raw epilogue parameters of TN channels from n0 into LDS at `lds` (bias, gamma, beta, mean, var,
// TN floats each), by one wave; ordered like lds_dma16.
template <int TN>
__device__ __forceinline__ void load_channel_params(const Epilogue &e, rsrc_t rs_bias, rsrc_t rs_bn, uint32_t n0, int lane, uint32_t lds) {
#pragma unroll
    for (int j = 0; j < TN / 64; ++j) {
        const uint32_t v = (n0 + (uint32_t)(64 * j + lane)) * 4u;
        if (e.flags & EPI_BIAS) buf_dma4(v, rs_bias, lds + (uint32_t)(256 * j));
        if (e.flags & EPI_BN)
#pragma unroll
            for (int k = 0; k < 4; ++k)
                buf_dma4(v + (uint32_t)k * (uint32_t)e.C * 4u, rs_bn, lds + (uint32_t)((k + 1) * TN * 4 + 256 * j));
    }
}

// Per-channel affine part (bias, then batch norm; scales, then shifts) from the raw parameters, both in LDS.
__device__ __forceinline__ void make_affine(const Epilogue &e, const char *raw0, char *aff0, int TN, int tid, int nt) {
    for (int c = tid; c < TN; c += nt) {
        const float *raw = reinterpret_cast<const float *>(raw0) + c;
        const float bias = (e.flags & EPI_BIAS) ? raw[0] : 0.0f;
        float sc = 1.0f, shf = bias;
        if (e.flags & EPI_BN) {
            sc = raw[TN] / sqrtf(raw[4 * TN] + e.eps);
            shf = (bias - raw[3 * TN]) * sc + raw[2 * TN];
        }
        float *aff = reinterpret_cast<float *>(aff0);
        aff[c] = sc;
        aff[TN + c] = shf;
    }
}

// Lanes 16..31 and 48..63 of a change places with lanes 0..15 and 32..47 of b.
__device__ __forceinline__ void exchange16(u32x4 &a, u32x4 &b) {
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        const auto sw = __builtin_amdgcn_permlane16_swap(a[k], b[k], false, false);
        a[k] = sw[0];
        b[k] = sw[1];
    }
}

// Epilogue of a wave's BP x BC blocks from registers: v = acc * sc + sh (+ residual), activation, one
// rounding, 16-byte stores.  Accumulator rows are output channels and columns output rows m: lane
// (hx, xl) of block (b, c) holds channels 8 q + 4 hx .. + 3 of quarter q for row xl of the block;
// row_of(b, x, row) places row x (in elements; false if outside).  A v_permlane32_swap
// per packed pair gives lanes 0..31 channels 16 h .. + 7 and lanes 32..63 16 h + 8 .. + 15, whole
// 16-byte pieces, and a v_permlane16_swap of the h = 0 and h = 1 pieces puts the four pieces of a
// row into one store: 64 contiguous bytes per row (32 without it: 96 x 512 x 512 x 64 products, all
// stores, 23.8 us at 256x128 against 22.9 for LDS-staged whole rows).  Every wave issues the same
// stores; pieces outside take an offset past the buffer.
// KEEP: a column block's scales and shifts stay in registers for all its row blocks; without it they are
// read with each quarter (a kernel that has no 32 registers to spare).
template <class T, bool KEEP = true, class Acc, int BP, int BC, class Rows>
__device__ __forceinline__ void finish_tile(const Epilogue &e, const char *aff0, int TN, int nl0, uint32_t n0, uint32_t Nc,
                                            __amdgpu_buffer_rsrc_t ry, __amdgpu_buffer_rsrc_t rr, Acc (&acc)[BP][BC], Rows &&row_of) {
    static_assert(sizeof(T) == 2, "16-bit results only");
    const int lane = threadIdx.x % kWave, hx = lane >> 5;
    auto finish = [&](auto actc, auto resc) {
        constexpr int ACT = decltype(actc)::value;
        constexpr bool RES = decltype(resc)::value != 0;
#pragma unroll
        for (int c = 0; c < BC; ++c) {
            const int nl = nl0 + c * 32;
            const float *aff = reinterpret_cast<const float *>(aff0) + nl + 4 * hx;
            f32x4 sc[4], shf[4];
            auto affine = [&](int g) {
                sc[g] = *reinterpret_cast<const f32x4 *>(aff + 8 * g);
                shf[g] = *reinterpret_cast<const f32x4 *>(aff + TN + 8 * g);
            };
            if constexpr (KEEP) {
#pragma unroll
                for (int g = 0; g < 4; ++g) affine(g);
            }
#pragma unroll
            for (int b = 0; b < BP; ++b) {
                // stored piece of this lane: channels 8 pc .. + 7 of rows (lane & 15) and 16 + (lane & 15)
                const int pc = ((lane >> 5) & 1) | ((lane >> 3) & 2);
                const uint32_t n = n0 + (uint32_t)(nl + 8 * pc);
                uint32_t off[2];
#pragma unroll
                for (int h = 0; h < 2; ++h) {
                    uint32_t row;
                    const bool in = row_of(b, 16 * h + (lane & 15), row);
                    off[h] = in & (n < Nc) ? (row + n) * 2u : kOutOfRange;
                }
                u32x4 o[2], r[2];
                if constexpr (RES) {
#pragma unroll
                    for (int h = 0; h < 2; ++h) r[h] = __builtin_bit_cast(u32x4, __builtin_amdgcn_raw_buffer_load_b128(rr, (int)off[h], 0, 0));
                    exchange16(r[0], r[1]);
                }
#pragma unroll
                for (int h = 0; h < 2; ++h) {  // channels 16 h .. 16 h + 15 of the block, quarters 2 h and 2 h + 1
                    uint32_t q[2][2], rq[2][2];
#pragma unroll
                    for (int k = 0; k < 2; ++k) {
                        if constexpr (RES) {
                            const auto sw = __builtin_amdgcn_permlane32_swap(r[h][k], r[h][2 + k], false, false);
                            rq[0][k] = sw[0];
                            rq[1][k] = sw[1];
                        }
                    }
#pragma unroll
                    for (int w = 0; w < 2; ++w) {
                        if constexpr (!KEEP) affine(2 * h + w);
#pragma unroll
                        for (int k = 0; k < 2; ++k) {
                            f32x2 v2;
#pragma unroll
                            for (int u = 0; u < 2; ++u) {
                                const int g = 2 * h + w;
                                float v = acc[b][c][4 * g + 2 * k + u] * sc[g][2 * k + u] + shf[g][2 * k + u];
                                if constexpr (RES)
                                    v += TypeOps<T>::to_f(__builtin_bit_cast(T, (uint16_t)(u ? rq[w][k] >> 16 : rq[w][k] & 0xffffu)));
                                v2[u] = act_t<T, ACT>(v);
                            }
                            typedef T t2 __attribute__((ext_vector_type(2)));
                            q[w][k] = __builtin_bit_cast(uint32_t, __builtin_convertvector(v2, t2));
                        }
                    }
#pragma unroll
                    for (int k = 0; k < 2; ++k) {
                        const auto sw = __builtin_amdgcn_permlane32_swap(q[0][k], q[1][k], false, false);
                        o[h][k] = sw[0];
                        o[h][2 + k] = sw[1];
                    }
                }
                exchange16(o[0], o[1]);
#pragma unroll
                for (int h = 0; h < 2; ++h) __builtin_amdgcn_raw_buffer_store_b128(o[h], ry, (int)off[h], 0, 0);
            }
        }
    };
    if (e.flags & EPI_RES) with_act(e.act, [&](auto actc) { finish(actc, ActTag<1>{}); });
    else with_act(e.act, [&](auto actc) { finish(actc, ActTag<0>{}); });
}

}  // namespace miriam
