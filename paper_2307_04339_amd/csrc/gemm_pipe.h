// Pipelined contraction that keeps a whole tile in the registers of one wave per SIMD: products,
// strided batched products and convolutions whose K chunks lie inside one filter tap (any K for one
// tap, C a multiple of the chunk otherwise), fp16 / bf16, 16-byte rows, K-major operands (or, for one tap,
// the right one stored [k][n]).
//
// What bounded the 4-stage kernel it replaces for these (igemm_dma_kernel) was the serial chain per
// 128-byte K chunk: meet, issue the loads, read the operands from LDS, multiply.  Two workgroups per
// CU hid part of it; a 64x64 tile still spent 0.45 us per chunk on 0.05 us of MFMA.  Here the operand
// reads of a k-step go out between the MFMAs of earlier ones, across chunk boundaries, and so do the
// loads that refill the ring, one at a time; the workgroup meets once per chunk.  The next tile's
// first loads are issued under the current tile's epilogue, which stores from registers.
//
// LDS: a ring of S stages of one 128-byte K chunk (64 values) of the TM output rows' and the TN output
// columns' operand rows, XOR-swizzled as in igemm_dma.h.  LA is how many k-steps ahead operands are read:
// one where a k-step holds four or more MFMAs, three for the small tiles, whose k-steps are shorter than
// the LDS latency.  With LA = 1 the wait before the last k-step also covers the chunk's own LDS reads, so
// its stage is refilled at once; with LA = 3, where LDS operations stay outstanding over the meeting, the
// stage of the chunk before is, and the writer of the epilogue's parameters waits for its writes itself.
//
// MFMA rows are output columns (channels) and MFMA columns output rows, as in the patch kernel, so
// that the epilogue stores 16 bytes per lane without staging.
//
// What bounds it: the load path.  128x128 chunks of a K = 3072 product arrive at 34 bytes per clock and
// CU, 0.42 us a chunk on 0.21 us of MFMA; wider tiles need fewer bytes per flop but leave CUs idle on
// small products (the tile rule and its times are in ops.cpp).  By the counters of 4096x768x3072 the matrix
// cores are busy 44% of a wave's life, which waits for loads or LDS 37% of it.  That product takes 26 us
// (igemm_dma_kernel 32), 8192x4096x1024 bf16 77 us, 0.90 PFLOP/s (88).
//
// K order per output element (fixed, whatever the elastic configuration): chunks in order, k-steps
// in order.
#pragma once

#include "tile_regs.h"

namespace miriam {

template <class T, int TM, int TN, int WM, int P>
struct PipeKernel {
    typedef Mfma<T, 32> MF;
    static constexpr int WN = kLogicalWaves / WM;
    static constexpr int BP = TM / WM / 32, BC = TN / WN / 32;
    static constexpr int NT = kWave * P;
    static_assert(sizeof(T) == 2, "16-bit operands only");
    static constexpr int KT = 64;                         // K per chunk
    static constexpr int NK = 4;                          // k-steps per chunk: 32 bytes of each row
    // Smaller physical blocks: a wave holds SL logical waves at once and walks K once for all of them (SM
    // of them along the rows times SN along the columns); the remaining ones in further rounds, each of
    // which loads the whole tile's operands again.  One at a time 8x56x56x128->256 3x3/2 took 21.7 us in
    // blocks of 128 and 52.0 of 64; so 13.6 and 20.3 (17.8 and 39.1 by igemm_dma_kernel).  Sixteen blocks
    // are half of a wave's registers; with them 256x128 tiles spill, up to 165 registers in blocks of 64,
    // which still beats a second walk there (2048x2304x768 55.1 us against 70.2, in blocks of 128 25.6
    // against 24.8)
    static constexpr int MOST = P == 2 ? 8 : 16;           // MFMA blocks
    static constexpr int FIT = MOST / (BP * BC) >= 4 ? 4 : (MOST / (BP * BC) >= 2 ? 2 : 1);
    static constexpr int SL = kLogicalWaves / P < FIT ? kLogicalWaves / P : FIT;
    static constexpr int SN = P == 1 && WN == 2 && SL > 1 ? 2 : 1, SM = SL / SN;
    static constexpr int MSTEP = SN * P / WN > 0 ? SN * P / WN : 1;  // logical rows between a wave's row slots
    static constexpr int RB = SM * BP, CB = SN * BC;      // MFMA blocks of a physical wave
    static constexpr int NM = RB * CB, NOP = RB + CB;        // MFMAs and operand reads per k-step
    static constexpr int LA = NM >= 4 ? 1 : 3;            // k-steps read ahead
    static constexpr int NS = LA + 1;                     // operand sets
    static constexpr int STAGE = (TM + TN) * 128;
    // one workgroup per CU from 128x64 on, two below
    static constexpr int BUDGET = (STAGE >= 24 * 1024 ? 160 : 80) * 1024 - 7 * TN * 4;
    static constexpr int S_FIT = BUDGET / STAGE, S_MOST = S_FIT > 5 ? 5 : S_FIT;
    // with fewer than four waves per workgroup and one step read ahead, three stages if more workgroups then
    // share a CU (two stages gained no more of them but for 128x128, and there left the loads too little
    // time: 4096x768x3072 in blocks of 128 46.1 us against 34.0)
    static constexpr int LDS_CU = 160 * 1024;
    static constexpr int S = P < 4 && LA == 1 && LDS_CU / (3 * STAGE + 7 * TN * 4) > LDS_CU / (S_MOST * STAGE + 7 * TN * 4) ? 3 : S_MOST;
    static constexpr int NIA = TM / 8 / P, NIB = TN / 8 / P, NL = NIA + NIB;  // loads per wave and chunk
    static constexpr int AHEAD = LA == 1 ? S : S - 1;     // chunks in flight or resident after a refill
    static constexpr int RAW0 = S * STAGE, AFF0 = RAW0 + 5 * TN * 4;
    static constexpr int LDS_BYTES = AFF0 + 2 * TN * 4;
    static constexpr int ROUNDS = kLogicalWaves / P / SL;
    static constexpr int NST = BP * BC * 2;
    static constexpr int HEAD = (NL + NK - 1) / NK;       // loads of a refill under the k-step it starts at
    static constexpr int PRE = HEAD + (LA - 1) * (NL - HEAD) / (NK - 1);  // and by the end of its LA-th k-step
    static_assert(S >= (LA == 1 ? 2 : 3), "ring");
    static_assert(TM % (8 * P) == 0 && TN % (8 * P) == 0 && TN % 64 == 0, "load instructions must divide evenly");
    static constexpr int vm(int n) { return n < 63 ? n : 63; }
};

// TAPS: filters of more than one tap; without, one tap (products, 1x1 convolutions) and any K.
// NB: right operand stored [k][n] (attention's values).  A chunk's 64 k rows of 64 columns are staged
// as they lie, 128 bytes each with the halves of rows 2 and 3 of every four swapped, and
// ds_read_b64_tr_b16 turns four rows into four K values per lane, two reads per operand.
template <class T, int TM, int TN, int WM, int P, bool TAPS, bool NB>
__global__ __launch_bounds__(kWave * P, (P == 4 && PipeKernel<T, TM, TN, WM, P>::STAGE < 24 * 1024 ? 2 : 1)) void pipe_kernel(IgemmArgs a, Shard sh) {
    typedef PipeKernel<T, TM, TN, WM, P> K_;
    typedef typename K_::MF MF;
    typedef typename MF::acc_t acc_t;
    constexpr int WN = K_::WN, BP = K_::BP, BC = K_::BC, RB = K_::RB, CB = K_::CB, SL = K_::SL, NIA = K_::NIA, NIB = K_::NIB, NL = K_::NL, NK = K_::NK, LA = K_::LA;
    constexpr int NS = K_::NS, S = K_::S, NM = K_::NM, NOP = K_::NOP, HEAD = K_::HEAD, PRE = K_::PRE, AHEAD = K_::AHEAD;
    constexpr int ROUNDS = K_::ROUNDS, NST = K_::NST, ES = 2, KT = K_::KT, VEC = 8;
    static_assert(!NB || (TN == 64 && !TAPS), "[k][n] operands: 64 columns, one tap");
    constexpr bool PIPE = P == 4 && LA == 1;  // next tile's first loads under the current epilogue

    __shared__ __attribute__((aligned(1024))) char smem_[K_::LDS_BYTES];
    const char *const smem = smem_;
    const uint32_t lds0 = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) char *)smem_;
    const int tid = threadIdx.x;
    const int pw = __builtin_amdgcn_readfirstlane(tid / kWave);
    const int lane = tid % kWave;
    const int hx = lane >> 5, xl = lane & 31;
    const rsrc_t rs_bias = make_rsrc(a.epi.bias, (uint32_t)a.epi.C * 4u), rs_bn = make_rsrc(a.epi.bn, (uint32_t)a.epi.C * 16u);
    const int64_t G = gridDim.x;
    const int64_t rank = wg_rank(blockIdx.x, G);
    const int64_t end = sh.begin + sh.len;
    const uint32_t M32 = (uint32_t)a.M, Nc32 = (uint32_t)a.Nc, Wo32 = (uint32_t)a.Wo, HoWo = (uint32_t)(a.Ho * a.Wo);
    const int32_t C32 = (int32_t)a.C, KW32 = a.KW, H32 = (int32_t)a.H, W32 = (int32_t)a.W, ldx32 = (int32_t)a.ldx;
    const int nch = (int)((a.K + KT - 1) / KT);
    const int lrow = lane >> 3;
    const int piece = (lane & 7) ^ ((lane >> 4) & 3);  // 16-byte piece this lane loads, but for bit 2 (see swz)

    // tile id = ((((b0 * bdiv + b1) * mgroups + mg) * nT + nt) * GM + mi: GM output-row tiles share a
    // column tile's operand rows before the next, so the tiles a die runs together form a block
    TileDigits<5> td;
    {
        const uint32_t radix[5] = {(uint32_t)a.tX, (uint32_t)a.nT, (uint32_t)a.tY, (uint32_t)a.bdiv, 0u};
        td.init((uint32_t)(sh.begin + rank), (uint32_t)G, radix);
    }

    // ---- the unit (tile, round) being loaded
    uint32_t voff_a[NIA], voff_b[NIB];
    int32_t row0[NIA], h0[NIA], w0[NIA];  // taps: element offset of tap (0, 0), first input row and column
    uint32_t m0 = 0, n0 = 0;
    uint64_t xbase = 0, wbase = 0;        // operands of the batch entry
    int64_t yoff = 0;
    int32_t ur = 0, us = 0, uc = 0;       // tap and channel base of the next chunk to load
    uint32_t kb = 0;                      // its byte offset within the weight rows
    int lch = 0;                          // and its number
    auto place_tap = [&]() __attribute__((always_inline)) {
        const int32_t toff = (ur * W32 + us) * ldx32;
        static_for<NIA>([&](auto j_) {
            constexpr int j = decltype(j_)::value;
            const bool ok = ((uint32_t)(h0[j] + ur) < (uint32_t)H32) & ((uint32_t)(w0[j] + us) < (uint32_t)W32);
            voff_a[j] = ok ? (uint32_t)(row0[j] + toff) * (uint32_t)ES : kOutOfRange;
        });
    };
    // rows 8 q .. 8 q + 7 of load q: row = 8 q + lrow, swizzle (row >> 1) & 7 = (4 q + (lrow >> 1)) & 7
    auto swz = [&](int q) __attribute__((always_inline)) { return (uint32_t)((piece ^ ((q & 1) << 2)) * VEC); };
    auto decode = [&](const TileDigits<5> &d) __attribute__((always_inline)) {
        m0 = (d.d[2] * (uint32_t)a.tX + d.d[0]) * (uint32_t)TM;
        n0 = d.d[1] * (uint32_t)TN;
        const int64_t b0 = d.d[4], b1 = d.d[3];
        xbase = (uint64_t)(uintptr_t)(static_cast<const T *>(a.x) + b0 * a.sx0 + b1 * a.sx1);
        wbase = (uint64_t)(uintptr_t)(static_cast<const T *>(a.w) + b0 * a.sw0 + b1 * a.sw1);
        yoff = b0 * a.sy0 + b1 * a.sy1;
        ur = us = uc = 0;
        kb = 0;
        lch = 0;
        static_for<NIB>([&](auto j_) {
            constexpr int j = decltype(j_)::value;
            const int q = j * P + pw;
            if constexpr (NB) {
                const uint32_t n = n0 + (uint32_t)(((lane & 7) ^ ((lrow << 1) & 4)) * VEC);
                voff_b[j] = n < Nc32 ? ((uint32_t)(8 * q + lrow) * (uint32_t)a.ldw + n) * (uint32_t)ES : kOutOfRange;
            } else {
                const uint32_t n = n0 + (uint32_t)(8 * q + lrow);
                voff_b[j] = n < Nc32 ? (n * (uint32_t)a.ldw + swz(q)) * (uint32_t)ES : kOutOfRange;
            }
        });
        static_for<NIA>([&](auto j_) {
            constexpr int j = decltype(j_)::value;
            const int q = j * P + pw;
            const uint32_t m = m0 + (uint32_t)(8 * q + lrow), mm = m < M32 ? m : 0u;
            const uint32_t img = fdiv(mm, a.fd_howo), pq = mm - img * HoWo;
            const uint32_t p = fdiv(pq, a.fd_wo), x = pq - p * Wo32;
            const int32_t h = (int32_t)p * a.stride - a.pad, w = (int32_t)x * a.stride - a.pad;
            const int32_t row = (int32_t)(img * (uint32_t)a.img_x) + (h * W32 + w) * ldx32 + (int32_t)swz(q);
            if constexpr (TAPS) {
                h0[j] = m < M32 ? h : -0x40000000;  // outside for every tap
                w0[j] = w;
                row0[j] = row;
            } else {
                const bool ok = (m < M32) & ((uint32_t)h < (uint32_t)H32) & ((uint32_t)w < (uint32_t)W32);
                voff_a[j] = ok ? (uint32_t)row * (uint32_t)ES : kOutOfRange;
            }
        });
        if constexpr (TAPS) place_tap();
    };
    // load u of chunk lch (the rows' loads, then the columns'); dst: its stage
    auto load1 = [&](auto u_, uint32_t dst) __attribute__((always_inline)) {
        constexpr int u = decltype(u_)::value;
        // past the last chunk: no bytes, reads zeros, so every chunk issues the same count
        const rsrc_t rs = make_rsrc(reinterpret_cast<const void *>(u < NIA ? xbase : wbase), lch < nch ? (u < NIA ? a.x_bytes : a.w_bytes) : 0u);
        if constexpr (u < NIA) buf_dma16(voff_a[u], rs, (uint32_t)uc * (uint32_t)ES, dst + (uint32_t)((u * P + pw) * 1024));
        else buf_dma16(voff_b[u - NIA], rs, kb, dst + (uint32_t)(TM * 128 + ((u - NIA) * P + pw) * 1024));
    };
    // one tap, the last chunk partial: pieces past K read zeros on both sides
    auto mask_tail = [&]() __attribute__((always_inline)) {
        if (lch == nch - 1 && nch * KT > C32) {
            static_for<NIA>([&](auto j_) {
                constexpr int j = decltype(j_)::value;
                voff_a[j] = uc + (int32_t)swz(j * P + pw) < C32 ? voff_a[j] : kOutOfRange;
            });
            static_for<NIB>([&](auto j_) {
                constexpr int j = decltype(j_)::value;
                const int32_t k = NB ? 8 * (j * P + pw) + lrow : (int32_t)swz(j * P + pw);
                voff_b[j] = uc + k < C32 ? voff_b[j] : kOutOfRange;
            });
        }
    };
    // on to the next chunk
    auto advance = [&]() __attribute__((always_inline)) {
        ++lch;
        kb += NB ? (uint32_t)(KT * ES) * (uint32_t)a.ldw : 128u;
        uc += KT;
        if constexpr (TAPS) {
            if (uc == C32) {
                uc = 0;
                if (++us == KW32) {
                    us = 0;
                    ++ur;
                }
                place_tap();
            }
        } else {
            mask_tail();
        }
    };
    auto stage_of = [&](int slot) __attribute__((always_inline)) { return lds0 + (uint32_t)(slot * K_::STAGE); };
    // first loads of a unit: epilogue parameters, then AHEAD chunks, of the last one only what
    // precedes the first chunk's share of that refill
    auto prologue = [&]() __attribute__((always_inline)) {
        if (pw == 0) load_channel_params<TN>(a.epi, rs_bias, rs_bn, n0, lane, lds0 + (uint32_t)K_::RAW0);
        if constexpr (!TAPS) mask_tail();
        static_for<AHEAD - 1>([&](auto c) {
            static_for<NL>([&](auto u) { load1(u, stage_of(decltype(c)::value)); });
            advance();
        });
        static_for<PRE>([&](auto u) { load1(u, stage_of(AHEAD - 1)); });
    };

    int64_t t = sh.begin + rank;
    if (t >= end) return;
    bool loaded = false;
    for (int iter = 0; t < end; t += G, ++iter) {
        trace_tile(sh, t, iter);
#pragma unroll 1
        for (int rd = 0; rd < ROUNDS; ++rd) {
            acc_t acc[RB][CB];
            if (!loaded) {
                decode(td);
                if ((PIPE ? 0 : iter) + rd > 0) wait_and_meet<0>();  // every wave is done with the ring and the parameters
                prologue();
                wait_and_meet<K_::vm((AHEAD - 2) * NL + PRE)>();
            } else {
                // the previous tile's stores were issued after this tile's first loads
                wait_and_meet<K_::vm((AHEAD - 2) * NL + PRE + (PIPE ? NST : 0))>();
            }
            loaded = false;
            const uint32_t tm0 = m0, tn0 = n0;
            const int64_t tyoff = yoff;
            const int lam = rd * SL * P + pw, wm = lam / WN, wn = lam % WN;  // the round's first slot
#pragma unroll
            for (int b = 0; b < RB; ++b)
#pragma unroll
                for (int c = 0; c < CB; ++c) acc[b][c] = acc_t{};

            // operand addresses: row r of a stage at 128 r, piece 2 kk + hx at slot ^ ((r >> 1) & 7); block
            // offsets are multiples of 32 rows and leave the swizzle alone
            u32x4 xo[NS][RB], wo[NS][CB];
            const uint32_t sw = (uint32_t)(hx ^ ((xl >> 1) & 7)) << 4;
            const uint32_t abase = (uint32_t)(wm * (TM / WM) + xl) * 128u + sw;
            const uint32_t bbase = (uint32_t)(TM + wn * (TN / WN) + xl) * 128u + sw;
            // NB: lane l of a group of 16 reads 8 bytes of k row (l & 15) / 4 (+ 8 for the upper half), at
            // column 4 (l & 3) of its group's 16; column block i flips bit 6 together with the row swizzle
            const uint32_t nbase = (uint32_t)(TM * 128) + (uint32_t)(8 * hx + ((lane >> 2) & 3)) * 128u +
                                   ((uint32_t)((((lane >> 3) & 1) << 2) ^ (wn * (TN / WN) / 8) ^ (((lane >> 3) & 2) | ((lane >> 1) & 1))) << 4) +
                                   (uint32_t)(lane & 1) * 8u;
            // row of the tile, from the wave's first, at which row block b starts
            auto block_row = [](int b) __attribute__((always_inline)) { return (b / BP) * K_::MSTEP * (TM / WM) + (b % BP) * 32; };
            // operand i (column blocks, then row blocks) of k-step kk of the stage at byte st
            auto fetch1 = [&](int i, int kk, uint32_t st, int set) __attribute__((always_inline)) {
                if constexpr (NB) {
                    if (i < CB) {
                        typedef short s16x4 __attribute__((ext_vector_type(4)));
                        typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
                        const uint32_t at = lds0 + (nbase ^ (uint32_t)(i << 6)) + st + (uint32_t)(kk * 2048);
#pragma unroll
                        for (int r = 0; r < 2; ++r) {
                            const u32x2 v = __builtin_bit_cast(
                                u32x2, __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) s16x4 *)(at + (uint32_t)(r * 512))));
                            wo[set][i][2 * r] = v[0];
                            wo[set][i][2 * r + 1] = v[1];
                        }
                        return;
                    }
                }
                if (i < CB) wo[set][i] = *reinterpret_cast<const u32x4 *>(smem + ((bbase ^ (uint32_t)(kk << 5)) + st + i * 4096));
                else xo[set][i - CB] = *reinterpret_cast<const u32x4 *>(smem + ((abase ^ (uint32_t)(kk << 5)) + st + block_row(i - CB) * 128));
            };
            static_for<LA>([&](auto k) {
                static_for<NOP>([&](auto i) { fetch1(decltype(i)::value, decltype(k)::value, 0u, decltype(k)::value); });
            });
            if (rd == 0) {
                make_affine(a.epi, smem_ + K_::RAW0, smem_ + K_::AFF0, TN, tid, K_::NT);
                // With LA = 3 the meetings of the chunk loop leave LDS operations outstanding; for a
                // single chunk the first of them is all that stands between this write and the other
                // waves' epilogue.  LA = 1: every meeting waits for them.
                if constexpr (LA > 1) wait_lds();
            }
            __builtin_amdgcn_sched_barrier(0);
            int slot = 0;                                        // stage of the current chunk
            uint32_t refill = stage_of(AHEAD - 1);               // stage the loads in progress go to
            for (int ch = 0; ch < nch; ++ch) {
                const int slot1 = slot + 1 < S ? slot + 1 : 0;
                uint32_t st = (uint32_t)(slot * K_::STAGE), st1 = (uint32_t)(slot1 * K_::STAGE);
                static_for<NK>([&](auto j_) {
                    constexpr int j = decltype(j_)::value;
                    constexpr int JB = NK - LA;  // k-step that first reads the next chunk
                    if constexpr (j == JB) {
                        // the refill in progress is complete; the next chunk has arrived
                        advance();
                        if constexpr (LA == 1) {
                            wait_and_meet<K_::vm((S - 2) * NL)>();
                            refill = stage_of(slot);
                        } else {
                            wait_and_meet_loads<K_::vm((S - 3) * NL)>();
                            refill = stage_of(slot > 0 ? slot - 1 : S - 1);
                        }
                    }
                    static_for<NM>([&](auto i_) {
                        constexpr int i = decltype(i_)::value, b = i / CB, c = i % CB;
                        acc[b][c] = MF::run(__builtin_bit_cast(typename MF::op_t, wo[j % NS][c]),
                                            __builtin_bit_cast(typename MF::op_t, xo[j % NS][b]), acc[b][c]);
                        // this MFMA's share of the operand reads LA k-steps ahead
                        static_for<NOP>([&](auto q_) {
                            constexpr int q = decltype(q_)::value;
                            if constexpr (q * (NM > 1 ? NM - 1 : 1) / NOP == i || (NM == 1 && i == 0))
                                fetch1(q, (j + LA) % NK, j + LA < NK ? st : st1, (j + LA) % NS);
                        });
                        // and of the refill: its head after the meeting, the rest over the k-steps to the next
                        constexpr int js = (j - JB + NK) % NK;   // k-steps since the meeting
                        if constexpr (js == 0) {
                            static_for<HEAD>([&](auto u) {
                                if constexpr (decltype(u)::value * NM / HEAD == i) load1(u, refill);
                            });
                        } else {
                            constexpr int w = (js - 1) * NM + i, W = (NK - 1) * NM;
                            constexpr int u0 = HEAD + w * (NL - HEAD) / W, u1 = HEAD + (w + 1) * (NL - HEAD) / W;
                            static_for<u1 - u0>([&](auto u) { load1(ActTag<u0 + decltype(u)::value>{}, refill); });
                        }
                        __builtin_amdgcn_sched_barrier(0);
                    });
                });
                slot = slot1;
            }
            if constexpr (PIPE) {
                if (t + G < end) {
                    // every wave is past the last meeting: this tile's LDS data has been read
                    TileDigits<5> nx = td;
                    nx.advance();
                    decode(nx);
                    prologue();
                    loaded = true;
                }
            }
            // ---- epilogue
#pragma unroll
            for (int sl = 0; sl < SL; ++sl) trace_wave(sh, t, lam + sl * P, pw, rd * SL + sl);
            const __amdgpu_buffer_rsrc_t ry = __builtin_amdgcn_make_buffer_rsrc(static_cast<T *>(a.y) + tyoff, (short)0, (int)a.y_bytes, 0x00020000);
            const __amdgpu_buffer_rsrc_t rr =
                __builtin_amdgcn_make_buffer_rsrc(static_cast<T *>(const_cast<void *>(a.res)) + tyoff, (short)0, (int)a.y_bytes, 0x00020000);
            finish_tile<T>(a.epi, smem + K_::AFF0, TN, wn * (TN / WN), tn0, Nc32, ry, rr, acc, [&](int b, int x, uint32_t &row) {
                const uint32_t m = tm0 + (uint32_t)(wm * (TM / WM) + block_row(b) + x);
                row = m * (uint32_t)a.ldy;
                return m < M32;
            });
        }
        td.advance();
    }
    wait_vmcnt<0>();  // no load into LDS outlives the workgroup
}

template <class T, int TM, int TN, int WM, bool TAPS, bool NB = false>
inline void pipe_table(const void *out[3], int *lds) {
    out[0] = reinterpret_cast<const void *>(&pipe_kernel<T, TM, TN, WM, 1, TAPS, NB>);
    out[1] = reinterpret_cast<const void *>(&pipe_kernel<T, TM, TN, WM, 2, TAPS, NB>);
    out[2] = reinterpret_cast<const void *>(&pipe_kernel<T, TM, TN, WM, 4, TAPS, NB>);
    *lds = PipeKernel<T, TM, TN, WM, 4>::LDS_BYTES;
}

// Right operand stored [k][n].
template <class T>
inline int pipe_nb_table_cfg(int cfg, const void *out[3], int *lds) {
    switch (cfg) {
    case CFG_PIPE_64: pipe_table<T, 64, 64, 2, false, true>(out, lds); return 0;
    case CFG_PIPE_128x64: pipe_table<T, 128, 64, 4, false, true>(out, lds); return 0;
    case CFG_PIPE_256x64: pipe_table<T, 256, 64, 4, false, true>(out, lds); return 0;
    default: return -1;
    }
}

template <class T, bool TAPS>
inline int pipe_table_cfg(int cfg, const void *out[3], int *lds) {
    switch (cfg) {
    case CFG_PIPE_64: pipe_table<T, 64, 64, 2, TAPS>(out, lds); return 0;
    case CFG_PIPE_128x64: pipe_table<T, 128, 64, 4, TAPS>(out, lds); return 0;
    case CFG_PIPE_128: pipe_table<T, 128, 128, 2, TAPS>(out, lds); return 0;
    case CFG_PIPE_256x128: pipe_table<T, 256, 128, 2, TAPS>(out, lds); return 0;
    case CFG_PIPE_256x192:
        if constexpr (TAPS) return -1;
        else pipe_table<T, 256, 192, 2, false>(out, lds);
        return 0;
    default: return -1;
    }
}

}  // namespace miriam
