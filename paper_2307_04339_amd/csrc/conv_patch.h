// Pipelined 3x3 stride-1 convolution that keeps the tile's input pixels in LDS (fp16 / bf16,
// C a multiple of 32).
//
// An implicit GEMM on a 3x3 layer loads each input pixel nine times, once per filter tap, and
// at 128x128 outputs per tile that stream (64 bytes per clock and CU at the MFMA rate) is what
// bounds it: the load path of a CU carries about 28 bytes per clock on such rows.  Here the tile
// is TM consecutive output pixels (image, row, column order, across row and image ends) times TN
// output channels, and for each chunk of 32 input channels the pixels the nine taps touch are
// loaded once.  In the padded pixel space (every image Ho + 2 rows of PW = Wo + 2 pixels, zeros
// outside the image) they are one contiguous run: pixel m sits at lin(m) = (image (Ho + 2) + p)
// PW + q and tap (r, s) reads lin(m) + r PW + s, so the run of a tile is lin(last) - lin(first) +
// 2 PW + 3 pixels (338 for 256 pixels of a 28-wide image, 492 of a 112-wide one).  Only the
// weights stream per tap: about 20 bytes per clock at 256x128.
//
// LDS: two patch buffers of NPX pixels x 64 bytes (chunk cc + 1 loads while chunk cc is
// multiplied) and a ring of three weight stages; a stage holds the three taps of one filter row,
// TN x 64 bytes each.  Piece c (16 bytes) of a 64-byte row i sits at slot c ^ ((i >> 2) & 3), so
// the operand reads of 32 consecutive rows spread over all banks.
//
// A step is one (chunk, filter row): six MFMA k-steps of 16.  The operands of k-step j + 1 are
// read while the MFMAs of k-step j run, across step boundaries too: before the last k-step of a
// step a wave waits for its own loads of the next step and its LDS reads, the workgroup meets at
// one barrier; the loads that replace the data just consumed follow between the MFMAs.  The next
// tile's first loads are issued at the last barrier of the current one and land during its
// epilogue, which works from registers alone.
//
// MFMA rows are output channels and columns are pixels, so a lane ends with four consecutive
// channels of one pixel per accumulator quarter; one v_permlane32_swap per packed pair gives 16
// contiguous bytes per lane to store, with no LDS staging and no barrier.
//
// What bounds it and what it measured (fp16, back to back in a captured graph, against the implicit
// GEMM before): the MFMA rate of one wave per SIMD.  A step of 256x128 takes 0.97 us on the whole
// chip (0.64 at the nominal clock, 0.73 without its LDS reads, 0.87 without its loads), so the
// matrix cores are busy two thirds of the K loop; a launch adds about 8 us for the first loads,
// the parameter decode and the last epilogue.  By the counters of 8x112x112x128->128 they are busy
// half of a wave's life, and a wave waits for loads or LDS 27% of it.  8x112x112x128->128 41.1 -> 33.6 us,
// 8x56x56x256->256 36.7 -> 30.0, 8x28x28x512->512 44.5 -> 32.1, 8x112x112x64->128 29.5 -> 24.0.
// Issued in one run per k-step instead of one by one between the MFMAs, the operand reads and loads
// cost 0.08 us a step.
//
// K order per output element (fixed, whatever the elastic configuration): channel chunk of 32
// outer, tap (r, s) in row-major order, channel innermost.
#pragma once

#include "tile_regs.h"

namespace miriam {

template <class T, int TM, int TN, int WM, int P, int NPX>
struct PatchKernel {
    typedef Mfma<T, 32> MF;
    static_assert(sizeof(T) == 2, "16-bit operands only");
    static constexpr int WN = kLogicalWaves / WM;         // logical waves: WM along pixels, WN along channels
    static constexpr int BP = TM / WM / 32, BC = TN / WN / 32;  // MFMA blocks of a logical wave
    static constexpr int NT = kWave * P;
    // smaller physical blocks: a wave holds SL logical waves at once (16 MFMA blocks, half of its registers),
    // SM of them along the pixels times SN along the channels; the remaining ones in further rounds, each of
    // which loads the tile's operands again.  8x28x28x512->512 in blocks of 128 / 64: one at a time 52.1 / 119.7
    // us, eight blocks 44.0 / 91.2, sixteen (with up to 69 spills in blocks of 64) 44.1 / 81.6 (igemm_dma_kernel
    // 51.6 / 107.5)
    static constexpr int FIT = 16 / (BP * BC);
    static constexpr int SL = kLogicalWaves / P < FIT ? kLogicalWaves / P : FIT;
    static constexpr int SN = P == 1 && WN == 2 && SL > 1 ? 2 : 1, SM = SL / SN;
    static constexpr int MSTEP = SN * P / WN > 0 ? SN * P / WN : 1;  // logical rows between a wave's pixel slots
    static constexpr int RB = SM * BP, CB = SN * BC;      // MFMA blocks of a physical wave
    static constexpr int KC = 32;                         // channels per chunk (64-byte rows)
    static constexpr int PATCH = NPX * 64;
    static constexpr int NPW = NPX / 16 / P;              // patch loads per wave (16 pixels each)
    static constexpr int PART = (NPW + 2) / 3;            // of a third of a chunk
    static constexpr int RG = TN / 16 / P;                // weight row groups (16 rows) per wave and tap
    static constexpr int NB = 3 * RG;                     // weight loads per wave and step
    static constexpr int BSTAGE = 3 * TN * 64;
    static constexpr int W0 = 2 * PATCH;                  // LDS offsets: weights, raw parameters, affine
    static constexpr int RAW0 = W0 + 3 * BSTAGE;
    static constexpr int AFF0 = RAW0 + 5 * TN * 4;
    static constexpr int LDS_BYTES = AFF0 + 2 * TN * 4;
    static constexpr int ROUNDS = kLogicalWaves / P / SL;
    static constexpr int NST = BP * BC * 2;               // output stores per wave and tile
    static_assert(NPX % (16 * P) == 0 && TN % (16 * P) == 0, "load instructions must divide evenly");
    static_assert(NB + PART + (P == 4 ? NST : 0) < 64, "vmcnt range");
    static_assert(LDS_BYTES <= 160 * 1024, "LDS");
};

template <class T, int TM, int TN, int WM, int P, int NPX>
__global__ __launch_bounds__(kWave * P, 1) void patch_conv_kernel(IgemmArgs a, Shard sh) {
    typedef PatchKernel<T, TM, TN, WM, P, NPX> K_;
    typedef typename K_::MF MF;
    typedef typename MF::op_t op_t;
    typedef typename MF::acc_t acc_t;
    constexpr int WN = K_::WN, BP = K_::BP, RB = K_::RB, CB = K_::CB, SL = K_::SL, NPW = K_::NPW, PART = K_::PART, RG = K_::RG, NB = K_::NB;
    constexpr int NST = K_::NST, ROUNDS = K_::ROUNDS;
    constexpr int NM = RB * CB, NOP = RB + CB;            // MFMAs and operand reads per k-step
    constexpr int NL = PART + NB, HEAD = PART < NM ? PART : NM;  // loads per step; of them under its last k-step

    __shared__ __attribute__((aligned(1024))) char smem_[K_::LDS_BYTES];
    const char *const smem = smem_;
    const uint32_t lds0 = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) char *)smem_;
    const int tid = threadIdx.x;
    const int pw = __builtin_amdgcn_readfirstlane(tid / kWave);
    const int lane = tid % kWave;
    const int hx = lane >> 5, xl = lane & 31;
    const rsrc_t rs_x = make_rsrc(a.x, a.x_bytes), rs_w = make_rsrc(a.w, a.w_bytes);
    const rsrc_t rs_bias = make_rsrc(a.epi.bias, (uint32_t)a.epi.C * 4u), rs_bn = make_rsrc(a.epi.bn, (uint32_t)a.epi.C * 16u);
    const __amdgpu_buffer_rsrc_t ry = __builtin_amdgcn_make_buffer_rsrc(a.y, (short)0, (int)a.y_bytes, 0x00020000);
    const __amdgpu_buffer_rsrc_t rr = __builtin_amdgcn_make_buffer_rsrc(const_cast<void *>(a.res), (short)0, (int)a.y_bytes, 0x00020000);
    const int64_t G = gridDim.x;
    const int64_t rank = wg_rank(blockIdx.x, G);
    const int64_t end = sh.begin + sh.len;
    const uint32_t Nc32 = (uint32_t)a.Nc;
    const uint32_t Wo32 = (uint32_t)a.Wo, Ho2 = (uint32_t)a.Ho + 2u, PW = Wo32 + 2u, HoWo = (uint32_t)(a.Ho * a.Wo);
    const uint32_t H32 = (uint32_t)a.H, W32 = (uint32_t)a.W, ldx32 = (uint32_t)a.ldx, C32 = (uint32_t)a.C;
    const int CC = (int)(a.C / K_::KC);
    const int piece_ = (lane & 3) ^ ((lane >> 4) & 3);  // 16-byte piece this lane loads into its slot

    // tile id = (group * mT + mt) * nT + nt; ids below 2^31 (checked at creation).  A group is the
    // whole batch, or one image where a tile that spans two would need too many pixels; its last
    // tile may be partial.
    const uint32_t group = (uint32_t)a.sx0;  // output pixels per group
    TileDigits<3> td;
    {
        const uint32_t radix[3] = {(uint32_t)a.nT, (uint32_t)a.mT, 0u};
        td.init((uint32_t)(sh.begin + rank), (uint32_t)G, radix);
    }
    // padded-space position of output pixel m
    auto lin_of = [&](uint32_t m) -> uint32_t {
        const uint32_t img = fdiv(m, a.fd_howo), pq = m - img * HoWo;
        const uint32_t p = fdiv(pq, a.fd_wo), q = pq - p * Wo32;
        return (img * Ho2 + p) * PW + q;
    };

    // ---- the unit (tile, round) being loaded
    uint32_t voff_p[NPW];   // byte offset of this lane's piece of each patch load, channel 0 (or out of range)
    uint32_t voff_w[RG];    // byte offset of this lane's piece of each weight row group, tap 0, channel 0
    uint32_t pxb[RB];       // LDS row of each block's operand pixel for tap (0, 0), with this lane's half
    uint32_t m0 = 0, n0 = 0, mlast = 0;  // first pixel and channel, last pixel
    // pixel of the tile, from the wave's first, at which block b starts
    auto block_row = [](int b) { return (b / BP) * K_::MSTEP * (TM / WM) + (b % BP) * 32; };
    auto decode = [&](const TileDigits<3> &d, int rd) {
        const uint32_t g0 = d.d[2] * group;
        m0 = g0 + d.d[1] * (uint32_t)TM;
        n0 = d.d[0] * (uint32_t)TN;
        const uint32_t last = (m0 + TM <= g0 + group ? m0 + TM : g0 + group) - 1;
        mlast = last;
        const uint32_t L0 = __builtin_amdgcn_readfirstlane(lin_of(m0));
        const uint32_t span = __builtin_amdgcn_readfirstlane(lin_of(last)) - L0 + 2u * PW + 3u;
#pragma unroll
        for (int j = 0; j < NPW; ++j) {
            const uint32_t i = (uint32_t)(16 * (j * P + pw) + (lane >> 2)), lin = L0 + i;
            const uint32_t g = fdiv(lin, a.fd_pw), col = lin - g * PW;
            const uint32_t img = fdiv(g, a.fd_ph), pr = g - img * Ho2;
            const uint32_t h = pr - (uint32_t)a.pad, w = col - (uint32_t)a.pad;
            const bool ok = (i < span) & (h < H32) & (w < W32);
            voff_p[j] = ok ? (((img * H32 + h) * W32 + w) * ldx32 + (uint32_t)piece_ * 8u) * 2u : kOutOfRange;
        }
#pragma unroll
        for (int j = 0; j < RG; ++j) {
            const uint32_t n = n0 + (uint32_t)(16 * (j * P + pw) + (lane >> 2));
            voff_w[j] = n < Nc32 ? (n * (uint32_t)a.ldw + (uint32_t)piece_ * 8u) * 2u : kOutOfRange;
        }
        const int wm = (rd * SL * P + pw) / WN;
#pragma unroll
        for (int b = 0; b < RB; ++b) {
            const uint32_t m = m0 + (uint32_t)(wm * (TM / WM) + block_row(b) + xl);
            pxb[b] = ((lin_of(m <= last ? m : last) - L0) << 6) | ((uint32_t)hx << 4);
        }
    };
    // Loads past the last chunk go out all the same, through a descriptor of no bytes (they
    // read zeros into a free buffer), so every step issues the same count and waits for the same.
    auto only_if = [](rsrc_t rs, bool on) {
        rs[2] = on ? rs[2] : 0;
        return rs;
    };
    // patch loads [j0, j1) of channel chunk ch
    auto issue_patch = [&](rsrc_t rs, int ch, int j0, int j1) {
        const uint32_t base = lds0 + (uint32_t)((ch & 1) * K_::PATCH);
        const uint32_t soff = (uint32_t)ch * 64u;
#pragma unroll
        for (int j = 0; j < NPW; ++j)
            if (j >= j0 && j < j1) buf_dma16(voff_p[j], rs, soff, base + (uint32_t)((j * P + pw) * 1024));
    };
    // weight load q (tap q / RG, row group q % RG) of filter row r, channel chunk ch
    auto issue_w1 = [&](rsrc_t rs, int ch, int r, int q) {
        const int tap = q / RG, rg = q % RG;
        const uint32_t soff = ((uint32_t)(r * 3 + tap) * C32 + (uint32_t)ch * 32u) * 2u;
        buf_dma16(voff_w[rg], rs, soff,
                  lds0 + (uint32_t)(K_::W0 + r * K_::BSTAGE + tap * TN * 64 + (rg * P + pw) * 1024));
    };
    auto issue_w = [&](int ch, int r) {
#pragma unroll
        for (int q = 0; q < NB; ++q) issue_w1(rs_w, ch, r, q);
    };
    // load u of the group that replaces step (chunk, filter row r): a third of the patch of channel
    // chunk pch, then weight row r of chunk wch
    auto replace = [&](int pch, int wch, int r, int u) {
        const int j = ((r + 1) % 3) * PART + u;
        if (u >= PART) issue_w1(only_if(rs_w, wch < CC), wch, r, u - PART);
        else if (j < NPW) issue_patch(only_if(rs_x, pch < CC), pch, j, j + 1);
    };
    // first loads of a unit: epilogue parameters, chunk 0 of the patch, the weights of its first
    // two filter rows, and the head of the group that the first step completes (a third of chunk 1,
    // the third filter row)
    auto prologue = [&]() {
        if (pw == 0) load_channel_params<TN>(a.epi, rs_bias, rs_bn, n0, lane, lds0 + (uint32_t)K_::RAW0);
        issue_patch(rs_x, 0, 0, NPW);
        issue_w(0, 0);
        issue_w(0, 1);
#pragma unroll
        for (int u = 0; u < HEAD; ++u) replace(1, 0, 2, u);
    };
    constexpr bool pipe = P == 4;  // next tile's first loads under the current epilogue
    int64_t t = sh.begin + rank;
    if (t >= end) return;
    bool loaded = false;
    for (int iter = 0; t < end; t += G, ++iter) {
        trace_tile(sh, t, iter);
        uint32_t tm0 = 0, tn0 = 0, tlast = 0;

        // ---- epilogue of round rd from registers: v = acc * sc + sh, + residual, activation,
        // one rounding, 16-byte stores
        auto epilogue = [&](int rd, acc_t (&acc)[RB][CB]) {
            const int lam = rd * SL * P + pw, wm = lam / WN, wn = lam % WN;  // the round's first slot
#pragma unroll
            for (int sl = 0; sl < SL; ++sl) trace_wave(sh, t, lam + sl * P, pw, rd * SL + sl);
            finish_tile<T>(a.epi, smem + K_::AFF0, TN, wn * (TN / WN), tn0, Nc32, ry, rr, acc, [&](int b, int x, uint32_t &row) {
                const uint32_t m = tm0 + (uint32_t)(wm * (TM / WM) + block_row(b) + x);
                row = m * (uint32_t)a.ldy;
                return m <= tlast;
            });
        };

#pragma unroll 1
        for (int rd = 0; rd < ROUNDS; ++rd) {
            acc_t acc[RB][CB];
            if (!loaded) {
                decode(td, rd);
                prologue();
                wait_and_meet<NB + HEAD>();
            } else {
                // the previous tile's stores were issued after this tile's first loads
                wait_and_meet<NB + HEAD + (P == 4 ? NST : 0)>();
            }
            loaded = false;
            tm0 = m0;
            tn0 = n0;
            tlast = mlast;
            const int wn = (rd * SL * P + pw) % WN;
#pragma unroll
            for (int b = 0; b < RB; ++b)
#pragma unroll
                for (int c = 0; c < CB; ++c) acc[b][c] = acc_t{};

            op_t xo[2][RB], wo[2][CB];
            // LDS addresses of the pixels of a tap: row px at 64 px, piece hx (the halves of a k-step
            // pair differ in bit 5) swizzled by px bits 2 and 3.  Taps of a filter row take the sets
            // 0, 1, 2 in turn; the next tap's are computed under the MFMAs of the current one.
            uint32_t ad[3][RB];
            const uint32_t hx4 = (uint32_t)hx << 4;
            const uint32_t wbase = (uint32_t)K_::W0 + (uint32_t)(wn * (TN / WN) + xl) * 64u + (hx4 ^ ((uint32_t)(xl << 2) & 0x30u));
            auto tap_offset = [&](int r, int s, uint32_t pb) -> uint32_t { return pb + (((uint32_t)r * PW + (uint32_t)s) << 6); };
            auto address1 = [&](int b, int set, uint32_t toff) {
                const uint32_t row = pxb[b] + toff;
                ad[set][b] = row ^ ((row >> 4) & 0x30u);
            };

            // operand i of half kk of tap (r, s): the channel blocks, then the pixel blocks (at
            // the tap's addresses)
            auto fetch1 = [&](int i, int r, int s, int kk, int set) {
                if (i < CB)
                    wo[set][i] = *reinterpret_cast<const op_t *>(smem + (wbase ^ (uint32_t)(kk << 5)) + r * K_::BSTAGE + s * TN * 64 + i * 2048);
                else
                    xo[set][i - CB] = *reinterpret_cast<const op_t *>(smem + (ad[s][i - CB] ^ (uint32_t)(kk << 5)));
            };

#pragma unroll
            for (int b = 0; b < RB; ++b) address1(b, 0, tap_offset(0, 0, 0u));
            static_for<NOP>([&](auto i) { fetch1(decltype(i)::value, 0, 0, 0, 0); });
            if (rd == 0) make_affine(a.epi, smem_ + K_::RAW0, smem_ + K_::AFF0, TN, tid, K_::NT);
            __builtin_amdgcn_sched_barrier(0);
            for (int cc = 0; cc < CC; ++cc) {
                const uint32_t pb = (uint32_t)((cc & 1) * K_::PATCH);
                static_for<18>([&](auto step) {
                    constexpr int r = decltype(step)::value / 6, j = decltype(step)::value % 6;
                    constexpr int r1 = r == 2 ? 0 : r + 1;  // filter row of the next step
                    constexpr int r0 = r == 0 ? 2 : r - 1;  // and of the one before
                    const uint32_t pb1 = r == 2 ? pb ^ (uint32_t)K_::PATCH : pb;
                    // at the last k-step of a step the next step's data must be there: all but the
                    // newest weight stage
                    if constexpr (j == 5) wait_and_meet<NB>();
                    // One MFMA at a time, each followed by its share of the next k-step's operand
                    // reads, of the next tap's addresses and of the loads that replace the data of
                    // the last finished step: issued in one run, any of these left the matrix core
                    // idle meanwhile.
                    uint32_t toff = 0;
                    if constexpr (j % 2 == 0) {
                        toff = j == 4 ? tap_offset(r1, 0, pb1) : tap_offset(r, j / 2 + 1, pb);
                        asm volatile("" : "+s"(toff));  // or all nine taps' addresses would be kept in registers
                    }
                    static_for<NM>([&](auto i_) {
                        constexpr int i = decltype(i_)::value, b = i / CB, c = i % CB;
                        acc[b][c] = MF::run(wo[j & 1][c], xo[j & 1][b], acc[b][c]);
                        static_for<NOP>([&](auto q_) {
                            constexpr int q = decltype(q_)::value;
                            if constexpr (q * (NM - 1) / NOP == i) {
                                if constexpr (j == 5) fetch1(q, r1, 0, 0, 0);
                                else fetch1(q, r, (j + 1) / 2, (j + 1) % 2, (j + 1) & 1);
                            }
                        });
                        if constexpr (j % 2 == 0)
                            static_for<RB>([&](auto b_) {
                                if constexpr (decltype(b_)::value * NM / RB == i) address1(decltype(b_)::value, (j / 2 + 1) % 3, toff);
                            });
                        if constexpr (j == 5) {
                            if constexpr (i < HEAD) replace(r == 2 ? cc + 2 : cc + 1, cc + 1, r, i);
                        } else {
                            constexpr int u0 = HEAD + ((j * NM + i) * (NL - HEAD)) / (5 * NM),
                                          u1 = HEAD + ((j * NM + i + 1) * (NL - HEAD)) / (5 * NM);
                            static_for<u1 - u0>([&](auto u) {
                                replace(cc + 1, r == 0 ? cc : cc + 1, r0, u0 + decltype(u)::value);
                            });
                        }
                        __builtin_amdgcn_sched_barrier(0);
                    });
                });
            }
            if (pipe && t + G < end) {
                // every wave is past the last barrier: this tile's LDS data has been read
                TileDigits<3> nx = td;
                nx.advance();
                decode(nx, 0);
                prologue();
                loaded = true;
            }
            epilogue(rd, acc);
        }
        td.advance();
    }
    wait_vmcnt<0>();  // no load into LDS outlives the workgroup
}

template <class T, int TM, int TN, int WM, int NPX>
inline void patch_table(const void *out[3], int *lds) {
    out[0] = reinterpret_cast<const void *>(&patch_conv_kernel<T, TM, TN, WM, 1, NPX>);
    out[1] = reinterpret_cast<const void *>(&patch_conv_kernel<T, TM, TN, WM, 2, NPX>);
    out[2] = reinterpret_cast<const void *>(&patch_conv_kernel<T, TM, TN, WM, 4, NPX>);
    *lds = PatchKernel<T, TM, TN, WM, 4, NPX>::LDS_BYTES;
}

template <class T>
inline int patch_table_cfg(int cfg, const void *out[3], int *lds) {
    switch (cfg) {
    case CFG_PATCH_128: patch_table<T, 256, 128, 2, kPatchPixels>(out, lds); return 0;
    case CFG_PATCH_64: patch_table<T, 256, 64, 4, kPatchPixels>(out, lds); return 0;
    case CFG_PATCH_64W: patch_table<T, 256, 64, 4, kPatchPixelsW>(out, lds); return 0;
    default: return -1;
    }
}

}  // namespace miriam
