// What the two direct convolutions with resident weights (conv_rw.h, conv_rw_regs.h) share: the tile and
// its walk, the input patch's stream into LDS, the weights' layout and the K loop.
//
// The tile is 4 x 32 output pixels of one image times 64 output channels (for 3x3 stride 1 the tile of the
// LDS-patch kernel, so the tile space, the shard plans and the tile map are the same), split 2 x 2 over
// the 4 logical waves; logical wave (wm, wn) owns tile rows 2wm, 2wm+1 and output channels 32wn .. 32wn+31
// of the tile's 64.  Tile id = ((image * tY + tile row) * tX + tile column) * nT + n tile.
//
// With at most 64 input channels the whole filter slice of a logical wave, 32 channels x KS*KS*C K values,
// fits its registers as MFMA operands (9C/4 VGPRs for 3x3: 144 for C = 64).  Only the input patch of a
// tile, the ((4-1) ST + KS) x ((32-1) ST + KS) pixels its taps touch, streams through LDS: it is DMA'd
// (buffer loads of 16 bytes per lane) into one of two buffers while the previous tile computes.  A pixel
// occupies C/8 16-byte slots, padded to an odd count, so the pixels of a tap map to distinct bank groups
// and every MFMA operand read is a ds_read_b128 with a compile-time offset.
//
// K order per output element (fixed, whatever the elastic configuration): MFMA step s covers
// k = 16s .. 16s+15 with k = tap * C + c (tap = KS r + s in row-major order, c fastest), the order of the
// [Cout][KH][KW][Cin] weight rows; when KS*KS*C is not a multiple of 16 the last step's upper half is zero
// on both operands.
//
// Elastic block: a physical block of P waves runs logical wave lambda on wave lambda mod P, as its
// (lambda div P)-th logical wave.  P = 2 runs both row halves of one channel half (same weights) at once;
// P = 1 runs the four logical waves in four rounds, loading the weights of each round's channel half.
// Each output element sees the same MFMA sequence in every configuration, so results are bit-identical
// for every shard plan, grid and physical block.
#pragma once

#include "igemm_dma.h"

namespace miriam {

template <class T, int C_, int P_, int KS_, int ST_>
struct RwTile {
    typedef Mfma<T, 32> MF;
    typedef typename MF::op_t op_t;
    typedef typename MF::acc_t acc_t;
    typedef T elem_t;
    static_assert(sizeof(T) == 2, "16-bit operands only");
    static_assert(C_ % 8 == 0 && C_ >= 8 && C_ <= 64, "C must be a multiple of 8 up to 64");
    // two MFMA operand halves share one tap unless one tap holds a single half (C = 8)
    static_assert(KS_ == 1 || C_ == 8 || C_ % 16 == 0, "3x3 needs C = 8 or a multiple of 16");
    static constexpr int C = C_, P = P_, KS = KS_, ST = ST_;
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
    static_assert(LW % SL == 0, "slots");
    static_assert(PW < 128 && PH <= 16 && SP <= 16, "packed patch geometry");

    // row half of slot sl of round rd
    __device__ static constexpr int row_half(int pw, int rd, int sl) { return P == 4 ? (pw >> 1) : (P == 2 ? sl : (rd >> 1)); }
    // patch pixel offset of filter tap `tap` (row-major KS x KS)
    __host__ __device__ static constexpr int tap_pixel(int tap) { return (tap / KS) * PW + tap % KS; }
};

// Tiles in steps of the grid, as mixed-radix digits (no division per tile).
struct RwCursor {
    uint32_t img, ty, tx, nt;
};
struct RwWalk {
    uint32_t tX, tY, nT, gn, gx, gy, gi;
    __device__ __forceinline__ RwWalk(const IgemmArgs &a, uint32_t grid) : tX((uint32_t)a.tX), tY((uint32_t)a.tY), nT((uint32_t)a.nT) {
        const uint32_t g1 = grid / nT, g2 = g1 / tX;
        gn = grid % nT;
        gx = g1 % tX;
        gy = g2 % tY;
        gi = g2 / tY;
    }
    __device__ __forceinline__ RwCursor at(uint32_t t) const {
        const uint32_t r1 = t / nT, r2 = r1 / tX;
        return RwCursor{r2 / tY, r2 % tY, r1 % tX, t % nT};
    }
    __device__ __forceinline__ RwCursor advance(RwCursor c) const {
        c.nt += gn;
        const uint32_t cn = c.nt >= nT ? 1u : 0u;
        c.nt -= cn * nT;
        c.tx += gx + cn;
        const uint32_t cx = c.tx >= tX ? 1u : 0u;
        c.tx -= cx * tX;
        c.ty += gy + cx;
        const uint32_t cy = c.ty >= tY ? 1u : 0u;
        c.ty -= cy * tY;
        c.img += gi + cy;
        return c;
    }
};

// Stream of a tile's patch into LDS: instruction j writes slots 64j .. 64j+63 of the buffer.  The slot a
// lane fills is the same in every tile, so its decode (patch row and column, 16-byte piece, whether the
// slot holds data) is done once and kept packed in one register per instruction: bits [0, 7) column,
// [7, 11) row, [11, 15) piece, bit 15 set for a data slot.  Per tile a lane then only adds the tile's
// origin, checks the image bounds and forms a 32-bit byte offset into the image (the library admits the
// kernels only for images of less than 2^31 bytes); pixels outside the image and padding slots take an
// offset past the buffer, which reads zeros.
template <class K_>
struct RwPatch {
    uint32_t geo[K_::NJ];
    __device__ __forceinline__ RwPatch(int pw, int lane) {
#pragma unroll
        for (int jj = 0; jj < K_::NJ; ++jj) {
            const int j = jj * K_::P + pw;
            const int q = j * kWave + lane;
            const int pr = q / K_::SP, sl = q - (q / K_::SP) * K_::SP;
            const int prow = pr / K_::PW, pcol = pr - (pr / K_::PW) * K_::PW;
            const bool ok = j < K_::NINS && pr < K_::PPIX && sl < K_::NP;
            geo[jj] = ok ? ((uint32_t)pcol | ((uint32_t)prow << 7) | ((uint32_t)sl << 11) | (1u << 15)) : 0u;
        }
    }
    __device__ __forceinline__ void issue(const IgemmArgs &a, const RwCursor &c, uint32_t base, int pw) const {
        typedef typename K_::elem_t T;
        const int32_t H32 = (int32_t)a.H, W32 = (int32_t)a.W, ldx32 = (int32_t)a.ldx;
        const int32_t iy0 = (int32_t)c.ty * K_::TH * K_::ST - a.pad, ix0 = (int32_t)c.tx * K_::TW * K_::ST - a.pad;
        const rsrc_t rs = make_rsrc(static_cast<const T *>(a.x) + (int64_t)c.img * a.img_x, (uint32_t)(a.img_x * (int64_t)sizeof(T)));
#pragma unroll
        for (int jj = 0; jj < K_::NJ; ++jj) {
            const int j = jj * K_::P + pw;
            if (j < K_::NINS) {
                uint32_t g = geo[jj];
                asm volatile("" : "+v"(g));  // unpacked here: hoisted out of the tile loop, the fields spilled
                const int32_t iy = iy0 + (int32_t)((g >> 7) & 15u), ix = ix0 + (int32_t)(g & 127u);
                const bool ok = (g >> 15) != 0u && (uint32_t)iy < (uint32_t)H32 && (uint32_t)ix < (uint32_t)W32;
                const uint32_t off = (uint32_t)((iy * W32 + ix) * ldx32 + (int32_t)((g >> 11) & 15u) * K_::VEC) * (uint32_t)sizeof(T);
                buf_dma16(ok ? off : kOutOfRange, rs, 0u, base + (uint32_t)(j * kWave * 16));
            }
        }
    }
};

// Weights of n tile nt, channel half wn: step s holds k = 16s + 8hx .. +7 of output channel
// 64 nt + 32 wn + xl.
template <class K_>
__device__ __forceinline__ void rw_load_weights(const IgemmArgs &a, typename K_::op_t *dst, uint32_t nt, int wn, int lane) {
    typedef typename K_::op_t op_t;
    const int64_t n = 64 * (int64_t)nt + 32 * wn + (lane & 31);
#pragma unroll
    for (int s = 0; s < K_::NS; ++s) {
        const int k = 16 * s + 8 * (lane >> 5);
        op_t v = op_t{};
        if (n < a.Nc && k < K_::KTOT) v = *reinterpret_cast<const op_t *>(static_cast<const typename K_::elem_t *>(a.w) + n * a.ldw + k);
        dst[s] = v;
    }
}

// MFMA operands of the pixels: blocks i = 0, 1 (tile rows) of every slot of round rd held at once.
template <class K_>
struct RwOperands {
    typedef typename K_::op_t op_t;
    const char *abase[K_::SL][2];  // patch pixel (tile row y, column xl) + this lane's half
    int hx;                        // MFMA operand half
    __device__ __forceinline__ RwOperands(const char *patch, int pw, int rd, int hx_, int xl) : hx(hx_) {
#pragma unroll
        for (int sl = 0; sl < K_::SL; ++sl)
#pragma unroll
            for (int i = 0; i < 2; ++i) {
                const int y = 2 * K_::row_half(pw, rd, sl) + i;
                abase[sl][i] = patch + (y * K_::ST * K_::PW + xl * K_::ST) * K_::PS + (K_::NP == 1 ? 0 : hx * 16);
            }
    }
    // of k-step s for every block; one 8-channel tap per operand half (C = 8, 3x3): halves take taps 2s
    // and 2s+1
    __device__ __forceinline__ void fetch(int s, op_t (&av)[K_::SL][2]) const {
        constexpr int KS = K_::KS, C = K_::C, PS = K_::PS;
#pragma unroll
        for (int sl = 0; sl < K_::SL; ++sl)
#pragma unroll
            for (int i = 0; i < 2; ++i) {
                if constexpr (K_::NP == 1 && KS == 3) {
                    const int t0 = 2 * s, t1 = 2 * s + 1;
                    const int off0 = K_::tap_pixel(t0) * PS;
                    const int d1 = t1 < 9 ? (K_::tap_pixel(t1) - K_::tap_pixel(t0)) * PS : PS;
                    op_t v = *reinterpret_cast<const op_t *>(abase[sl][i] + off0 + hx * d1);
                    if (16 * s + 8 * hx >= K_::KTOT) v = op_t{};
                    av[sl][i] = v;
                } else {
                    // both halves in one tap (channels c0 .. c0 + 15); 1x1: the one tap
                    const int k0 = 16 * s, tap = KS == 1 ? 0 : k0 / C, c0 = KS == 1 ? k0 : k0 % C;
                    const int off = K_::tap_pixel(tap) * PS + (c0 / 8) * 16;
                    op_t v = *reinterpret_cast<const op_t *>(abase[sl][i] + off);
                    if (K_::KTOT % 16 != 0 && 16 * s + 8 * hx >= K_::KTOT) v = op_t{};
                    av[sl][i] = v;
                }
            }
    }
};

// Software pipeline of the K loops, in program order: the operand reads of step s + LA are issued before
// the MFMAs of step s, and a scheduling fence after each step keeps the compiler from sinking the reads
// next to their use (it otherwise waited on every read and ran each block's MFMAs as one dependent
// chain).  Within a step the blocks' MFMAs are independent.  (The loops stand in the kernels: moved into a
// function, the C = 64 kernel in blocks of 128 spills 36 registers, 68.9 -> 104.5 us.)
template <class K_>
constexpr int kRwAhead = K_::SL == 1 ? 2 : 1;

}  // namespace miriam
