// Parts of the window-attention block that its GEMMs and the fused transformer
// layer share: the argument block, the pixel of a token, and the LDS layout of
// the register-resident GEMM.
#pragma once

#include "internal.hpp"
#include "tile_common.hpp"

namespace nystra {
namespace {

using namespace tile;

struct BlockArgs {
    int64_t rows;                 // tokens, B H W
    int H, W, C, heads, dh, w, N, shift, nwx, nwy;
    int ncols;                    // 3C (QKV) or C (PROJ)
    int rtiles, ctiles;           // tile grid
    const void *a;                // X (QKV) or O (PROJ)
    const void *wt;               // [C][ncols]
    const void *wpk;              // wt packed as the register-resident kernel's LDS tiles
    const void *bias;             // [ncols] or null
    void *out0, *out1, *out2;     // Q, K, V (QKV) or Y (PROJ)
    bool pair;                    // register-resident kernel: store adjacent column pairs
    int64_t ostride;              // register-resident kernel: elements from Q to K and K to V
    int groups;                   // weight-resident kernel: column groups (ctiles tiles in each)
    const void *lnw, *lnb;        // LayerNorm of the rows of A before the product (LN)
    float eps;
};

// Flat pixel (b H + y) W + x of token t of window `win`.
__device__ inline int64_t pixel_of(const BlockArgs &a, int64_t win, int t)
{
    const int per = a.nwy * a.nwx;
    const int64_t b = win / per;
    const int wi = int(win - b * per);
    const int wy = wi / a.nwx, wx = wi - wy * a.nwx;
    const int ty = t / a.w, tx = t - ty * a.w;
    int y = wy * a.w + ty + a.shift, x = wx * a.w + tx + a.shift;
    if (y >= a.H)
        y -= a.H;
    if (x >= a.W)
        x -= a.W;
    return (b * a.H + y) * a.W + x;
}

template <class E>
__device__ inline float ld(const void *p, int64_t i)
{
    return E::load(static_cast<const typename E::T *>(p), i);
}

// Register-resident GEMM for C <= 256 (K padded to KP, a multiple of 32).
// Each wave holds its 16 rows of A for the whole contraction in registers, in the
// operand layout of the matrix cores: lane group g takes the contiguous quarter
// k in [g KP/4, (g+1) KP/4), so A is read from memory exactly once.  The
// workgroup's waves (128 rows) stream W through LDS one tile of CT columns at a
// time, double-buffered: the next tile's loads are in flight while the current
// one is multiplied.  W tiles in LDS: transposed bf16, [n][k] (eight k per
// 16-byte read); fp32 operands are carried as three bf16 terms (mfma_split3), A
// split once into registers, W on the way into LDS, a tile there holding the
// three planes one after another.
// What bounds it is latency: with the matrix instructions, the stores or the loads
// of A taken out, 35 us (bf16, 65536 rows, C = 180, 540 columns) fall to no less
// than 30; two row tiles per wave, which halve the LDS reads, measured the same
// (bf16) or slower (fp32, few rows: 74 -> 92 us a block).  CT is the widest tile
// that lets two workgroups share a CU's 160 KB.
constexpr int kRkRows = 128, kRkThreads = 512;   // eight waves of one row tile

template <class E, int KP>
struct RkLds {
    static constexpr bool BF = E::bytes == 2;
    static constexpr int NP = BF ? 1 : 3;    // bf16 planes
    static constexpr int CT = BF ? 64 : (KP <= 192 ? 32 : 16);   // columns per W tile
    static constexpr int PH = KP + 8;        // [n][k]: halves per column
    static constexpr int plane = CT * PH / 2;                 // words
    static constexpr int tile = NP * plane;                   // words per buffer
    // Packed image in memory, by 64-column tiles: the LDS image (bf16), or
    // fp32 [n][k] with pitch KP (the last 4 KP words of a tile unused).
    static constexpr int image = BF ? tile : 68 * KP;         // words per 64 columns
    static constexpr int SR = BF ? kRkRows : (KP <= 192 ? 64 : 32);   // A rows staged at a time
    static constexpr int AWL = KP / (BF ? 2 : 1);             // words per staged row
    // row pitch (words; + 8: fewer bank conflicts than + 4 in the operand reads)
    static constexpr int AP = AWL + 8;
    static constexpr int astage = SR * AP;
    static constexpr int total = 2 * tile > astage ? 2 * tile : astage;
};

// LDS of the weight-resident GEMM: tiles of CT columns, NP planes of [n][k] with
// pitch PH halves each; NT tiles at most, so that two workgroups share a CU's
// 160 KB (fp32 from KP = 192 on: one workgroup with as much as fits, since its
// registers allow no second).
constexpr int kRwThreads = 512;

template <class E, int KP>
struct RwLds {
    static constexpr bool BF = E::bytes == 2;
    static constexpr int NP = BF ? 1 : 3;
    static constexpr int CT = BF ? 64 : 32;
    static constexpr int PH = KP + 8;
    static constexpr int plane = CT * PH / 2, tile = NP * plane;   // words
    static constexpr int room = BF || KP < 192 ? 72 * 1024 + (KP == 192 ? 5 * 1024 : 0) : 154 * 1024;
    static constexpr int NT = room / (4 * tile) > 12 ? 12 : room / (4 * tile);
    static_assert(NT >= 1, "a tile fits");
    // steps of 32 that lie below C for every C of this KP (above the next smaller)
    static constexpr int full = KP == 32 ? 0 : KP == 64 ? 1 : KP == 128 ? 2 : KP == 192 ? 4 : 6;
};

// Words per batch of the A stage: the largest divisor of n up to 16.
constexpr int stage_batch(int n)
{
    for (int b = 16; b > 1; --b)
        if (n % b == 0)
            return b;
    return 1;
}

}  // namespace
}  // namespace nystra
