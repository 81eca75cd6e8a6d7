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

constexpr int kRkRows = 128;
template <class E>
constexpr int rk_rt() { return E::bytes == 2 ? 1 : 1; }   // row tiles per wave
template <class E>
constexpr int rk_threads() { return 64 * (kRkRows / (16 * rk_rt<E>())); }


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
    static constexpr int rowbase = SR * AP, colofs = rowbase + kRkRows;
    static constexpr int astage = colofs + AWL;               // the stage and its offset tables
    static constexpr int total = 2 * tile > astage ? 2 * tile : astage;
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
