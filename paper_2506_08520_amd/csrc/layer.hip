// The second half of a transformer layer in one kernel (bf16): output projection
// of the attention, residual, LayerNorm, MLP (fc1, GELU, fc2) and residual.
//
// As separate passes (projection GEMM, add, LayerNorm, fc1, GELU, fc2, add) the
// layer moved the map through memory fourteen times, four of them twice as wide;
// here O and X are read once and Y is written once.  Each wave keeps 16 rows of
// the map in registers throughout.  Every product is computed transposed, W^T
// as the left operand, so a result tile holds four consecutive channels of one
// row per lane (lane (g, c): channels 16t + 4g + i of row c) -- which is the
// right operand of the next product, once its weights are read with the
// contraction in the same order: slot (g, j) of 32 is channel 4g + j (j < 4) or
// 16 + 4g + j - 4.  No activation passes through LDS; the weights stream through
// it, double-buffered, 32 hidden units (rows of W1, columns of W2) at a time.
// LDS reads of the weights and the GELU arithmetic bound the loop.
// 65536 rows, C = 180, hidden 360: whole layer 352 us as separate kernels, 155 us
// fused (by kernel trace this kernel 81, the QKV product with its LayerNorm 49 and the
// attention 24 us); error against 64 bits 3.3e-3 -> 2.3e-3.
#include "block_common.hpp"

namespace nystra {
namespace {

struct TailArgs {
    BlockArgs p;                   // the projection: a = O, wpk, bias, out0 = Y, geometry
    const void *x, *lnw, *lnb, *w1, *b1, *w2, *b2;
    float eps;
    int hidden;
};

constexpr int kChunk = 32;         // hidden units per step

template <int KP>
struct TailLds {
    using R = RkLds<BF16, KP>;
    static constexpr int PH = KP + 8, P2 = kChunk + 8;        // pitches (halves) of W1, W2 rows
    static constexpr int w1 = 0, w2 = kChunk * PH / 2;        // words within a buffer
    static constexpr int b1 = w2 + KP * P2 / 2;
    static constexpr int buf = b1 + kChunk;                   // words per buffer
    static constexpr int stage = R::total > 2 * buf ? R::total : 2 * buf;
    static constexpr int tabs = stage;                        // [4][KP] floats
    static constexpr int total = tabs + 4 * KP;
};

struct __attribute__((aligned(4))) U8B {
    uint32_t w[2];
};

// v Phi(v) with Phi from Abramowitz & Stegun 7.1.26: erfc(x) = (a1 t + ... +
// a5 t^5) exp(-x^2), t = 1 / (1 + p x), within 1.5e-7; the result is rounded
// to bf16 right after.
__device__ inline float gelu(float v)
{
    const float x = fabsf(v) * 0.70710678f;
    const float t = __builtin_amdgcn_rcpf(fmaf(0.3275911f, x, 1.f));
    float p = fmaf(1.061405429f, t, -1.453152027f);
    p = fmaf(p, t, 1.421413741f);
    p = fmaf(p, t, -0.284496736f);
    p = fmaf(p, t, 0.254829592f);
    const float half_erfc = 0.5f * p * t * fast_exp2(-kLog2e * x * x);
    return v * (v < 0.f ? half_erfc : 1.f - half_erfc);
}

template <int KP>
__global__ void __launch_bounds__(512) __attribute__((amdgpu_waves_per_eu(KP <= 64 ? 4 : 2)))
layer_tail_kernel(TailArgs a)
{
    using L = TailLds<KP>;
    using R = RkLds<BF16, KP>;
    constexpr int KQ = KP / 4, NT = KP / 16, AWL = R::AWL, AP = R::AP, T = 512;
    static_assert(kRkThreads == T && kRkRows == 128, "one row tile per wave");
    __shared__ __align__(16) float lds[L::total];
    float *tbp = lds + L::tabs, *tlw = tbp + KP, *tlb = tlw + KP, *tb2 = tlb + KP;
    const int tid = threadIdx.x, lane = tid & 63, g = lane >> 4, c = lane & 15;
    const int wv = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int64_t m0 = int64_t(blockIdx.x) * kRkRows;
    const int C = a.p.C;

    // This lane's row (row c of its wave) at its pixel.
    const int64_t row = m0 + 16 * wv + c;
    const bool rok = row < a.p.rows;
    const int64_t rr = rok ? row : a.p.rows - 1;
    const int64_t wn = rr / a.p.N;
    const int64_t pix = pixel_of(a.p, wn, int(rr - wn * a.p.N)) * C;
    for (int n = tid; n < KP; n += T) {
        const bool ok = n < C;
        tbp[n] = ok && a.p.bias ? ld<BF16>(a.p.bias, n) : 0.f;
        tlw[n] = ok ? ld<BF16>(a.lnw, n) : 0.f;
        tlb[n] = ok ? ld<BF16>(a.lnb, n) : 0.f;
        tb2[n] = ok && a.b2 ? ld<BF16>(a.b2, n) : 0.f;
    }

    // ---- Projection: O's rows staged in LDS with coalesced 4-byte loads, then
    // the operand slots k = g KQ + s of row c into registers.
    __shared__ int rowbase[kRkRows], colofs[AWL];   // of row r (-1: none), of word w
    if (tid < kRkRows) {
        const int64_t r = m0 + tid;
        int base = -1;
        if (r < a.p.rows) {
            const int w = int(r / a.p.N), tt = int(r - int64_t(w) * a.p.N);
            base = int((int64_t(w) * a.p.heads * a.p.N + tt) * a.p.dh);
        }
        rowbase[tid] = base;
    }
    for (int w = tid; w < AWL; w += T) {
        const int k = 2 * w, hh = k / a.p.dh;
        colofs[w] = k < C ? hh * a.p.N * a.p.dh + (k - hh * a.p.dh) : -1;
    }
    typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
    constexpr int kPieces = R::tile / 4, kPer = (kPieces + T - 1) / T, NCT = (KP + 63) / 64;
    u32x4 wr[kPer];
    const u32x4 *wsrc = static_cast<const u32x4 *>(a.p.wpk);
    auto pfetch = [&](int ct) {
#pragma unroll
        for (int j = 0; j < kPer; ++j) {
            const int idx = tid + j * T;
            wr[j] = wsrc[int64_t(ct) * kPieces + (idx < kPieces ? idx : kPieces - 1)];
        }
    };
    auto pstash = [&](int buf) {
        u32x4 *dst = reinterpret_cast<u32x4 *>(lds + buf * R::tile);
#pragma unroll
        for (int j = 0; j < kPer; ++j) {
            const int idx = tid + j * T;
            if (kPer * T == kPieces || idx < kPieces)
                dst[idx] = wr[j];
        }
    };
    pfetch(0);
    __syncthreads();
    {
        constexpr int kPerT = kRkRows * AWL / T, kBatch = stage_batch(kPerT);
        static_assert(kPerT * T == kRkRows * AWL, "whole words per thread");
        const uint32_t *src = static_cast<const uint32_t *>(a.p.a);
        uint32_t *dst = reinterpret_cast<uint32_t *>(lds);
        for (int b0 = 0; b0 < kPerT; b0 += kBatch) {
            uint32_t x[kBatch];
            bool ok[kBatch];
#pragma unroll
            for (int u = 0; u < kBatch; ++u) {
                const int j = tid + (b0 + u) * T, r = j / AWL, w = j - r * AWL;
                const int rb = rowbase[r], co = colofs[w];
                ok[u] = rb >= 0 && co >= 0;
                x[u] = src[ok[u] ? (rb + co) >> 1 : 0];
            }
#pragma unroll
            for (int u = 0; u < kBatch; ++u) {
                const int j = tid + (b0 + u) * T, r = j / AWL, w = j - r * AWL;
                dst[r * AP + w] = ok[u] ? x[u] : 0u;
            }
        }
    }
    __syncthreads();
    bf8 ab[KQ / 8];
    {
        const float *arow = lds + (16 * wv + c) * AP;
#pragma unroll
        for (int s = 0; s < KQ / 8; ++s)
            ab[s] = *reinterpret_cast<const bf8 *>(arow + (g * KQ + 8 * s) / 2);
    }
    __syncthreads();   // the stage becomes the W tiles
    pstash(0);
    __syncthreads();

    // ---- the MLP weights of one step
    constexpr int kP1 = (kChunk * KP / 4 + T - 1) / T;
    constexpr int kP2 = (KP * kChunk / 4 + T - 1) / T;
    U8B r1[kP1], r2[kP2];
    float rb1 = 0.f;
    auto fetch = [&](int h0) {
#pragma unroll
        for (int j = 0; j < kP1; ++j) {   // W1 rows h0 + n, channels 4 k4 ..
            const int idx = tid + j * T, n = idx / (KP / 4), k = 4 * (idx - n * (KP / 4));
            const bool ok = n < kChunk && h0 + n < a.hidden && k < C;
            const U8B x = *reinterpret_cast<const U8B *>(
                static_cast<const uint16_t *>(a.w1) + (ok ? int64_t(h0 + n) * C + k : 0));
            const uint32_t keep = ok ? 0xffffffffu : 0u;
            r1[j].w[0] = x.w[0] & keep;
            r1[j].w[1] = x.w[1] & keep;
        }
#pragma unroll
        for (int j = 0; j < kP2; ++j) {   // W2 row n, hidden units h0 + 4 k4 ..
            const int idx = tid + j * T, n = idx / (kChunk / 4), k = 4 * (idx % (kChunk / 4));
            const bool ok = n < C && h0 + k < a.hidden;
            const U8B x = *reinterpret_cast<const U8B *>(
                static_cast<const uint16_t *>(a.w2) + (ok ? int64_t(n) * a.hidden + h0 + k : 0));
            const uint32_t keep = ok ? 0xffffffffu : 0u;
            r2[j].w[0] = x.w[0] & keep;
            r2[j].w[1] = x.w[1] & keep;
        }
        if (tid < kChunk) {
            const bool ok = a.b1 && h0 + tid < a.hidden;
            rb1 = ok ? ld<BF16>(a.b1, h0 + tid) : 0.f;
        }
    };
    // channel k of a 32-deep step -> its slot: 4g + j -> 8g + j, 16 + 4g + j -> 8g + 4 + j
    auto slot = [](int k) { return (k & ~31) + ((k & 12) << 1) + ((k & 16) >> 2); };
    auto stash = [&](int b) {
        float *base = lds + b * L::buf;
        uint16_t *w1 = reinterpret_cast<uint16_t *>(base + L::w1);
        uint16_t *w2 = reinterpret_cast<uint16_t *>(base + L::w2);
#pragma unroll
        for (int j = 0; j < kP1; ++j) {
            const int idx = tid + j * T, n = idx / (KP / 4), k = 4 * (idx - n * (KP / 4));
            if (kP1 * T == kChunk * KP / 4 || n < kChunk)
                *reinterpret_cast<uint2 *>(w1 + n * L::PH + slot(k)) =
                    make_uint2(r1[j].w[0], r1[j].w[1]);
        }
#pragma unroll
        for (int j = 0; j < kP2; ++j) {
            const int idx = tid + j * T, n = idx / (kChunk / 4), k = 4 * (idx % (kChunk / 4));
            if (kP2 * T == kChunk * KP / 4 || n < KP)
                *reinterpret_cast<uint2 *>(w2 + n * L::P2 + slot(k)) =
                    make_uint2(r2[j].w[0], r2[j].w[1]);
        }
        if (tid < kChunk)
            base[L::b1 + tid] = rb1;
    };

    f4 acc[NT];
#pragma unroll
    for (int t = 0; t < NT; ++t)
        acc[t] = f4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int it = 0; it < NCT; ++it) {
        if (it + 1 < NCT)
            pfetch(it + 1);
        const uint16_t *h = reinterpret_cast<const uint16_t *>(lds + (it & 1) * R::tile);
#pragma unroll
        for (int s = 0; s < KQ / 8; ++s)
#pragma unroll
            for (int q = 0; q < 4; ++q)
                if (4 * it + q < NT)   // compile-time
                    acc[4 * it + q] = mfma_bf16(
                        *reinterpret_cast<const bf8 *>(&h[(16 * q + c) * R::PH + g * KQ + 8 * s]),
                        ab[s], acc[4 * it + q]);
        __builtin_amdgcn_sched_barrier(0);
        if (it + 1 < NCT)
            pstash((it + 1) & 1);
        __syncthreads();
    }
    fetch(0);
    U8B res[NT];
#pragma unroll
    for (int t = 0; t < NT; ++t) {
        const int n = 16 * t + 4 * g;   // C is a multiple of 4: whole pieces
        res[t] = *reinterpret_cast<const U8B *>(static_cast<const uint16_t *>(a.x) + pix +
                                                (n < C ? n : 0));
        const uint32_t keep = n < C ? 0xffffffffu : 0u;
        res[t].w[0] &= keep;
        res[t].w[1] &= keep;
    }
    __builtin_amdgcn_sched_barrier(0);
    stash(0);   // the W tiles' buffers are free

    // ---- x1 = X + projection, its LayerNorm as bf16 operands, and x1 + b2 as
    // the accumulator of fc2.  Channels from C on are zero throughout.
    float sum = 0.f, sq = 0.f;
#pragma unroll
    for (int t = 0; t < NT; ++t) {
        const int n = 16 * t + 4 * g;
        const f4 bp = *reinterpret_cast<const f4 *>(tbp + n);
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const uint32_t w = res[t].w[i >> 1];
            const float xv = __uint_as_float(i & 1 ? w & 0xffff0000u : w << 16);
            acc[t][i] += bp[i] + xv;   // zeros from C on
            sum += acc[t][i];
        }
        __builtin_amdgcn_sched_barrier(0);
    }
    const float mean = sum_groups(sum) / float(C);
#pragma unroll
    for (int t = 0; t < NT; ++t)
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const float d = acc[t][i] - mean;
            sq = fmaf(d, 16 * t + 4 * g < C ? d : 0.f, sq);
        }
    const float rstd = 1.f / sqrtf(sum_groups(sq) / float(C) + a.eps);
    bf8 hb[KP / 32];
#pragma unroll
    for (int s = 0; s < KP / 32; ++s) {
        U16B u;
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            const int t = 2 * s + h, n = 16 * t + 4 * g;
            const f4 w = *reinterpret_cast<const f4 *>(tlw + n);
            const f4 b = *reinterpret_cast<const f4 *>(tlb + n);
            float y[4];
#pragma unroll
            for (int i = 0; i < 4; ++i)
                y[i] = fmaf((acc[t][i] - mean) * rstd, w[i], b[i]);   // w = b = 0 from C on
            u.w[2 * h] = cvt_bf16x2(y[0], y[1]);
            u.w[2 * h + 1] = cvt_bf16x2(y[2], y[3]);
        }
        hb[s] = __builtin_bit_cast(bf8, u);
        __builtin_amdgcn_sched_barrier(0);   // keeps the operands in flight few: 128 registers
    }
#pragma unroll
    for (int t = 0; t < NT; ++t)
        acc[t] += *reinterpret_cast<const f4 *>(tb2 + 16 * t + 4 * g);
    __syncthreads();

    // ---- MLP, 32 hidden units per step.
    int b = 0;
    for (int h0 = 0; h0 < a.hidden; h0 += kChunk, b ^= 1) {
        const bool more = h0 + kChunk < a.hidden;   // uniform
        if (more)
            fetch(h0 + kChunk);
        const float *base = lds + b * L::buf;
        const uint16_t *w1 = reinterpret_cast<const uint16_t *>(base + L::w1);
        const uint16_t *w2 = reinterpret_cast<const uint16_t *>(base + L::w2);
        f4 hid[2] = {*reinterpret_cast<const f4 *>(base + L::b1 + 4 * g),
                     *reinterpret_cast<const f4 *>(base + L::b1 + 16 + 4 * g)};
#pragma unroll
        for (int s = 0; s < KP / 32; ++s)
#pragma unroll
            for (int u = 0; u < 2; ++u)
                hid[u] = mfma_bf16(
                    *reinterpret_cast<const bf8 *>(w1 + (16 * u + c) * L::PH + 32 * s + 8 * g),
                    hb[s], hid[u]);
        __builtin_amdgcn_sched_barrier(0);
        U16B gu;
#pragma unroll
        for (int u = 0; u < 2; ++u)
#pragma unroll
            for (int p = 0; p < 2; ++p)
                gu.w[2 * u + p] = cvt_bf16x2(gelu(hid[u][2 * p]), gelu(hid[u][2 * p + 1]));
        const bf8 gb = __builtin_bit_cast(bf8, gu);
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int t = 0; t < NT; ++t)
            acc[t] = mfma_bf16(
                *reinterpret_cast<const bf8 *>(w2 + (16 * t + c) * L::P2 + 8 * g), gb, acc[t]);
        __builtin_amdgcn_sched_barrier(0);
        if (more)
            stash(b ^ 1);
        __syncthreads();
    }

    if (!rok)
        return;
#pragma unroll
    for (int t = 0; t < NT; ++t) {
        const int n = 16 * t + 4 * g;
        if (n < C) {
            const U8B u = {{cvt_bf16x2(acc[t][0], acc[t][1]), cvt_bf16x2(acc[t][2], acc[t][3])}};
            *reinterpret_cast<U8B *>(static_cast<uint16_t *>(a.p.out0) + pix + n) = u;
        }
    }
}

template <int KP>
void launch_tail(const TailArgs &a, hipStream_t stream)
{
    const unsigned blocks = unsigned((a.p.rows + kRkRows - 1) / kRkRows);
    hipLaunchKernelGGL((layer_tail_kernel<KP>), dim3(blocks), dim3(512), 0, stream, a);
}

}  // namespace

bool layer_supported(int64_t rows, int C, int heads, int dtype, int hidden)
{
    // Offsets of Q, K and V from one base are unsigned 32-bit (elements), the
    // grid is below 2^32 work-items.
    return dtype == 1 && C % 4 == 0 && C <= 256 && (C / heads) % 2 == 0 && hidden >= 1 &&
           hidden % 4 == 0 && 3 * (rows * int64_t(C) + 128) < (int64_t(1) << 32) &&
           rows * int64_t(C) < (int64_t(1) << 31) && rows / kRkRows < (int64_t(1) << 22);
}

hipError_t launch_layer_tail(const LayerTail &t, hipStream_t stream)
{
    TailArgs a{};
    const BlockGemm &g = t.gemm;
    a.p.rows = g.rows;
    a.p.H = g.H;
    a.p.W = g.W;
    a.p.C = g.C;
    a.p.heads = g.heads;
    a.p.dh = g.C / g.heads;
    a.p.w = g.w;
    a.p.N = g.w * g.w;
    a.p.shift = g.shift;
    a.p.nwx = g.W / g.w;
    a.p.nwy = g.H / g.w;
    a.p.a = g.a;
    a.p.wpk = g.wpk;
    a.p.bias = g.bias;
    a.p.out0 = g.out0;
    a.x = t.x;
    a.lnw = t.lnw;
    a.lnb = t.lnb;
    a.w1 = t.w1;
    a.b1 = t.b1;
    a.w2 = t.w2;
    a.b2 = t.b2;
    a.eps = t.eps;
    a.hidden = t.hidden;
    if (g.C <= 32)
        launch_tail<32>(a, stream);
    else if (g.C <= 64)
        launch_tail<64>(a, stream);
    else if (g.C <= 128)
        launch_tail<128>(a, stream);
    else if (g.C <= 192)
        launch_tail<192>(a, stream);
    else
        launch_tail<256>(a, stream);
    return hipGetLastError();
}

}  // namespace nystra
