// Window-attention block around the PnP-Nystra operator, the structure of
// Sec. 1 for SwinIR / Uformer-style models: the map is cut into w x w windows
// (after a cyclic shift s for shifted windows), Q, K, V = X W_qkv + b per
// token, every (window, head) attends, the heads are concatenated, and
// Y = O W_proj + b goes back to the token's pixel.
//
// Two launches of one MFMA GEMM surround the attention kernels:
//   QKV   rows = tokens in window order, A row r = the pixel of token r in X;
//         the epilogue writes Q, K, V straight into [window][head][N][d_h].
//   PROJ  A row r = token r's d_h-wide slices of O, one per head (the head
//         concatenation is a gather); the epilogue writes Y at the pixel.
// Four kernels compute them.  C <= 256 (weights packed beforehand): the row-resident and
// the weight-resident GEMM, launch_rk_ln() says which.  Above, widths that are
// multiples of 8: 128 x 128 tiles (wide).  Everything else (odd widths, unaligned
// tensors, few fp32 rows past 256 channels): block_gemm_kernel, a 64 x 64 tile of the
// product over 32-deep chunks of the contraction staged in LDS, the next chunk's loads in
// flight while the current one is multiplied; four waves each own a 32 x 32 quarter (2 x 2
// MFMA tiles).  Tiles are mapped so that the column tiles of one row tile run on the
// same XCD and share its L2 for the gathered rows.
#include <type_traits>

#include "block_common.hpp"

namespace nystra {
namespace {

using namespace tile;

constexpr int kBM = 64, kBN = 64, kBK = 32;

// Block id -> (row tile, column tile), so that consecutive logical tiles (the
// column tiles of one row tile) land on one XCD (ids go round-robin over 8).
__device__ inline void tile_of(const BlockArgs &a, int &rt, int &ct)
{
    const int T = a.rtiles * a.ctiles, q = T / 8, r = T % 8;
    const int b = int(blockIdx.x), x = b % 8, local = b / 8;
    const int L = (x < r ? x * (q + 1) : r * (q + 1) + (x - r) * q) + local;
    rt = L / a.ctiles;
    ct = L - rt * a.ctiles;
}

template <class E, bool PROJ>
__global__ void __launch_bounds__(256) block_gemm_kernel(BlockArgs a)
{
    constexpr bool BF = E::bytes == 2;
    // fp32: A [64][36], B [32][68] floats.  bf16: A [64][40], B^T [64][40] halves.
    constexpr int PA = BF ? kBK + 8 : kBK + 4, PB = BF ? kBK + 8 : kBN + 4;
    __shared__ __align__(16) typename E::T As[kBM * PA];
    __shared__ __align__(16) typename E::T Bs[BF ? kBN * PB : kBK * PB];
    int rt, ct;
    tile_of(a, rt, ct);
    const int tid = threadIdx.x, lane = tid & 63, g = lane >> 4, c = lane & 15;
    const int wv = __builtin_amdgcn_readfirstlane(tid >> 6), wr = wv >> 1, wc = wv & 1;
    const int64_t m0 = int64_t(rt) * kBM;
    const int n0 = ct * kBN;

    // This thread's A row (fixed over the contraction) and B row of a chunk.
    const int arow = tid >> 2, ak = (tid & 3) * 8;
    const int64_t r = m0 + arow;
    const bool rok = r < a.rows;
    const int64_t win = rok ? r / a.N : 0;
    const int t = rok ? int(r - win * a.N) : 0;
    int64_t abase;   // QKV: element offset of the pixel row; PROJ: of head 0's slice
    if constexpr (PROJ)
        abase = (win * a.heads * a.N + t) * int64_t(a.dh);
    else
        abase = pixel_of(a, win, t) * int64_t(a.C);
    const int64_t headstride = int64_t(a.N) * a.dh;
    const int bk = tid >> 3, bn = (tid & 7) * 8;

    float ra[8], rb[8];
    auto fetch = [&](int k0) {
        int k = k0 + ak;
        int hh = 0, dd = 0;
        if constexpr (PROJ) {
            hh = k / a.dh;
            dd = k - hh * a.dh;
        }
#pragma unroll
        for (int j = 0; j < 8; ++j) {
            float x = 0.f;
            if (rok && k < a.C) {
                if constexpr (PROJ)
                    x = ld<E>(a.a, abase + hh * headstride + dd);
                else
                    x = ld<E>(a.a, abase + k);
            }
            ra[j] = x;
            ++k;
            if constexpr (PROJ) {
                if (++dd == a.dh) {
                    dd = 0;
                    ++hh;
                }
            }
        }
        const int kb = k0 + bk;
#pragma unroll
        for (int j = 0; j < 8; ++j) {
            const int n = n0 + bn + j;
            rb[j] = (kb < a.C && n < a.ncols) ? ld<E>(a.wt, int64_t(kb) * a.ncols + n) : 0.f;
        }
    };
    auto stash = [&]() {
        if constexpr (BF) {
            U16B u;
#pragma unroll
            for (int p = 0; p < 4; ++p)
                u.w[p] = cvt_bf16x2(ra[2 * p], ra[2 * p + 1]);   // exact: bf16 values
            *reinterpret_cast<U16B *>(&As[arow * PA + ak]) = u;
#pragma unroll
            for (int j = 0; j < 8; ++j)
                Bs[(bn + j) * PB + bk] = uint16_t(cvt_bf16x2(rb[j], 0.f));
        } else {
#pragma unroll
            for (int j = 0; j < 8; ++j) {
                As[arow * PA + ak + j] = ra[j];
                Bs[bk * PB + bn + j] = rb[j];
            }
        }
    };

    f4 acc[2][2];
#pragma unroll
    for (int i = 0; i < 2; ++i)
        acc[i][0] = acc[i][1] = f4{0.f, 0.f, 0.f, 0.f};
    fetch(0);
    stash();
    __syncthreads();
    for (int k0 = 0; k0 < a.C; k0 += kBK) {
        const bool more = k0 + kBK < a.C;   // uniform
        if (more)
            fetch(k0 + kBK);
        if constexpr (BF) {
#pragma unroll
            for (int ti = 0; ti < 2; ++ti) {
                const bf8 av = *reinterpret_cast<const bf8 *>(&As[(32 * wr + 16 * ti + c) * PA + 8 * g]);
#pragma unroll
                for (int tj = 0; tj < 2; ++tj) {
                    const bf8 bv =
                        *reinterpret_cast<const bf8 *>(&Bs[(32 * wc + 16 * tj + c) * PB + 8 * g]);
                    acc[ti][tj] = mfma_bf16(av, bv, acc[ti][tj]);
                }
            }
        } else {
            // The chunk is summed by itself: a sum over C is two short chains of
            // roundings, not one.
            f4 part[2][2];
#pragma unroll
            for (int i = 0; i < 2; ++i)
                part[i][0] = part[i][1] = f4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int s = 0; s < kBK / 4; ++s) {
                float av[2], bv[2];
#pragma unroll
                for (int i = 0; i < 2; ++i) {
                    av[i] = As[(32 * wr + 16 * i + c) * PA + 4 * s + g];
                    bv[i] = Bs[(4 * s + g) * PB + 32 * wc + 16 * i + c];
                }
#pragma unroll
                for (int ti = 0; ti < 2; ++ti)
#pragma unroll
                    for (int tj = 0; tj < 2; ++tj)
                        part[ti][tj] = mfma4(av[ti], bv[tj], part[ti][tj]);
            }
#pragma unroll
            for (int i = 0; i < 2; ++i)
#pragma unroll
                for (int j = 0; j < 2; ++j)
                    acc[i][j] += part[i][j];
        }
        __syncthreads();
        if (more) {
            stash();
            __syncthreads();
        }
    }

    // Epilogue: lane (g, c) holds rows 4g + i, column c of each 16 x 16 tile.
#pragma unroll
    for (int tj = 0; tj < 2; ++tj) {
        const int n = n0 + 32 * wc + 16 * tj + c;
        if (n >= a.ncols)
            continue;
        const float bias = a.bias ? ld<E>(a.bias, n) : 0.f;
        int which = 0, hh = 0, dd = n;
        if constexpr (!PROJ) {
            which = n / a.C;
            const int cc = n - which * a.C;
            hh = cc / a.dh;
            dd = cc - hh * a.dh;
        }
        typename E::T *dst = static_cast<typename E::T *>(which == 0 ? a.out0
                                                          : which == 1 ? a.out1 : a.out2);
#pragma unroll
        for (int ti = 0; ti < 2; ++ti)
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const int64_t row = m0 + 32 * wr + 16 * ti + 4 * g + i;
                if (row >= a.rows)
                    continue;
                const int64_t wn = row / a.N;
                const int tt = int(row - wn * a.N);
                const float v = acc[ti][tj][i] + bias;
                if constexpr (PROJ)
                    E::store(dst, pixel_of(a, wn, tt) * a.C + n, v);
                else
                    E::store(dst, ((wn * a.heads + hh) * a.N + tt) * int64_t(a.dh) + dd, v);
            }
    }
}

// Wide variant (C > 256, where the weights are not packed): a workgroup of
// four waves computes a 128 x 128 tile, each wave a 64 x 64 quarter, over chunks
// of 64 (bf16) or 32 (fp32) of the contraction.  What bounds it is the operand
// traffic: every 16-byte operand read from LDS feeds four matrix instructions,
// global reads are 16-byte pieces of A rows and 8-byte pieces of W rows whose
// 8 x 4 (8 x 2) blocks are transposed in registers, and the next chunk's loads
// are in flight while this one is multiplied.  fp32 operands are split into
// three bf16 terms on the way into LDS (mfma_split3).  LDS rows hold their
// 16-byte slots permuted by the row (slot()), which keeps both the transposed
// stores and the operand reads free of bank conflicts without padding.
// The product is computed transposed, so that a lane holds four adjacent
// columns of one row and stores them in one piece.
// Whole block calls, old 64 x 64 tiles with 2- and 4-byte loads -> this kernel:
// C = 512, 8192 rows bf16 361 -> 66 us, fp32 488 -> 179 us; C = 384, 36864 rows
// bf16 935 -> 178 us; C = 320, 1024 rows bf16 66 -> 39 us.  The fp32 error against
// 64 bits falls from 5.2e-7 to 4.6e-7 (C = 320): fewer roundings per sum.
template <class E>
struct WideCfg {
    static constexpr bool BF = E::bytes == 2;
    static constexpr int BM = 128, BN = 128, BK = BF ? 64 : 32;
    static constexpr int planes = BF ? 1 : 3;
    static constexpr int slots = BK / 8;         // 16-byte slots per LDS row
    static constexpr int wcols = BF ? 4 : 2;     // W columns per 8-byte piece
    static constexpr int ap = BM * slots / 256;  // A pieces (8 values) per thread
};

template <class E>
__device__ inline int wide_slot(int row, int kp)
{
    using F = WideCfg<E>;
    const int f = F::BF ? (row ^ (row >> 2)) & 7 : (row >> 1) & 3;
    return row * F::slots + (kp ^ f);
}

template <class E, bool PROJ>
__global__ void __launch_bounds__(256) block_gemm_wide_kernel(BlockArgs a)
{
    using F = WideCfg<E>;
    constexpr bool BF = F::BF;
    constexpr int kSlots = F::BM * F::slots;     // slots of one operand plane
    __shared__ bf8 As[F::planes * kSlots], Bs[F::planes * kSlots];
    // fp32: a value of A or W is not finite; the tile is then computed again on the
    // fp32 matrix cores.
    __shared__ int infinite;
    if (!BF && threadIdx.x == 0)
        infinite = 0;
    int rt, ct;
    tile_of(a, rt, ct);
    const int tid = threadIdx.x, lane = tid & 63, g = lane >> 4, c = lane & 15;
    const int wv = __builtin_amdgcn_readfirstlane(tid >> 6), wr = wv >> 1, wc = wv & 1;
    const int64_t m0 = int64_t(rt) * F::BM;
    const int n0 = ct * F::BN;

    // This thread's A pieces: rows (tid + 256 j) / slots, the same k slot in each.
    const int akp = tid % F::slots;
    const typename E::T *arow[F::ap];
    bool aok[F::ap];
#pragma unroll
    for (int j = 0; j < F::ap; ++j) {
        const int64_t r = m0 + (tid + 256 * j) / F::slots;
        aok[j] = r < a.rows;
        const int64_t rr = aok[j] ? r : a.rows - 1;
        const int64_t win = rr / a.N;
        const int t = int(rr - win * a.N);
        arow[j] = static_cast<const typename E::T *>(a.a) +
                  (PROJ ? (win * a.heads * a.N + t) * int64_t(a.dh)
                        : pixel_of(a, win, t) * int64_t(a.C));
    }
    const int64_t headstride = int64_t(a.N) * a.dh;
    // ... and its W block: rows k0 + 8 bkp .., columns n0 + wcols bcg ..
    constexpr int cgs = F::BN / F::wcols;
    const int bkp = tid / cgs, bn = (tid % cgs) * F::wcols;
    const bool bok = n0 + bn < a.ncols;   // whole pieces: ncols is a multiple of 8
    const typename E::T *wcol = static_cast<const typename E::T *>(a.wt) + (bok ? n0 + bn : 0);

    struct __attribute__((aligned(4))) U8B { uint32_t w[2]; };
    constexpr int APW = BF ? 1 : 2;   // 16-byte loads per A piece
    U16B ra[F::ap][APW];
    U8B rb[8];
    auto fetch = [&](int k0) {
        const int k = k0 + 8 * akp;
        const bool kok = k < a.C;     // whole pieces: C is a multiple of 8
        int64_t off = kok ? k : 0;
        if constexpr (PROJ) {         // d_h is a multiple of 8: a piece lies in one head
            const int hh = int(off) / a.dh;
            off = hh * headstride + (int(off) - hh * a.dh);
        }
#pragma unroll
        for (int j = 0; j < F::ap; ++j)
#pragma unroll
            for (int h = 0; h < APW; ++h) {
                U16B x = *reinterpret_cast<const U16B *>(arow[j] + off + 4 * h);
#pragma unroll
                for (int w = 0; w < 4; ++w)
                    ra[j][h].w[w] = aok[j] && kok ? x.w[w] : 0u;
            }
        const int kb = k0 + 8 * bkp;
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            const bool ok = bok && kb + e < a.C;
            const U8B x = *reinterpret_cast<const U8B *>(
                wcol + int64_t(kb + e < a.C ? kb + e : 0) * a.ncols);
            rb[e].w[0] = ok ? x.w[0] : 0u;
            rb[e].w[1] = ok ? x.w[1] : 0u;
        }
    };
    u16x2 top = {0, 0};
    auto stash = [&](auto clean) {
#pragma unroll
        for (int j = 0; j < F::ap; ++j) {
            const int at = wide_slot<E>((tid + 256 * j) / F::slots, akp);
            if constexpr (BF) {
                As[at] = __builtin_bit_cast(bf8, ra[j][0]);
            } else {
                float x[8];
#pragma unroll
                for (int e = 0; e < 8; ++e)
                    x[e] = __uint_as_float(ra[j][e >> 2].w[e & 3]);
                split3_bf16<clean>(x, As[at], As[kSlots + at], As[2 * kSlots + at], top);
            }
        }
#pragma unroll
        for (int j = 0; j < F::wcols; ++j) {
            const int at = wide_slot<E>(bn + j, bkp);
            if constexpr (BF) {
                U16B u;
#pragma unroll
                for (int p = 0; p < 4; ++p)   // halves j of rows 2p and 2p + 1
                    u.w[p] = __builtin_amdgcn_perm(rb[2 * p + 1].w[j >> 1], rb[2 * p].w[j >> 1],
                                                   j & 1 ? 0x07060302u : 0x05040100u);
                Bs[at] = __builtin_bit_cast(bf8, u);
            } else {
                float x[8];
#pragma unroll
                for (int e = 0; e < 8; ++e)
                    x[e] = __uint_as_float(rb[e].w[j]);
                split3_bf16<clean>(x, Bs[at], Bs[kSlots + at], Bs[2 * kSlots + at], top);
            }
        }
    };

    f4 acc[4][4];   // [row tile][column tile]: lane (g, c) row c, columns 4g + i
    auto product = [&](auto f32) {   // f32: on the fp32 matrix cores
#pragma unroll
        for (int i = 0; i < 4; ++i)
#pragma unroll
            for (int j = 0; j < 4; ++j)
                acc[i][j] = f4{0.f, 0.f, 0.f, 0.f};
        fetch(0);
        for (int k0 = 0; k0 < a.C; k0 += F::BK) {
            stash(f32);   // the first time as if every value were finite
            __syncthreads();
            if (k0 + F::BK < a.C)   // uniform
                fetch(k0 + F::BK);
#pragma unroll
            for (int s = 0; s < F::BK / 32; ++s) {
                bf8 av[4][F::planes];
#pragma unroll
                for (int i = 0; i < 4; ++i)
#pragma unroll
                    for (int p = 0; p < F::planes; ++p)
                        av[i][p] = As[p * kSlots + wide_slot<E>(64 * wr + 16 * i + c, 4 * s + g)];
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    bf8 bv[F::planes];
#pragma unroll
                    for (int p = 0; p < F::planes; ++p)
                        bv[p] = Bs[p * kSlots + wide_slot<E>(64 * wc + 16 * j + c, 4 * s + g)];
#pragma unroll
                    for (int i = 0; i < 4; ++i) {
                        if constexpr (BF) {
                            acc[i][j] = mfma_bf16(bv[0], av[i][0], acc[i][j]);
                        } else if constexpr (f32) {
                            float x[8], w[8];
                            join3_bf16(av[i][0], av[i][1], av[i][2], x);
                            join3_bf16(bv[0], bv[1], bv[2], w);
                            acc[i][j] = mfma_f32x8(w, x, acc[i][j]);
                            __builtin_amdgcn_sched_barrier(0);   // few registers
                        } else {
                            acc[i][j] = mfma_split3(bv[0], bv[1], bv[2], av[i][0], av[i][1],
                                                    av[i][2], acc[i][j]);
                        }
                    }
                }
            }
            __syncthreads();
        }
    };
    product(std::false_type{});
    if constexpr (!BF) {
        if (not_finite(top))
            infinite = 1;
        __syncthreads();
        if (__builtin_amdgcn_readfirstlane(infinite))   // uniform
            product(std::true_type{});
    }

    // Epilogue: four adjacent columns of one row per lane and tile, in one head
    // (d_h is a multiple of 8) and on one side of ncols.
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        const int n = n0 + 64 * wc + 16 * j + 4 * g;
        if (n >= a.ncols)
            continue;
        float bias[4];
#pragma unroll
        for (int e = 0; e < 4; ++e)
            bias[e] = a.bias ? ld<E>(a.bias, n + e) : 0.f;
        int which = 0, hh = 0, dd = n;
        if constexpr (!PROJ) {
            which = n / a.C;
            const int cc = n - which * a.C;
            hh = cc / a.dh;
            dd = cc - hh * a.dh;
        }
        typename E::T *dst = static_cast<typename E::T *>(which == 0 ? a.out0
                                                          : which == 1 ? a.out1 : a.out2);
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const int64_t row = m0 + 64 * wr + 16 * i + c;
            if (row >= a.rows)
                continue;
            const int64_t wn = row / a.N;
            const int tt = int(row - wn * a.N);
            typename E::T *d = dst + (PROJ ? pixel_of(a, wn, tt) * a.C + n
                                           : ((wn * a.heads + hh) * a.N + tt) * int64_t(a.dh) + dd);
            const f4 v = acc[i][j];
            if constexpr (BF) {
                U8B u = {{cvt_bf16x2(v[0] + bias[0], v[1] + bias[1]),
                          cvt_bf16x2(v[2] + bias[2], v[3] + bias[3])}};
                *reinterpret_cast<U8B *>(d) = u;
            } else {
                U16B u;
#pragma unroll
                for (int e = 0; e < 4; ++e)
                    u.w[e] = __float_as_uint(v[e] + bias[e]);
                *reinterpret_cast<U16B *>(d) = u;
            }
        }
    }
}

// Whole 16-byte pieces of A and of a head, 8-byte pieces of W and of the
// outputs, all on 4-byte addresses.
bool wide_ok(const BlockArgs &a, bool proj)
{
    const uintptr_t p = uintptr_t(a.a) | uintptr_t(a.wt) | uintptr_t(a.out0) |
                        (proj ? 0 : uintptr_t(a.out1) | uintptr_t(a.out2));
    return a.C % 8 == 0 && a.dh % 8 == 0 && p % 4 == 0;
}

// Packs W [C][ncols], transposed, by 64-column tiles, one after another: [n][k]
// with pitch PH halves (bf16, the tile's LDS image) or KP floats.  Every slot
// outside W (k >= C, n >= ncols, the pitch padding) is zero.  The second matrix's
// pieces follow the first's in the grid.
struct WPackArgs {
    const void *w0, *w1;   // W_qkv [C][3C], W_proj [C][C]
    uint32_t *d0, *d1;     // their packed images
    int C, words0, words1;
};

template <class E, int KP>
__global__ void __launch_bounds__(256) block_wpack_kernel(WPackArgs p)
{
    // One thread per 16-byte piece: eight (bf16) or four (fp32) k of a column.
    using L = RkLds<E, KP>;
    constexpr int kPieces = L::image / 4, EP = E::bytes == 2 ? 8 : 4;
    const int64_t gi = int64_t(blockIdx.x) * 256 + threadIdx.x;
    const int64_t p0 = p.words0 / 4;
    const bool second = gi >= p0;
    const int64_t pi = second ? gi - p0 : gi;
    if (pi >= (second ? p.words1 / 4 : p0))
        return;
    const int ncols = second ? p.C : 3 * p.C;
    const typename E::T *W = static_cast<const typename E::T *>(second ? p.w1 : p.w0);
    const int ct = int(pi / kPieces), r = int(pi - int64_t(ct) * kPieces), n0 = 64 * ct;
    // column n = r mod 64 (consecutive threads: consecutive columns of EP rows
    // of W), elements k0 .. k0 + EP - 1 of its image row.  Branch-free: every
    // load reads an in-bounds element (indices clamped) and a select zeroes the
    // slots outside W, so a thread's loads issue together.
    const int n = r & 63, k0 = EP * (r >> 6);
    uint32_t x[EP];
#pragma unroll
    for (int e = 0; e < EP; ++e) {
        const int k = k0 + e;
        const bool ok = k < p.C && n0 + n < ncols;
        const int64_t i = int64_t(k < p.C ? k : p.C - 1) * ncols + (n0 + n < ncols ? n0 + n : ncols - 1);
        uint32_t w;
        if constexpr (E::bytes == 2)
            w = uint32_t(reinterpret_cast<const uint16_t *>(W)[i]);
        else
            w = __float_as_uint(W[i]);
        x[e] = ok ? w : 0u;
    }
    typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
    u32x4 out;
    int dst;   // piece index within the tile image
    if constexpr (E::bytes == 2) {
#pragma unroll
        for (int e = 0; e < 4; ++e)
            out[e] = x[2 * e] | (x[2 * e + 1] << 16);
        dst = (n * L::PH + k0) / 8;
    } else {
#pragma unroll
        for (int e = 0; e < 4; ++e)
            out[e] = x[e];
        dst = k0 < KP ? (n * KP + k0) / 4 : r;   // past the rows: the unused words
    }
    reinterpret_cast<u32x4 *>(second ? p.d1 : p.d0)[int64_t(ct) * kPieces + dst] = out;
}

// acc[q] = A (KS steps of 32 k, NP planes) times column tile q of a W tile in LDS;
// h points at this lane's slot of the tile's first column, steps lie `step`
// halves apart.
template <class L, int KS>
__device__ inline void tile_product(const bf8 (&ab)[L::NP][KS], const uint16_t *h, int step,
                                    f4 (&acc)[L::CT / 16])
{
    constexpr int NQ = L::CT / 16;
#pragma unroll
    for (int q = 0; q < NQ; ++q)
        acc[q] = f4{0.f, 0.f, 0.f, 0.f};
    if constexpr (L::NP == 1) {
#pragma unroll
        for (int s = 0; s < KS; ++s)
#pragma unroll
            for (int q = 0; q < NQ; ++q)
                acc[q] = mfma_bf16(
                    ab[0][s], *reinterpret_cast<const bf8 *>(&h[16 * q * L::PH + step * s]), acc[q]);
    } else {
        // The six products of mfma_split3, the small ones in accumulators of their
        // own and the column tiles side by side: several chains of dependent
        // instructions at a time.
        f4 low[NQ];
#pragma unroll
        for (int q = 0; q < NQ; ++q)
            low[q] = f4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int s = 0; s < KS; ++s) {
            bf8 bv[NQ][3];
#pragma unroll
            for (int q = 0; q < NQ; ++q)
#pragma unroll
                for (int p = 0; p < 3; ++p)
                    bv[q][p] = *reinterpret_cast<const bf8 *>(
                        &h[2 * p * L::plane + 16 * q * L::PH + step * s]);
#pragma unroll
            for (int q = 0; q < NQ; ++q) {
                low[q] = mfma_bf16(ab[2][s], bv[q][0], low[q]);
                acc[q] = mfma_bf16(ab[1][s], bv[q][0], acc[q]);
            }
#pragma unroll
            for (int q = 0; q < NQ; ++q) {
                low[q] = mfma_bf16(ab[0][s], bv[q][2], low[q]);
                acc[q] = mfma_bf16(ab[0][s], bv[q][1], acc[q]);
            }
#pragma unroll
            for (int q = 0; q < NQ; ++q) {
                low[q] = mfma_bf16(ab[1][s], bv[q][1], low[q]);
                acc[q] = mfma_bf16(ab[0][s], bv[q][0], acc[q]);
            }
        }
#pragma unroll
        for (int q = 0; q < NQ; ++q)
            acc[q] += low[q];
    }
}

// The same on the fp32 matrix cores, for operands that are not all finite.
template <class L, int KS>
__device__ inline void tile_product_f32(const bf8 (&ab)[L::NP][KS], const uint16_t *h, int step,
                                        f4 (&acc)[L::CT / 16])
{
#pragma unroll
    for (int q = 0; q < L::CT / 16; ++q)
        acc[q] = f4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int s = 0; s < KS; ++s) {
        // Joined here, on this rare path: the compiler must not keep the joined
        // rows in registers over the tiles.
        bf8 t[3];
#pragma unroll
        for (int p = 0; p < 3; ++p) {
            t[p] = ab[p % L::NP][s];
            asm volatile("" : "+v"(t[p]));
        }
        float x[8];
        join3_bf16(t[0], t[1], t[2], x);
#pragma unroll
        for (int q = 0; q < L::CT / 16; ++q) {
            const uint16_t *w = &h[16 * q * L::PH + step * s];
            float y[8];
            join3_bf16(*reinterpret_cast<const bf8 *>(w),
                       *reinterpret_cast<const bf8 *>(w + 2 * L::plane),
                       *reinterpret_cast<const bf8 *>(w + 4 * L::plane), y);
            acc[q] = mfma_f32x8(x, y, acc[q]);
            __builtin_amdgcn_sched_barrier(0);   // few registers
        }
    }
}

// Stores a tile of CT columns from column n0 on: lane (g, c) holds rows 4g + i,
// column c of each 16 x 16 tile; destination = row part (rowoff) + column part
// (coltab).  With a.pair, lanes c and c ^ 1 swap one value per two rows so that
// the even lane holds columns (c, c + 1) of row 4g + 2p and the odd lane those
// of row 4g + 2p + 1: one 4-byte (bf16) or 8-byte (fp32) store per two outputs.
// Pairs never straddle a head or Q/K/V (d_h and C even).
template <class E, class L>
__device__ inline void store_tile(const BlockArgs &a, const f4 (&acc)[L::CT / 16], int n0, int c,
                                  const uint32_t (&rowoff)[4], const bool (&rowok)[4],
                                  const float *bias, const uint32_t *coltab)
{
    constexpr bool BF = E::bytes == 2;
    typename E::T *dst = static_cast<typename E::T *>(a.out0);
    const bool odd = c & 1;
    if (a.pair) {   // uniform
#pragma unroll
        for (int q = 0; q < L::CT / 16; ++q) {
            const int j = 16 * q + c;
            if (n0 + j >= a.ncols)   // column pairs lie on one side of ncols
                continue;
            const float b = bias[j];
            const uint32_t col = coltab[j & ~1];
#pragma unroll
            for (int pp = 0; pp < 2; ++pp) {
                const float v0 = acc[q][2 * pp] + b, v1 = acc[q][2 * pp + 1] + b;
                const float recv = dpp_xor1(odd ? v0 : v1);
                const float lo = odd ? recv : v0, hi = odd ? v1 : recv;
                const bool ok = odd ? rowok[2 * pp + 1] : rowok[2 * pp];
                const uint32_t ro = odd ? rowoff[2 * pp + 1] : rowoff[2 * pp];
                if (ok) {
                    if constexpr (BF)
                        *reinterpret_cast<uint32_t *>(dst + (ro + col)) = cvt_bf16x2(lo, hi);   // RNE
                    else
                        *reinterpret_cast<float2 *>(dst + (ro + col)) = make_float2(lo, hi);
                }
            }
        }
    } else {
#pragma unroll
        for (int q = 0; q < L::CT / 16; ++q) {
            const int j = 16 * q + c;
            if (n0 + j >= a.ncols)
                continue;
            const float b = bias[j];
            const uint32_t col = coltab[j];
#pragma unroll
            for (int i = 0; i < 4; ++i)
                if (rowok[i]) {
                    const float v = acc[q][i] + b;
                    if constexpr (BF)
                        dst[rowoff[i] + col] = uint16_t(cvt_bf16x2(v, 0.f));   // RNE
                    else
                        dst[rowoff[i] + col] = v;
                }
        }
    }
}

// LN (bf16, QKV): the rows of A are normalised (LayerNorm over C, affine) once
// they are in registers -- a row's quarters lie in the four lane groups, so its
// sums take two cross-lane steps -- and rounded to bf16 as the norm's own output
// would be: the map is neither written nor read in between.
// Four waves per SIMD, so two workgroups per CU, where the registers allow it.
template <class E, bool PROJ, int KP, bool LN>
constexpr int rk_waves() { return LN || (E::bytes == 4 && (KP > 128 || (PROJ && KP == 128))) ? 2 : 4; }

template <class E, bool PROJ, int KP, bool LN = false>
__global__ void __launch_bounds__(kRkThreads)
__attribute__((amdgpu_waves_per_eu(rk_waves<E, PROJ, KP, LN>())))
block_gemm_rk_kernel(BlockArgs a)
{
    constexpr bool BF = E::bytes == 2;
    using L = RkLds<E, KP>;
    constexpr int KQ = KP / 4;               // contraction slots per lane group
    constexpr int NQ = L::CT / 16;
    __shared__ __align__(16) float lds_all[L::total];
    auto wbuf = [&](int b) { return lds_all + b * L::tile; };
    const int tid = threadIdx.x, lane = tid & 63, g = lane >> 4, c = lane & 15;
    const int wv = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int64_t m0 = int64_t(blockIdx.x) * kRkRows;

    // ---- A: the workgroup's 128 rows are staged in LDS, SR at a time, with
    // coalesced 4-byte loads (lanes take consecutive words of a row; bf16 words
    // hold two elements), then each lane copies its operand slots -- rows
    // 16 wv + c, k = g KQ + s -- into registers.  The stage shares LDS with the W
    // tiles; its offset tables have their own (in the stage's array they would be
    // read again after every store to it: 0.7 us of 12 at 25600 rows, C = 180).
    constexpr int EPW = BF ? 2 : 1;              // elements per 4-byte word
    constexpr int AWL = L::AWL, AP = L::AP;
    __shared__ int rowbase[kRkRows];   // row r's element offset (-1: none)
    __shared__ int colofs[AWL];        // word w's offset in a row
    float *astage = lds_all;
    if (tid < kRkRows) {
        const int64_t row = m0 + tid;
        int base = -1;
        if (row < a.rows) {
            const int wn = int(row / a.N), tt = int(row - int64_t(wn) * a.N);
            base = int(PROJ ? (int64_t(wn) * a.heads * a.N + tt) * a.dh
                            : pixel_of(a, wn, tt) * a.C);
        }
        rowbase[tid] = base;
    }
    __shared__ float lnt[LN ? 2 * KP : 1];   // weight and bias of the norm, zero from C on
    if constexpr (LN) {
        for (int k = tid; k < KP; k += kRkThreads) {
            lnt[k] = k < a.C ? ld<E>(a.lnw, k) : 0.f;
            lnt[KP + k] = k < a.C ? ld<E>(a.lnb, k) : 0.f;
        }
    }
    for (int w = tid; w < AWL; w += kRkThreads) {
        const int k = w * EPW;
        int off = k;
        if constexpr (PROJ) {
            const int hh = k / a.dh;
            off = hh * a.N * a.dh + (k - hh * a.dh);
        }
        colofs[w] = k < a.C ? off : -1;
    }
    // ---- W tiles: the packed image of a tile goes global -> registers -> LDS
    // in 16-byte pieces.  bf16: the image is the LDS tile, padding included, so
    // consecutive lanes copy consecutive pieces.  fp32: a thread takes eight k
    // of a column (two pieces), splits them and stores one piece per plane.
    typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
    constexpr int kPieces = BF ? L::tile / 4 : L::CT * KP / 8;
    constexpr int kPer = (kPieces + kRkThreads - 1) / kRkThreads;
    constexpr int WPP = BF ? 1 : 2;        // loads per piece
    u32x4 wr[kPer][WPP];
    const int nct = (a.ncols + L::CT - 1) / L::CT;
    const u32x4 *wsrc = static_cast<const u32x4 *>(a.wpk);
    auto wfetch = [&](int ct) {
        constexpr int per = 64 / L::CT;    // tiles per 64-column image
        const u32x4 *src = wsrc + int64_t(ct / per) * (L::image / 4) + (ct % per) * kPieces * WPP;
#pragma unroll
        for (int j = 0; j < kPer; ++j) {   // past the image: re-read its last piece
            const int idx = tid + j * kRkThreads;
#pragma unroll
            for (int h = 0; h < WPP; ++h)
                wr[j][h] = src[(idx < kPieces ? idx : kPieces - 1) * WPP + h];
        }
    };
    // fp32: the last tile (of even, of odd ones) with a value that is not finite
    __shared__ int inftile[2];
    if (!BF && tid < 2)
        inftile[tid] = -1;
    auto wstash = [&](int it) {
        u32x4 *dst = reinterpret_cast<u32x4 *>(wbuf(it & 1));
        u16x2 top = {0, 0};
#pragma unroll
        for (int j = 0; j < kPer; ++j) {
            const int idx = tid + j * kRkThreads;
            if (kPer * kRkThreads == kPieces || idx < kPieces) {
                if constexpr (BF) {
                    dst[idx] = wr[j][0];
                } else {
                    float x[8];
#pragma unroll
                    for (int e = 0; e < 8; ++e)
                        x[e] = __uint_as_float(wr[j][e / 4][e % 4]);
                    const int n = idx / (KP / 8), kp = idx - n * (KP / 8);
                    bf8 *d = reinterpret_cast<bf8 *>(dst) + n * (L::PH / 8) + kp;
                    split3_bf16(x, d[0], d[L::plane / 4], d[2 * (L::plane / 4)], top);
                }
            }
        }
        if (!BF && not_finite(top))
            inftile[it & 1] = it;
    };
    // Workgroups start at different column tiles, so that at any moment they
    // read different tiles of W instead of all hitting the same L2 lines.
    const int start = int(blockIdx.x % unsigned(nct));
    auto phys = [&](int i) { return i + start < nct ? i + start : i + start - nct; };
    // The first W tile and the bias are requested now, their latency hidden
    // behind the A stage; the bias of every column is staged in LDS once (a
    // global load in the epilogue would wait behind the next tile's W pieces
    // in flight).
    wfetch(phys(0));
    __shared__ float colbias[3 * KP];
    constexpr int kBiasPer = (3 * KP + kRkThreads - 1) / kRkThreads;
    float bz[kBiasPer];
#pragma unroll
    for (int j = 0; j < kBiasPer; ++j) {
        const int n = tid + j * kRkThreads;
        const int nc = n < a.ncols ? n : a.ncols - 1;
        bz[j] = a.bias ? ld<E>(a.bias, nc) : 0.f;
    }
    bf8 ab[L::NP][KQ / 8];
    u16x2 atop = {0, 0};
    const uint32_t *asrc = static_cast<const uint32_t *>(a.a);
    uint32_t *adst = reinterpret_cast<uint32_t *>(astage);
#pragma unroll
    for (int ph = 0; ph < kRkRows / L::SR; ++ph) {
        __syncthreads();   // the tables are complete; the last stage has been read
        // Each thread copies kPerT words, in batches whose loads are all in
        // flight before the first is waited for (a loop of load, wait, store
        // would chain kPerT memory round trips).
        constexpr int kPerT = L::SR * AWL / kRkThreads;
        constexpr int kBatch = stage_batch(kPerT);
        static_assert(kPerT * kRkThreads == L::SR * AWL, "whole words per thread");
        for (int b0 = 0; b0 < kPerT; b0 += kBatch) {
            uint32_t x[kBatch];
            bool ok[kBatch];
#pragma unroll
            for (int u = 0; u < kBatch; ++u) {
                const int j = tid + (b0 + u) * kRkThreads;
                const int row = j / AWL, w = j - row * AWL;
                const int rb = rowbase[ph * L::SR + row], co = colofs[w];
                ok[u] = rb >= 0 && co >= 0;
                const int e = ok[u] ? rb + co : 0;
                x[u] = asrc[BF ? e >> 1 : e];
            }
#pragma unroll
            for (int u = 0; u < kBatch; ++u) {
                const int j = tid + (b0 + u) * kRkThreads;
                const int row = j / AWL, w = j - row * AWL;
                adst[row * AP + w] = ok[u] ? x[u] : 0u;
            }
        }
        __syncthreads();
        if (16 * wv / L::SR == ph) {   // uniform: this wave's rows
            const float *arow = astage + (16 * wv % L::SR + c) * AP;
#pragma unroll
            for (int s = 0; s < KQ / 8; ++s) {
                if constexpr (BF) {
                    ab[0][s] = *reinterpret_cast<const bf8 *>(arow + (g * KQ + 8 * s) / 2);
                } else {
                    const f4 lo = *reinterpret_cast<const f4 *>(arow + g * KQ + 8 * s);
                    const f4 hi = *reinterpret_cast<const f4 *>(arow + g * KQ + 8 * s + 4);
                    const float x[8] = {lo[0], lo[1], lo[2], lo[3], hi[0], hi[1], hi[2], hi[3]};
                    split3_bf16(x, ab[0][s], ab[L::NP / 2][s], ab[L::NP - 1][s], atop);
                }
            }
        }
    }
    const bool rowsinf = !BF && __builtin_amdgcn_ballot_w64(not_finite(atop)) != 0;
    if constexpr (LN) {
        static_assert(BF, "LayerNorm in the prologue: bf16");
        // The rows stay packed between the three passes over them: without
        // this the unpacked values of the first pass are kept, and spilled.
        auto keep_packed = [&]() {
#pragma unroll
            for (int s = 0; s < KQ / 8; ++s)
                asm volatile("" : "+v"(ab[0][s]));
        };
        float sum = 0.f, sq = 0.f;
#pragma unroll
        for (int s = 0; s < KQ / 8; ++s) {
            float f[8];
            unpack_bf8(ab[0][s], f);
#pragma unroll
            for (int e = 0; e < 8; ++e)
                sum += f[e];   // zero from k = C on
        }
        const float mean = sum_groups(sum) / float(a.C);
        keep_packed();
#pragma unroll
        for (int s = 0; s < KQ / 8; ++s) {
            float f[8];
            unpack_bf8(ab[0][s], f);
#pragma unroll
            for (int e = 0; e < 8; ++e) {
                const float d = g * KQ + 8 * s + e < a.C ? f[e] - mean : 0.f;
                sq = fmaf(d, d, sq);
            }
        }
        const float rstd = 1.f / sqrtf(sum_groups(sq) / float(a.C) + a.eps);
        keep_packed();
#pragma unroll
        for (int s = 0; s < KQ / 8; ++s) {
            float f[8];
            unpack_bf8(ab[0][s], f);
            const float *lw = lnt + g * KQ + 8 * s, *lb = lw + KP;
            U16B u;
#pragma unroll
            for (int p = 0; p < 4; ++p)   // weight and bias are zero from C on
                u.w[p] = cvt_bf16x2(fmaf((f[2 * p] - mean) * rstd, lw[2 * p], lb[2 * p]),
                                    fmaf((f[2 * p + 1] - mean) * rstd, lw[2 * p + 1], lb[2 * p + 1]));
            ab[0][s] = __builtin_bit_cast(bf8, u);
            __builtin_amdgcn_sched_barrier(0);   // few table reads in flight: registers
        }
    }
    __syncthreads();   // the stage becomes the W tiles

    // Column part of the destination for the columns of the current tile,
    // from out0: (QKV) output tensor `which` at which * ostride, head h,
    // feature f -> h N d_h + f; (PROJ) the column.
    __shared__ uint32_t coltab[2][L::CT];
    auto cfill = [&](int ct, int buf) {
        if (tid < L::CT) {
            const int n = L::CT * ct + tid;
            int which = 0, col = n;
            if constexpr (!PROJ) {
                which = n / a.C;
                const int cc = n - which * a.C;
                const int hh = cc / a.dh;
                col = hh * a.N * a.dh + (cc - hh * a.dh);
            }
            coltab[buf][tid] = uint32_t(which * a.ostride + col);
        }
    };

    // Row part of the destination of this lane's output rows 4g + i: QKV
    // (window wn, token tt) -> wn N C + tt d_h; PROJ -> pixel C.  Offsets are
    // unsigned 32-bit (tensors under 2^31 elements); rows past the end are
    // not stored.
    uint32_t rowoff[4];
    bool rowok[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const int row = int(m0) + 16 * wv + 4 * g + i;   // rows < 2^31
        rowok[i] = row < a.rows;
        const int rr = rowok[i] ? row : 0;
        const int wn = rr / a.N, tt = rr - wn * a.N;
        rowoff[i] = uint32_t(PROJ ? pixel_of(a, wn, tt) * a.C
                                  : int64_t(wn) * a.N * a.C + int64_t(tt) * a.dh);
    }

#pragma unroll
    for (int j = 0; j < kBiasPer; ++j) {
        const int n = tid + j * kRkThreads;
        if (n < a.ncols)
            colbias[n] = bz[j];
    }
    wstash(0);
    cfill(phys(0), 0);
    __syncthreads();
    for (int it = 0; it < nct; ++it) {
        const int ct = phys(it);
        const bool more = it + 1 < nct;   // uniform
        if (more)
            wfetch(phys(it + 1));
        const float *wt = wbuf(it & 1);
        f4 acc[NQ];
        const uint16_t *h = reinterpret_cast<const uint16_t *>(wt);
        tile_product<L, KQ / 8>(ab, h + c * L::PH + g * KQ, 8, acc);
        if constexpr (!BF) {
            if (rowsinf || __builtin_amdgcn_readfirstlane(inftile[it & 1]) == it)   // uniform
                tile_product_f32<L, KQ / 8>(ab, h + c * L::PH + g * KQ, 8, acc);
        }
        // The next tile goes to the idle buffer before this tile's stores are
        // issued: the wait for its loads counts every earlier vector memory
        // operation, stores included, so stashing after the stores would
        // wait for their completion on every tile.
        if (more) {
            wstash(it + 1);
            cfill(phys(it + 1), (it + 1) & 1);
        }
        store_tile<E, L>(a, acc, L::CT * ct, c, rowoff, rowok, colbias + L::CT * ct, coltab[it & 1]);
        __syncthreads();
    }
}

// Weight-resident GEMM for C <= 256: a workgroup keeps a group of columns of W in
// LDS for its whole life, and its eight waves walk over row tiles of 16 on their
// own -- rows straight from memory into the operand registers (lane (g, c): row
// c, k = 32 s + 8 g ..), the next tile's rows in flight while this one is
// multiplied, no barrier after W has arrived.  Streaming W past resident rows
// instead (64 columns at a time, one barrier each) chained every step to the
// stores of the one before: memory operations complete in order, so the wait for
// the next W tile waited for them too.
// fp32: A is split into three bf16 terms in registers, W on its way into LDS.
// LN (bf16, QKV): the rows are normalised (LayerNorm over C, affine) in registers
// -- a row lies in the four lane groups, so its sums take two cross-lane steps --
// and rounded to bf16 as the norm's own output would be: the map is neither
// written nor read in between.
// launch_rk_ln() says where this measured faster.
template <class E, bool PROJ, int KP, bool LN = false>
__global__ void __launch_bounds__(kRwThreads)
__attribute__((amdgpu_waves_per_eu(E::bytes == 2 && !LN ? 4 : 2)))
block_gemm_rw_kernel(BlockArgs a)
{
    constexpr bool BF = E::bytes == 2;
    using L = RwLds<E, KP>;
    constexpr int KS = KP / 32, T = kRwThreads, NQ = L::CT / 16;
    typedef typename E::T ET;
    typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
    extern __shared__ __align__(16) float lds_all[];
    const int tid = threadIdx.x, lane = tid & 63, g = lane >> 4, c = lane & 15;
    const int wv = __builtin_amdgcn_readfirstlane(tid >> 6);
    int *colofs = reinterpret_cast<int *>(lds_all);            // element k's offset in a row of A
    float *lnt = lds_all + KP;                                 // LN: weight, bias (zero from C on)
    float *colbias = lnt + (LN ? 2 * KP : 0);
    uint32_t *coltab = reinterpret_cast<uint32_t *>(colbias + a.ctiles * L::CT);
    float *wbase = reinterpret_cast<float *>(coltab + a.ctiles * L::CT);

    // Block -> (row block, column group): the groups of one row block run on one
    // XCD and share its L2 for the rows.
    const int total = int(gridDim.x), q8 = total / 8, r8 = total % 8;
    const int xcd = int(blockIdx.x) % 8, local = int(blockIdx.x) / 8;
    const int lb = (xcd < r8 ? xcd * (q8 + 1) : r8 * (q8 + 1) + (xcd - r8) * q8) + local;
    const int rb = lb / a.groups, grp = lb - rb * a.groups, rblocks = total / a.groups;
    const int t0 = grp * a.ctiles;                             // first CT-column tile
    const int nt = min(a.ctiles, (a.ncols + L::CT - 1) / L::CT - t0);

    // ---- rows
    const int ntiles = int((a.rows + 15) / 16), stride = rblocks * (T / 64);
    uint32_t inoff = 0, outoff = 0;   // of lane's row c, tile rt + g stride
    auto rows4 = [&](int rt) {
        const int64_t r64 = int64_t(rt + int64_t(g) * stride) * 16 + c;
        const uint32_t row = uint32_t(r64 < a.rows ? r64 : a.rows - 1);
        const uint32_t wn = row / uint32_t(a.N), tt = row - wn * uint32_t(a.N);
        const uint32_t per = uint32_t(a.nwy) * uint32_t(a.nwx);
        const uint32_t b = wn / per, wi = wn - b * per;
        const uint32_t wy = wi / uint32_t(a.nwx), wx = wi - wy * uint32_t(a.nwx);
        const uint32_t ty = tt / uint32_t(a.w), tx = tt - ty * uint32_t(a.w);
        uint32_t y = wy * a.w + ty + a.shift, x = wx * a.w + tx + a.shift;
        y -= y >= uint32_t(a.H) ? a.H : 0;
        x -= x >= uint32_t(a.W) ? a.W : 0;
        const uint32_t pix = ((b * a.H + y) * a.W + x) * uint32_t(a.C);
        inoff = PROJ ? (wn * a.heads * a.N + tt) * uint32_t(a.dh) : pix;
        outoff = PROJ ? pix : wn * uint32_t(a.N) * uint32_t(a.C) + tt * uint32_t(a.dh);
    };
    const ET *asrc = static_cast<const ET *>(a.a);
    constexpr int RW = BF ? 4 : 8;    // words per step
    uint32_t raw[KS][RW], rawn[KS][RW];
    // Rows as words: whole 16-byte pieces where the eight k of a step are adjacent
    // (QKV; PROJ with d_h a multiple of 8), pairs (or single fp32 elements) of
    // known offsets otherwise; slots from C on are zeroed when they are used.
    const bool vec8 = !PROJ || a.dh % 8 == 0, pairs = BF || (a.C % 2 == 0 && (!PROJ || a.dh % 2 == 0));
    auto fetch = [&](uint32_t base, uint32_t (&x)[KS][RW]) {
        const ET *p = asrc + base;
#pragma unroll
        for (int s = 0; s < KS; ++s) {
            const int k0 = 32 * s + 8 * g;
            if (vec8 && (s < L::full || 32 * s + 32 <= a.C)) {   // uniform
                const ET *q = p + (PROJ ? colofs[k0] : k0);
#pragma unroll
                for (int h = 0; h < RW / 4; ++h) {
                    const U16B v = *reinterpret_cast<const U16B *>(q + 4 * h);
#pragma unroll
                    for (int w = 0; w < 4; ++w)
                        x[s][4 * h + w] = v.w[w];
                }
            } else if (pairs) {   // uniform
#pragma unroll
                for (int w = 0; w < 4; ++w) {
                    const int o = max(PROJ ? colofs[k0 + 2 * w] : (k0 + 2 * w < a.C ? k0 + 2 * w : 0), 0);
                    if constexpr (BF) {
                        x[s][w] = *reinterpret_cast<const uint32_t *>(p + o);
                    } else {
                        struct __attribute__((aligned(4))) P2 { uint32_t w[2]; };
                        const P2 v = *reinterpret_cast<const P2 *>(p + o);
                        x[s][2 * w] = v.w[0];
                        x[s][2 * w + 1] = v.w[1];
                    }
                }
            } else if constexpr (!BF) {
#pragma unroll
                for (int w = 0; w < 8; ++w)
                    x[s][w] = __float_as_uint(p[max(colofs[k0 + w], 0)]);
            }
        }
    };

    // ---- prologue: W's pieces and the first rows are requested together, so
    // that one memory latency covers them, then W goes to LDS.
    // bf16: the packed image is the LDS image.  fp32: eight k of a column at a
    // time (two pieces), split, one 16-byte piece per plane.
    constexpr int WPP = BF ? 1 : 2, kUnit = BF ? L::tile / 4 : L::CT * KP / 8;
    constexpr int kPer = (L::NT * kUnit + T - 1) / T;
    const int units = nt * kUnit;
    const u32x4 *wsrc = static_cast<const u32x4 *>(a.wpk);
    constexpr int kBatch = kPer * WPP <= 12 ? kPer : 12 / WPP;   // pieces in flight
    u32x4 wx[kBatch][WPP];
    auto wfetch = [&](int j0) {
#pragma unroll
        for (int u = 0; u < kBatch; ++u) {
            const int j = min(j0 + tid + u * T, units - 1);
            if constexpr (BF) {
                wx[u][0] = wsrc[int64_t(t0) * kUnit + j];
            } else {
                const int col = t0 * L::CT + j / (KP / 8), kp = j % (KP / 8);
                const u32x4 *src = wsrc + int64_t(col / 64) * (RkLds<E, KP>::image / 4) +
                                   ((col % 64) * KP + 8 * kp) / 4;
#pragma unroll
                for (int h = 0; h < WPP; ++h)
                    wx[u][h] = src[h];
            }
        }
    };
    __shared__ int winf;   // fp32: this block's columns of W hold a value that is not finite
    if (!BF && tid == 0)
        winf = 0;
    auto wstash = [&](int j0) {
        u16x2 top = {0, 0};
#pragma unroll
        for (int u = 0; u < kBatch; ++u) {
            const int j = j0 + tid + u * T;
            if (j < units) {
                if constexpr (BF) {
                    reinterpret_cast<u32x4 *>(wbase)[j] = wx[u][0];
                } else {
                    float f[8];
#pragma unroll
                    for (int e = 0; e < 8; ++e)
                        f[e] = __uint_as_float(wx[u][e / 4 % WPP][e % 4]);
                    const int cj = j / (KP / 8), kp = j % (KP / 8);
                    bf8 *d = reinterpret_cast<bf8 *>(wbase + (cj / L::CT) * L::tile) +
                             (cj % L::CT) * (L::PH / 8) + kp;
                    split3_bf16(f, d[0], d[L::plane / 4], d[2 * (L::plane / 4)], top);
                }
            }
        }
        if (!BF && not_finite(top))
            winf = 1;
    };
    wfetch(0);
    for (int k = tid; k < KP; k += T) {
        int off = k;
        if constexpr (PROJ) {
            const int hh = k / a.dh;
            off = hh * a.N * a.dh + (k - hh * a.dh);
        }
        colofs[k] = k < a.C ? off : -1;
        if constexpr (LN) {
            lnt[k] = k < a.C ? ld<E>(a.lnw, k) : 0.f;
            lnt[KP + k] = k < a.C ? ld<E>(a.lnb, k) : 0.f;
        }
    }
    // Column part of the destination, from out0: (QKV) output tensor `which` at
    // which * ostride, head h, feature f -> h N d_h + f; (PROJ) the column.
    for (int j = tid; j < nt * L::CT; j += T) {
        const int n = t0 * L::CT + j;
        int which = 0, col = n;
        if constexpr (!PROJ) {
            which = n / a.C;
            const int cc = n - which * a.C;
            const int hh = cc / a.dh;
            col = hh * a.N * a.dh + (cc - hh * a.dh);
        }
        coltab[j] = uint32_t(which * a.ostride + col);
        colbias[j] = a.bias && n < a.ncols ? ld<E>(a.bias, n) : 0.f;
    }
    int rt = rb * (T / 64) + wv;
    rows4(rt);   // clamped past the last row
    int sub = 0;   // which of the four tiles of rows4 is current
    if (PROJ || !BF)
        __syncthreads();   // colofs, winf
    fetch(__shfl(inoff, c, 64), raw);
    wstash(0);
    for (int j0 = kBatch * T; j0 < units; j0 += kBatch * T) {
        wfetch(j0);
        wstash(j0);
    }
    __syncthreads();
    const bool colsinf = !BF && __builtin_amdgcn_readfirstlane(winf) != 0;
    for (; rt < ntiles; rt += stride) {
        // output offsets of rows 4g + i, then the next tile's rows
        uint32_t rowoff[4];
        bool rowok[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            rowoff[i] = __shfl(outoff, 16 * sub + 4 * g + i, 64);
            rowok[i] = int64_t(rt) * 16 + 4 * g + i < a.rows;
        }
        // operands of this tile, zero from C on
        bf8 ab[L::NP][KS];
#pragma unroll
        for (int s = 0; s < KS; ++s) {
            const int k0 = 32 * s + 8 * g;
            if (s >= L::full && 32 * s + 32 > a.C) {   // uniform
                constexpr int EW = BF ? 2 : 1;   // elements per word
#pragma unroll
                for (int w = 0; w < RW; ++w)
                    raw[s][w] = k0 + EW * w < a.C ? raw[s][w] : 0u;
            }
        }
        u16x2 atop = {0, 0};
        auto take = [&](auto clean) {
#pragma unroll
            for (int s = 0; s < KS; ++s) {
                if constexpr (BF) {
                    const U16B u = {{raw[s][0], raw[s][1], raw[s][2], raw[s][3]}};
                    ab[0][s] = __builtin_bit_cast(bf8, u);
                } else {
                    float f[8];
#pragma unroll
                    for (int e = 0; e < 8; ++e)
                        f[e] = __uint_as_float(raw[s][e]);
                    split3_bf16<clean>(f, ab[0][s], ab[L::NP / 2][s], ab[L::NP - 1][s], atop);
                }
            }
        };
        take(std::false_type{});
        const bool inf = !BF && (colsinf || __builtin_amdgcn_ballot_w64(not_finite(atop)) != 0);
        if constexpr (!BF) {
            if (inf)   // uniform
                take(std::true_type{});
        }
        if (++sub == 4) {   // uniform
            sub = 0;
            rows4(rt + stride);
        }
        if (rt + stride < ntiles)   // uniform
            fetch(__shfl(inoff, 16 * sub + c, 64), rawn);
        if constexpr (LN) {
            static_assert(BF, "LayerNorm in the prologue: bf16");
            // The rows stay packed between the three passes over them: without
            // this the unpacked values of the first pass are kept, and spilled.
            auto keep_packed = [&]() {
#pragma unroll
                for (int s = 0; s < KS; ++s)
                    asm volatile("" : "+v"(ab[0][s]));
            };
            float sum = 0.f, sq = 0.f;
#pragma unroll
            for (int s = 0; s < KS; ++s) {
                float f[8];
                unpack_bf8(ab[0][s], f);
#pragma unroll
                for (int e = 0; e < 8; ++e)
                    sum += f[e];
            }
            const float mean = sum_groups(sum) / float(a.C);
            keep_packed();
#pragma unroll
            for (int s = 0; s < KS; ++s) {
                float f[8];
                unpack_bf8(ab[0][s], f);
#pragma unroll
                for (int e = 0; e < 8; ++e) {
                    const float d = f[e] - mean;
                    sq = fmaf(d, s < L::full || 32 * s + 8 * g + e < a.C ? d : 0.f, sq);
                }
            }
            const float rstd = 1.f / sqrtf(sum_groups(sq) / float(a.C) + a.eps);
            keep_packed();
#pragma unroll
            for (int s = 0; s < KS; ++s) {
                float f[8];
                unpack_bf8(ab[0][s], f);
                const float *lw = lnt + 32 * s + 8 * g, *lb = lw + KP;
                U16B u;
#pragma unroll
                for (int p = 0; p < 4; ++p)   // weight and bias are zero from C on
                    u.w[p] = cvt_bf16x2(
                        fmaf((f[2 * p] - mean) * rstd, lw[2 * p], lb[2 * p]),
                        fmaf((f[2 * p + 1] - mean) * rstd, lw[2 * p + 1], lb[2 * p + 1]));
                ab[0][s] = __builtin_bit_cast(bf8, u);
                __builtin_amdgcn_sched_barrier(0);   // few table reads in flight: registers
            }
        }
        for (int ct = 0; ct < nt; ++ct) {
            const uint16_t *h = reinterpret_cast<const uint16_t *>(wbase + ct * L::tile);
            f4 acc[NQ];
            tile_product<L, KS>(ab, h + c * L::PH + 8 * g, 32, acc);
            if constexpr (!BF) {
                if (inf)   // uniform
                    tile_product_f32<L, KS>(ab, h + c * L::PH + 8 * g, 32, acc);
            }
            store_tile<E, L>(a, acc, (t0 + ct) * L::CT, c, rowoff, rowok, colbias + ct * L::CT,
                             coltab + ct * L::CT);
        }
#pragma unroll
        for (int s = 0; s < KS; ++s)
#pragma unroll
            for (int w = 0; w < RW; ++w)
                raw[s][w] = rawn[s][w];
    }
}

// Column groups and row blocks: groups as wide as LDS allows (fewer passes over
// the rows), narrower ones while that leaves compute units without a block, and
// as many row blocks as fit on the chip at once.
template <class E, bool PROJ, int KP, bool LN>
void launch_rw_ln(BlockArgs &a, hipStream_t stream)
{
    using L = RwLds<E, KP>;
    const int nct = (a.ncols + L::CT - 1) / L::CT;
    const int64_t want = (a.rows + 127) / 128;       // blocks of eight row tiles
    int per = L::NT;
    while (per > 1 && want * ((nct + per - 1) / per) < 256)
        per = (per + 1) / 2;
    a.groups = (nct + per - 1) / per;
    a.ctiles = (nct + a.groups - 1) / a.groups;
    a.groups = (nct + a.ctiles - 1) / a.ctiles;
    const size_t lds = 4 * (size_t(KP) * (LN ? 3 : 1) + size_t(a.ctiles) * (2 * L::CT + L::tile));
    const int64_t fit = 256 * (lds * 2 <= 160 * 1024 ? 2 : 1);
    int64_t rblocks = fit / a.groups;
    if (rblocks < 1)
        rblocks = 1;
    if (rblocks > want)
        rblocks = want;
    hipLaunchKernelGGL((block_gemm_rw_kernel<E, PROJ, KP, LN>), dim3(unsigned(rblocks * a.groups)),
                       dim3(kRwThreads), lds, stream, a);
}

template <class E, bool PROJ, int KP, bool LN>
void launch_rk_ln(BlockArgs &a, hipStream_t stream)
{
    const int64_t blocks = (a.rows + kRkRows - 1) / kRkRows;
    // Few rows (fewer row blocks than half the compute units): column groups on
    // more of the chip.  With more rows every group's pass over them costs more than
    // the streaming's waits.  Whole blocks of 8 x 8 windows, row-resident against
    // weight-resident (us), at 64, 120, 136 and 512 row blocks:
    //   bf16 C =  64  19.4/17.9  22.4/22.5  23.7/24.3  31.7/34.6
    //   bf16 C = 180  41.0/29.9  45.9/41.6  46.2/42.6  74.2/75.3
    //   bf16 C = 256  51.9/39.6  56.4/58.1  58.6/63.0  100/129
    //   fp32 C =  64  29.3/26.4  34.7/32.0  37.6/39.3  50.2/52.9
    //   fp32 C = 128  51.2/43.4  55.1/64.4  58.4/69.6  93.5/139
    //   fp32 C = 256  131/63.0   139/107    144/120    303/332
    // fp32 from 65 to 128 channels changes sides earlier (80 row blocks: 53.1/54.8,
    // C = 96 47.1/45.1; 96: 53.4/63.1, 49.1/55.3).  fp32 from 129 to 192 channels is
    // weight-resident at any size (C = 180: 86.1/67.7 at 96, 185/183 at 512, 259/232 at
    // 648): 128 columns a group fit there, and the row-resident kernel has one
    // workgroup's registers per CU to hide latency.
    constexpr int kFew = E::bytes == 4 && KP == 128 ? 88 : 128;
    if constexpr (!(E::bytes == 4 && KP == 192)) {
        if (blocks >= kFew) {
            hipLaunchKernelGGL((block_gemm_rk_kernel<E, PROJ, KP, LN>), dim3(unsigned(blocks)),
                               dim3(kRkThreads), 0, stream, a);
            return;
        }
    }
    launch_rw_ln<E, PROJ, KP, LN>(a, stream);
}

template <class E, bool PROJ, int KP>
void launch_rk(BlockArgs &a, hipStream_t stream)
{
    if constexpr (!PROJ && E::bytes == 2) {
        if (a.lnw) {
            launch_rk_ln<E, PROJ, KP, true>(a, stream);
            return;
        }
    }
    launch_rk_ln<E, PROJ, KP, false>(a, stream);
}

template <class E, bool PROJ>
bool try_rk(const BlockArgs &a, hipStream_t stream)
{
    if (!a.wpk)
        return false;   // the weights were not packed (C > 256)
    if (a.rows * int64_t(a.C) >= (int64_t(1) << 31) ||
        int64_t(a.C) * a.ncols >= (int64_t(1) << 31))
        return false;   // 32-bit element offsets
    if ((a.rows + kRkRows - 1) / kRkRows * kRkThreads >= (int64_t(1) << 32))
        return false;   // fewer than 2^32 work-items in the grid
    // A as 4-byte words: bf16 needs an even C, and in PROJ an even d_h (a word
    // never straddles two heads); the A base 4-byte aligned
    if (uintptr_t(a.a) % 4 != 0 || (E::bytes == 2 && (a.C % 2 != 0 || (PROJ && a.dh % 2 != 0))))
        return false;
    // One output base: Q, K, V at a uniform element stride from out0, every
    // offset under 2^32 elements.
    BlockArgs b = a;
    b.ostride = 0;
    if constexpr (!PROJ) {
        const int64_t s1 = static_cast<const char *>(a.out1) - static_cast<const char *>(a.out0);
        const int64_t s2 = static_cast<const char *>(a.out2) - static_cast<const char *>(a.out1);
        if (s1 != s2 || s1 < 0 || s1 % E::bytes != 0)
            return false;
        b.ostride = s1 / E::bytes;
        if (3 * b.ostride >= (int64_t(1) << 32) || b.ostride < a.rows * int64_t(a.C))
            return false;
    }
    // paired column stores: even widths, outputs aligned to two elements
    const uintptr_t al = 2 * E::bytes;
    b.pair = a.ncols % 2 == 0 && a.dh % 2 == 0 && uintptr_t(a.out0) % al == 0 &&
             (PROJ || (uintptr_t(a.out1) % al == 0 && uintptr_t(a.out2) % al == 0));
    if (a.C <= 32)
        launch_rk<E, PROJ, 32>(b, stream);
    else if (a.C <= 64)
        launch_rk<E, PROJ, 64>(b, stream);
    else if (a.C <= 128)
        launch_rk<E, PROJ, 128>(b, stream);
    else if (a.C <= 192)
        launch_rk<E, PROJ, 192>(b, stream);
    else if (a.C <= 256)
        launch_rk<E, PROJ, 256>(b, stream);
    else
        return false;
    return true;
}

template <class E, bool PROJ>
hipError_t launch_gemm(const BlockArgs &a, hipStream_t stream)
{
    if (try_rk<E, PROJ>(a, stream))
        return hipGetLastError();
    // The kernels below have no LayerNorm.  layer_supported() and the plan of the
    // workspace keep every layer on the path above.
    if (a.lnw)
        return hipErrorInvalidValue;
    // fp32 with no more 64 x 64 tiles than compute units: those are done in one go,
    // and a 128 x 128 tile takes longer than one of them.  Whole blocks, wide kernel
    // -> this rule: C = 264, 1024 rows (208 tiles of the QKV product) 62 -> 49 us, C = 1024,
    // 256 rows (192) 179 -> 161 us; C = 384, 1024 rows (288) 77 us with the wide kernel, 92
    // without.  (bf16: the wide kernel is faster at every size.)
    const bool few = E::bytes == 4 && a.rtiles * a.ctiles <= 256;
    if (!few && wide_ok(a, PROJ)) {
        using F = WideCfg<E>;
        BlockArgs b = a;
        b.rtiles = int((a.rows + F::BM - 1) / F::BM);
        b.ctiles = (a.ncols + F::BN - 1) / F::BN;
        hipLaunchKernelGGL((block_gemm_wide_kernel<E, PROJ>),
                           dim3(unsigned(b.rtiles) * unsigned(b.ctiles)), dim3(256), 0, stream, b);
        return hipGetLastError();
    }
    const unsigned blocks = unsigned(a.rtiles) * unsigned(a.ctiles);
    hipLaunchKernelGGL((block_gemm_kernel<E, PROJ>), dim3(blocks), dim3(256), 0, stream, a);
    return hipGetLastError();
}

}  // namespace

bool block_gemm_supported(int64_t rows, int C)
{
    const int64_t rt = (rows + kBM - 1) / kBM, ct = (3 * int64_t(C) + kBN - 1) / kBN;
    return rt * ct * 256 < (int64_t(1) << 32);
}

// Contraction length of the register-resident kernel for C (0: not used).
static int rk_kp(int C)
{
    return C <= 32 ? 32 : C <= 64 ? 64 : C <= 128 ? 128 : C <= 192 ? 192 : C <= 256 ? 256 : 0;
}

template <class E, int KP>
size_t wpack_words(int ncols)
{
    return size_t((ncols + 63) / 64) * RkLds<E, KP>::image;
}

template <class E>
size_t wpack_words_e(int C, int ncols)
{
    switch (rk_kp(C)) {
    case 32: return wpack_words<E, 32>(ncols);
    case 64: return wpack_words<E, 64>(ncols);
    case 128: return wpack_words<E, 128>(ncols);
    case 192: return wpack_words<E, 192>(ncols);
    case 256: return wpack_words<E, 256>(ncols);
    default: return 0;
    }
}

size_t block_wpack_bytes(int C, int ncols, int dtype)
{
    return 4 * (dtype == 0 ? wpack_words_e<F32>(C, ncols) : wpack_words_e<BF16>(C, ncols));
}

template <class E, int KP>
void launch_wpack_k(const WPackArgs &p, hipStream_t stream)
{
    const int64_t pieces = (int64_t(p.words0) + p.words1) / 4;   // tiles are whole pieces
    hipLaunchKernelGGL((block_wpack_kernel<E, KP>), dim3(unsigned((pieces + 255) / 256)),
                       dim3(256), 0, stream, p);
}

template <class E>
void launch_wpack_e(const WPackArgs &p, hipStream_t stream)
{
    switch (rk_kp(p.C)) {
    case 32: launch_wpack_k<E, 32>(p, stream); break;
    case 64: launch_wpack_k<E, 64>(p, stream); break;
    case 128: launch_wpack_k<E, 128>(p, stream); break;
    case 192: launch_wpack_k<E, 192>(p, stream); break;
    default: launch_wpack_k<E, 256>(p, stream); break;
    }
}

hipError_t launch_block_wpack(const void *wqkv, const void *wproj, int C, int dtype, void *pk_qkv,
                              void *pk_proj, hipStream_t stream)
{
    WPackArgs p;
    p.w0 = wqkv;
    p.w1 = wproj;
    p.d0 = static_cast<uint32_t *>(pk_qkv);
    p.d1 = static_cast<uint32_t *>(pk_proj);
    p.C = C;
    p.words0 = int(block_wpack_bytes(C, 3 * C, dtype) / 4);
    p.words1 = int(block_wpack_bytes(C, C, dtype) / 4);
    if (dtype == 0)
        launch_wpack_e<F32>(p, stream);
    else
        launch_wpack_e<BF16>(p, stream);
    return hipGetLastError();
}

hipError_t launch_block_gemm(const BlockGemm &g, hipStream_t stream)
{
    BlockArgs a;
    a.rows = g.rows;
    a.H = g.H;
    a.W = g.W;
    a.C = g.C;
    a.heads = g.heads;
    a.dh = g.C / g.heads;
    a.w = g.w;
    a.N = g.w * g.w;
    a.shift = g.shift;
    a.nwx = g.W / g.w;
    a.nwy = g.H / g.w;
    a.ncols = g.proj ? g.C : 3 * g.C;
    a.rtiles = int((g.rows + kBM - 1) / kBM);
    a.ctiles = (a.ncols + kBN - 1) / kBN;
    a.a = g.a;
    a.wt = g.wt;
    a.wpk = g.wpk;
    a.bias = g.bias;
    a.out0 = g.out0;
    a.out1 = g.out1;
    a.out2 = g.out2;
    a.pair = false;
    a.ostride = 0;
    a.lnw = g.lnw;
    a.lnb = g.lnb;
    a.eps = g.eps;
    if (g.dtype == 0)
        return g.proj ? launch_gemm<F32, true>(a, stream) : launch_gemm<F32, false>(a, stream);
    return g.proj ? launch_gemm<BF16, true>(a, stream) : launch_gemm<BF16, false>(a, stream);
}

}  // namespace nystra
