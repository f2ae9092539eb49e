// The row-parallel linear layer with the compression in its epilogue (paper Sec. 2: device i
// computes f^(i)(x^(i)) = x^(i) W^(i) and sends C^(i) of it; Sec. 3, "Selecting High Precision
// Features": the selection before the exchange is the method's overhead).  The partial sums
// never reach memory: a workgroup's tile of the product is rounded to bf16 in registers,
// and group statistics, codes and the bf16 features go straight to the message.
//
// What makes that possible without a gather: the selected features are static (Sec. 3), and so
// are the weights, so the weight rows are reordered once, offline, into message order -- the
// r features that are quantised, ascending, then the k that stay bf16 (k_gemm_weights).  The
// product then comes out compacted: output feature n < r is compacted feature n, its group is
// n / G, and the tail n >= r is the outlier section.
//
// The product itself is a dense contraction: bf16 MFMA 32x32x16, fp32 accumulators.  The
// operands are "k-contiguous" on both sides (X [T][K], Wp [E][K]), the weights are the MFMA's
// row operand and the tokens its column operand, so that a lane's 16 accumulators of a 32x32
// block are 16 features of ONE token: the per-token statistics stay inside a lane (and its
// partner 32 lanes on), and the nibbles of a chunk sit in at most two lanes.
//
// How it is fed.  A wave owns 128 features x 32 NTB tokens, so a k-step of 16 costs it 4 + NTB
// fragment reads from LDS for 4 NTB products (with 64 x 64 per wave, LDS reads alone take as long
// as the products).  Operands go straight from memory to LDS (buffer loads with the LDS bit) in
// stages of 32 k, through a ring of 5 or more stages, so that a stage has 2 to 5 stages' time to
// arrive; the two stages that share the rows' cache lines are loaded together, the second one
// from L1.  Between two products stands at most one fetch or load wherever there are as many
// products, in that order (the scheduler is pinned), and a stage costs one barrier.  One
// workgroup holds a compute unit, one wave a SIMD.
//
// What bounds it, at T = 2048, E = 5120, K = 1728 (one MI355X): 37.9 to 38.5 us a launch timed by itself, 39.4 to 40.6
// behind other kernels (920 to 890 TFLOP/s), 43.8 in a loop of nothing else, which the chip's power limit slows down;
// operands that went through registers, 64 x 64 per wave and two barriers a stage took 54 to 61.  The matrix cores are
// busy for 62 % of a wave's 66 thousand cycles; the rest is mostly the ends (first loads, epilogue), which a single
// round of tiles cannot hide.  With few tokens a tile is bound by its stages, 0.19 us each from barrier to barrier: k_gemm_few
// instead.
#include <algorithm>
#include <atomic>

#include "tpq_device.h"
#include "tpq_internal.h"

namespace tpq {

typedef __bf16 bf16x8_t __attribute__((ext_vector_type(8)));
typedef float f32x16 __attribute__((ext_vector_type(16)));

// Rows of Wt ([E][ldW], one row per output feature) -> Wp [E][K] in message order.
__global__ __launch_bounds__(256) void k_gemm_weights(const uint8_t *plan, int E, int k, int G, int r,
                                                      int off_idx, int off_src, const uint16_t *Wt,
                                                      int64_t ldW, int K, uint16_t *Wp)
{
    if (plan_header_bad(plan, E, k, G)) return;
    const int n = blockIdx.x;
    const int col = n < r ? reinterpret_cast<const uint16_t *>(plan + off_src)[n]
                          : reinterpret_cast<const int32_t *>(plan + off_idx)[n - r];
    const u32x4 *src = reinterpret_cast<const u32x4 *>(Wt + static_cast<int64_t>(col) * ldW);
    u32x4 *dst = reinterpret_cast<u32x4 *>(Wp + static_cast<int64_t>(n) * K);
    for (int p = threadIdx.x; p < K / 8; p += 256) dst[p] = src[p];
}

struct GemmArgs {
    const uint16_t *X;
    int64_t ldX, T;
    const uint16_t *Wp;
    int32_t K, E, k, G, r, ng;
    uint8_t *codes, *scale, *zero, *outl;
    int64_t pitch_codes, pitch_meta, pitch_outl;
    uint16_t *Ymsg;  // optional: the rounded product itself, [T][ldYm] in message order
    int64_t ldYm;
};

// Tile of a workgroup: FW x TW waves, each with 128 features x 32 NTB tokens.  A group (up to 128 features) lies in
// one wave, groups of 256 in the two waves of FW = 2.
constexpr int kTileBK = 32;  // k per stage
template <int FW, int TW, int NTB>
struct TileShape {
    static constexpr int waves = FW * TW, threads = 64 * waves;
    static constexpr int ft = 128 * FW, tt = 32 * NTB * TW;          // features and tokens of the tile
    static constexpr int stage = (ft + tt) * kTileBK * 2;            // LDS bytes of a stage
    static constexpr int nla = ft / (16 * waves), nl = nla + tt / (16 * waves);  // loads of a wave per stage: weights, all
    static constexpr int n1 = (2 * nl + 2) / 3, n2 = (2 * nl + 1 - n1) / 2 + n1;  // loads of a pair: three phases' shares
    // pairs of stages on their way in: as many as LDS holds beside the half pair that is being freed, and the wait
    // counter (63) can tell apart
    static constexpr int pairs_lds = (163840 / stage - 1) / 2, pairs_cnt = (63 - n2) / (2 * nl) + 2;
    static constexpr int pairs = pairs_lds < pairs_cnt ? pairs_lds : pairs_cnt;
    static constexpr int nbuf = 2 * pairs + 1;
    static constexpr int lds = nbuf * stage;
    static_assert(pairs >= 2 && tt * (ft * 2 + 16) <= lds, "tile fits");
    static_assert((pairs - 2) * 2 * nl + n2 <= 63 && (pairs - 1) * 2 * nl <= 63, "the loop's and the prologue's waits can be counted");
};

#define TPQ_PIN __builtin_amdgcn_sched_barrier(0)

// the value of lane ^ 32 beside the lane's own, in a fixed order: x = lower half's, y = upper half's
__device__ __forceinline__ void both_halves(uint32_t v, uint32_t &x, uint32_t &y)
{
    const auto r = __builtin_amdgcn_permlane32_swap(v, v, false, false);
    x = r[0];
    y = r[1];
}

// A workgroup's tile in LDS, one row of FT features per token: the features that stay bf16, [r, E) of its columns, to the
// outlier section; and the whole of it to the optional product.  Eight rows' reads at once: with one wave per SIMD
// nothing else hides the LDS latency.
template <int FT, int THREADS>
__device__ __forceinline__ void rows_selected(const GemmArgs &a, const uint8_t *tile, uint32_t tileF, int64_t tileT,
                                              int n_tok, uint32_t tid)
{
    constexpr uint32_t pitch = FT * 2 + 16;
    const int o0 = max(static_cast<int>(tileF) - a.r, 0), o1 = min(static_cast<int>(tileF) + FT, a.E) - a.r;
    if (o1 <= o0) return;
    const int n_live = a.T - tileT < n_tok ? static_cast<int>(a.T - tileT) : n_tok;
    const uint8_t *col0 = tile + 2 * (a.r - static_cast<int>(tileF));  // position 0 of the section (o0 on lies in the tile)
    uint8_t *out0 = a.outl + tileT * a.pitch_outl;
    const uint32_t po = static_cast<uint32_t>(a.pitch_outl);
    // positions that share their 32-bit word with another tile's
    for (uint32_t tt = tid; tt < static_cast<uint32_t>(n_live); tt += THREADS) {
        if (o0 & 1)
            *reinterpret_cast<uint16_t *>(out0 + tt * po + 2u * o0) = *reinterpret_cast<const uint16_t *>(col0 + tt * pitch + 2 * o0);
        if (o1 & 1)
            *reinterpret_cast<uint16_t *>(out0 + tt * po + 2u * (o1 - 1)) =
                *reinterpret_cast<const uint16_t *>(col0 + tt * pitch + 2 * (o1 - 1));
    }
    const int d0 = (o0 + 1) >> 1, nd = (o1 >> 1) - d0;  // whole words
    int lg = 3;                                         // lanes per token: 8 .. 64
    while (lg < 6 && (1 << lg) < nd) ++lg;
    const uint32_t step = static_cast<uint32_t>(THREADS) >> lg;
    for (int d = static_cast<int>(tid & ((1u << lg) - 1u)); d < nd; d += 1 << lg) {
        const uint8_t *src = col0 + 4 * (d0 + d);
        uint8_t *dst = out0 + 4u * static_cast<uint32_t>(d0 + d);
        for (uint32_t tt0 = tid >> lg; tt0 < static_cast<uint32_t>(n_live); tt0 += 8 * step) {
            uint32_t x[8];
#pragma unroll
            for (int u = 0; u < 8; ++u) {
                const uint8_t *q = src + min(tt0 + u * step, static_cast<uint32_t>(n_live) - 1u) * pitch;
                x[u] = *reinterpret_cast<const uint16_t *>(q) | (static_cast<uint32_t>(*reinterpret_cast<const uint16_t *>(q + 2)) << 16);
            }
#pragma unroll
            for (int u = 0; u < 8; ++u) {  // (rows past the last write its values again)
                const uint32_t tt = min(tt0 + u * step, static_cast<uint32_t>(n_live) - 1u);
                *reinterpret_cast<uint32_t *>(dst + tt * po) = x[u];
            }
        }
    }
}

template <int FT, int THREADS>
__device__ __forceinline__ void rows_product(const GemmArgs &a, const uint8_t *tile, uint32_t tileF, int64_t tileT,
                                             int n_tok, uint32_t tid)
{
    constexpr uint32_t pitch = FT * 2 + 16, LPT = FT / 8, STEP = THREADS / LPT;  // lanes per token, tokens at once
    const uint32_t c = tid % LPT, n0 = tileF + 8u * c;
    if (n0 >= static_cast<uint32_t>(a.E)) return;
    for (uint32_t tt = tid / LPT; tt < static_cast<uint32_t>(n_tok); tt += STEP)
        if (tileT + tt < a.T)
            *reinterpret_cast<u32x4 *>(a.Ymsg + (tileT + tt) * a.ldYm + n0) =
                *reinterpret_cast<const u32x4 *>(tile + tt * pitch + 16u * c);
}

// One block of 32 tokens of a wave's accumulators (128 features from F0 on) -> message.
template <int G>
__device__ __forceinline__ void tile_epilogue(const GemmArgs &a, float (&y)[4][16], bool ragged, uint32_t F0, int64_t t,
                                              bool t_ok, uint32_t h, float *xch, uint32_t wf, uint32_t tslot)
{
    constexpr float kBig = 3.3895314e38f;
    constexpr int NG = G >= 128 ? 1 : 128 / G, BPG = 4 / NG;  // groups of the wave, blocks of 32 features per group
    if (ragged) {
        // positions past the quantised features repeat their group's first one, so that the range stays its own
        // (a group without any is not stored; groups of 256: one that starts past the row's end takes the other wave's
        // range, which the exchange below leaves alone)
        int lim = a.r - static_cast<int>(F0 + 4u * h);
        asm volatile("" : "+v"(lim));  // (64 comparisons anew per block of tokens, not 64 kept masks)
#pragma unroll
        for (int g = 0; g < NG; ++g) {
            uint32_t first, other;
            both_halves(__float_as_uint(y[g * BPG][0]), first, other);
#pragma unroll
            for (int b = 0; b < BPG; ++b)
#pragma unroll
                for (int v = 0; v < 16; ++v) {
                    const int fb = g * BPG + b;
                    y[fb][v] = 32 * fb + 8 * (v >> 2) + (v & 3) < lim ? y[fb][v] : __uint_as_float(first);
                }
        }
    }
    float mn[NG], mx[NG];
#pragma unroll
    for (int g = 0; g < NG; ++g) {
        float lo = kBig, hi = -kBig;
#pragma unroll
        for (int b = 0; b < BPG; ++b)
#pragma unroll
            for (int v = 0; v < 16; ++v) {
                const int fb = g * BPG + b;
                lo = fminf(lo, y[fb][v]);
                hi = fmaxf(hi, y[fb][v]);
            }
        uint32_t p, q;
        both_halves(__float_as_uint(lo), p, q);
        mn[g] = fminf(__uint_as_float(p), __uint_as_float(q));
        both_halves(__float_as_uint(hi), p, q);
        mx[g] = fmaxf(__uint_as_float(p), __uint_as_float(q));
    }
    if (G == 256) {  // the two waves that share a group meet in LDS
        float2 *x = reinterpret_cast<float2 *>(xch);
        const bool none = ragged && F0 >= static_cast<uint32_t>(a.r);
        if (h == 0) x[2u * tslot + wf] = none ? make_float2(kBig, -kBig) : make_float2(mn[0], mx[0]);
        __syncthreads();
        const float2 o = x[2u * tslot + (wf ^ 1u)];
        mn[0] = none ? o.x : fminf(mn[0], o.x);
        mx[0] = none ? o.y : fmaxf(mx[0], o.y);
    }
    float inv[NG];
#pragma unroll
    for (int g = 0; g < NG; ++g) {
        mn[g] = mn[g] + 0.0f;
        const float s32 = div_by_15(mx[g] - mn[g]);
        const uint32_t sb = pack_bf16x2(s32, s32) & 0xFFFFu;
        const float s = bf16_bits_to_f32(sb);
        const bool constant = s < 1e-30f;
        inv[g] = constant ? 0.0f : reciprocal_of_scale(s);
        const uint32_t gi = F0 / static_cast<uint32_t>(G) + g;
        if (t_ok && (G < 256 || wf == 0) && (!ragged || gi < static_cast<uint32_t>(a.ng)))
            reinterpret_cast<uint16_t *>((h ? a.zero : a.scale) + t * a.pitch_meta)[gi] =
                static_cast<uint16_t>(h ? __float_as_uint(mn[g]) >> 16 : (constant ? 0u : sb));
    }
    uint8_t *crow = a.codes + t * a.pitch_codes;
#pragma unroll
    for (int fp = 0; fp < 4; fp += 2) {
        uint32_t A[2][2];
#pragma unroll
        for (int b = 0; b < 2; ++b) {
            const int fb = fp + b, g = fb / BPG;
            uint32_t q[4];
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                float p[4];
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    const float df = y[fb][4 * j + e] - mn[g];
                    p[e] = df * inv[g];
                }
                uint32_t w = __builtin_amdgcn_cvt_pk_u8_f32(p[1], 0u, 0u);
                w = __builtin_amdgcn_cvt_pk_u8_f32(p[0], 1u, w);
                w = __builtin_amdgcn_cvt_pk_u8_f32(p[3], 2u, w);
                w = __builtin_amdgcn_cvt_pk_u8_f32(p[2], 3u, w);
                q[j] = (w << 12) | w;
            }
            A[b][0] = __builtin_amdgcn_perm(q[1], q[0], 0x07050301u);
            A[b][1] = __builtin_amdgcn_perm(q[3], q[2], 0x07050301u);
        }
        // lower lanes take block fp, upper lanes block fp + 1
        u32x4 o;
        {
            const auto r0 = __builtin_amdgcn_permlane32_swap(A[0][0], A[1][0], false, false);
            const auto r1 = __builtin_amdgcn_permlane32_swap(A[0][1], A[1][1], false, false);
            const uint32_t x0 = r0[0], y0 = r0[1], x1 = r1[0], y1 = r1[1];
            o.x = __builtin_amdgcn_perm(y0, x0, 0x05040100u);
            o.y = __builtin_amdgcn_perm(y0, x0, 0x07060302u);
            o.z = __builtin_amdgcn_perm(y1, x1, 0x05040100u);
            o.w = __builtin_amdgcn_perm(y1, x1, 0x07060302u);
        }
        const uint32_t ch = F0 / 8u + 4u * (fp + h);
        if (!ragged) {
            if (t_ok) *reinterpret_cast<u32x4 *>(crow + 4u * ch) = o;
        } else if (t_ok) {
            const uint32_t w4[4] = {o.x, o.y, o.z, o.w};
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const int n_valid = a.r - 8 * static_cast<int>(ch + e);
                if (n_valid > 0)
                    *reinterpret_cast<uint32_t *>(crow + 4u * (ch + e)) = n_valid < 8 ? w4[e] & ((1u << (4 * n_valid)) - 1u) : w4[e];
            }
        }
    }
}

template <int G, int FW, int TW, int NTB>
__global__ __launch_bounds__(64 * FW * TW, 1) void k_gemm_tile(GemmArgs a, uint32_t tiles_t)
{
    typedef TileShape<FW, TW, NTB> S;
    static_assert(G <= 128 * FW, "a group lies inside the tile");
    constexpr int NL = S::nl, NF = 4 + NTB;  // loads per stage; fragments per k-step: 4 of the weights, NTB of the tokens
    extern __shared__ u32x4 smem_gemm[];
    uint8_t *lds = reinterpret_cast<uint8_t *>(smem_gemm);
    const uint32_t tid = threadIdx.x, ln = tid & 63u;
    const uint32_t wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const uint32_t wf = wave % FW, wt = wave / FW;
    const uint32_t id = xcd_contiguous_index(blockIdx.x, gridDim.x);
    const uint32_t tf = id / tiles_t, tt = id - tf * tiles_t;
    const uint32_t tileF = tf * static_cast<uint32_t>(S::ft);
    const int64_t tileT = static_cast<int64_t>(tt) * S::tt;
    if (tileF >= static_cast<uint32_t>(a.E)) return;
    const int K = a.K;

    // a wave's load instruction fills 16 rows of 64 bytes
    const uint32_t prow = tid / 4, slot = tid % 4;
    const int pk = static_cast<int>(slot ^ ((prow >> 1) & 3u)) * 8;
    const int pkc = min(pk, K - 8);
    uint32_t voff[NL];
#pragma unroll
    for (int i = 0; i < S::nla; ++i)
        voff[i] = (min(tileF + prow + 16 * S::waves * i, static_cast<uint32_t>(a.E) - 1u) * static_cast<uint32_t>(K) + pkc) * 2u;
#pragma unroll
    for (int i = 0; i < NL - S::nla; ++i) {
        const int64_t t = min(tileT + prow + 16 * S::waves * i, a.T - 1);
        voff[S::nla + i] = static_cast<uint32_t>((t * a.ldX + pkc) * 2);
    }
    const uint64_t pa = reinterpret_cast<uint64_t>(a.Wp), pb = reinterpret_cast<uint64_t>(a.X);
    const u32x4 ra = {static_cast<uint32_t>(pa), static_cast<uint32_t>(pa >> 32),
                      static_cast<uint32_t>(static_cast<int64_t>(a.E) * K * 2), 0x00020000u};
    const u32x4 rb = {static_cast<uint32_t>(pb), static_cast<uint32_t>(pb >> 32),
                      static_cast<uint32_t>(((a.T - 1) * a.ldX + K) * 2), 0x00020000u};
    const uint32_t lds0 = static_cast<uint32_t>(reinterpret_cast<uintptr_t>((__attribute__((address_space(3))) uint8_t *)lds)) + wave * 1024u;
    const int nkt = (K + kTileBK - 1) / kTileBK, np = (nkt + 1) / 2;
    const int k_last = max(K - kTileBK, 0);
    auto k_bytes = [&](int kt) { return static_cast<uint32_t>(2 * min(kt * kTileBK, k_last)); };
    // (m0 is reserved, so it cannot be named as changed: the compiler keeps nothing in it, and no other
    // instruction of this kernel needs it)
    auto dma = [&](int i, uint32_t kb2, uint32_t buf) {
        const uint32_t m = lds0 + buf + 1024u * S::waves * i;
        if (i < S::nla)
            asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tbuffer_load_dwordx4 %1, %2, %3 offen lds" ::"s"(m), "v"(voff[i]), "s"(ra), "s"(kb2) : "memory");
        else
            asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tbuffer_load_dwordx4 %1, %2, %3 offen lds" ::"s"(m), "v"(voff[i]), "s"(rb), "s"(kb2) : "memory");
    };

    f32x16 acc[4][NTB];
#pragma unroll
    for (int fb = 0; fb < 4; ++fb)
#pragma unroll
        for (int tb = 0; tb < NTB; ++tb)
#pragma unroll
            for (int v = 0; v < 16; ++v) acc[fb][tb][v] = 0.0f;

    // fragment i: 0..3 the weights' blocks, 4.. the tokens'
    const uint32_t row = ln & 31u, h = ln >> 5;
    const uint32_t fk0 = ((0u + h) ^ ((row >> 1) & 3u)) * 16u, fk1 = ((2u + h) ^ ((row >> 1) & 3u)) * 16u;
    const uint32_t fa = (128u * wf + row) * 64u, fbt = (static_cast<uint32_t>(S::ft) + 32u * NTB * wt + row) * 64u;
    u32x4 fr[2][NF];
    auto fetch = [&](int i, int ks, uint32_t buf) {
        const uint32_t at = buf + (i < 4 ? fa + 2048u * i : fbt + 2048u * (i - 4)) + (ks ? fk1 : fk0);
        fr[ks][i] = *reinterpret_cast<const u32x4 *>(lds + at);
    };
    auto mfma = [&](int ks, int j) {
        const int fb = j / NTB, tb = j % NTB;
        acc[fb][tb] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8_t, fr[ks][fb]),
                                                              __builtin_bit_cast(bf16x8_t, fr[ks][4 + tb]), acc[fb][tb], 0, 0, 0);
    };
    auto next_buf = [&](uint32_t b) { return b + S::stage == S::lds ? 0u : b + S::stage; };
    auto prev_buf = [&](uint32_t b) { return b == 0u ? static_cast<uint32_t>(S::lds - S::stage) : b - S::stage; };
    // load j of a pair of stages: piece j / 2 of stage j % 2 (the two halves of a row's cache line
    // one after the other)
    auto dma_pair = [&](int j, uint32_t k0, uint32_t k1, uint32_t b0, uint32_t b1) {
        dma(j >> 1, (j & 1) ? k1 : k0, (j & 1) ? b1 : b0);
    };
    // One phase: the 4 NTB products of k-step KS, and between them the fetch of the other k-step's
    // fragments and loads D0 .. D1 - 1 of the pair that is on its way in -- the fetches first, one memory
    // instruction behind each product where there are as many.
#define TPQ_PHASE(KS, FK, FBUF, D0, D1)                                                             \
    _Pragma("unroll") for (int j = 0; j < SLOTS; ++j)                                               \
    {                                                                                               \
        if (j < 4 * NTB) mfma(KS, j);                                                               \
        if (j < NF) fetch(j, FK, FBUF);                                                             \
        const int q = D1 - 1 - (SLOTS - 1 - j);                                                     \
        if (q >= D0 && q < D1) dma_pair(q, kb0, kb1, d0, d1);                                       \
        TPQ_PIN;                                                                                    \
    }
    constexpr int SLOTS = 4 * NTB > NF ? (4 * NTB > S::n1 ? 4 * NTB : S::n1) : (NF > S::n1 ? NF : S::n1);
    constexpr int N1 = S::n1, N2 = S::n2;
    // prologue
    if (np >= S::pairs) {
#pragma unroll
        for (int p = 0; p < S::pairs; ++p)
#pragma unroll
            for (int j = 0; j < 2 * NL; ++j)
                dma_pair(j, k_bytes(2 * p), k_bytes(2 * p + 1), (2 * p) * S::stage, (2 * p + 1) * S::stage);
        asm volatile("s_waitcnt vmcnt(%0)" ::"n"((S::pairs - 1) * 2 * NL) : "memory");
    } else {  // a short K has fewer stages than the ring: no loads for the others (T = 13, E = 5120, K = 128 6.3 -> 5.8 us)
#pragma nounroll
        for (int p = 0; p < np; ++p)
#pragma unroll
            for (int j = 0; j < 2 * NL; ++j)
                dma_pair(j, k_bytes(2 * p), k_bytes(2 * p + 1), (2 * p) * S::stage, (2 * p + 1) * S::stage);
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    }
    __builtin_amdgcn_s_barrier();
    uint32_t b0 = 0;
#pragma unroll
    for (int i = 0; i < NF; ++i) fetch(i, 0, b0);
    for (int p = 0; p < np - 1; ++p) {
        const uint32_t b1 = next_buf(b0), b2 = next_buf(b1);
        const uint32_t d0 = prev_buf(b0), d1 = b0;
        const uint32_t kb0 = k_bytes(2 * (p + S::pairs)), kb1 = k_bytes(2 * (p + S::pairs) + 1);
        TPQ_PIN;
        TPQ_PHASE(0, 1, b0, 0, 0)
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
        __builtin_amdgcn_s_barrier();
        TPQ_PIN;
        TPQ_PHASE(1, 0, b1, 0, N1)
        TPQ_PHASE(0, 1, b1, N1, N2)
        asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)" ::"n"((S::pairs - 2) * 2 * NL + N2) : "memory");
        __builtin_amdgcn_s_barrier();
        TPQ_PIN;
        TPQ_PHASE(1, 0, b2, N2, 2 * NL)
        b0 = b2;
    }
    // the last pair: k past the row's end counts as zero
    {
        const uint32_t b1 = next_buf(b0);
#pragma unroll
        for (int q = 0; q < 2; ++q) {
            const int kt = 2 * np - 2 + q, kb = static_cast<int>(k_bytes(kt)) / 2;
            const int p0 = kb + 8 * static_cast<int>(h), p1 = p0 + 16;
            const bool ok0 = p0 >= kt * kTileBK && p0 < K, ok1 = p1 >= kt * kTileBK && p1 < K;
            if (q == 1) {
#pragma unroll
                for (int i = 0; i < NF; ++i) fetch(i, 0, b1);
            }
#pragma unroll
            for (int i = 0; i < NF; ++i) fetch(i, 1, q ? b1 : b0);
#pragma unroll
            for (int i = 4; i < NF; ++i) {
                fr[0][i] = ok0 ? fr[0][i] : u32x4{0u, 0u, 0u, 0u};
                fr[1][i] = ok1 ? fr[1][i] : u32x4{0u, 0u, 0u, 0u};
            }
#pragma unroll
            for (int j = 0; j < 4 * NTB; ++j) mfma(0, j);
#pragma unroll
            for (int j = 0; j < 4 * NTB; ++j) mfma(1, j);
        }
    }
#undef TPQ_PHASE
    asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)" ::: "memory");
    __builtin_amdgcn_s_barrier();

    const uint32_t F0 = tileF + 128u * wf;
    const bool ragged = tileF + static_cast<uint32_t>(S::ft) > static_cast<uint32_t>(a.r);
    if (a.Ymsg || ragged) {
#pragma unroll
        for (int tb = 0; tb < NTB; ++tb) {
            uint8_t *orow = lds + (32u * (NTB * wt + tb) + row) * (S::ft * 2 + 16) + (128u * wf + 4u * h) * 2u;
#pragma unroll
            for (int fb = 0; fb < 4; ++fb)
#pragma unroll
                for (int j = 0; j < 4; ++j)
                    *reinterpret_cast<uint2 *>(orow + (32 * fb + 8 * j) * 2) =
                        make_uint2(pack_bf16x2(acc[fb][tb][4 * j], acc[fb][tb][4 * j + 1]),
                                   pack_bf16x2(acc[fb][tb][4 * j + 2], acc[fb][tb][4 * j + 3]));
        }
        __syncthreads();
        rows_selected<S::ft, S::threads>(a, lds, tileF, tileT, S::tt, tid);
        if (a.Ymsg) rows_product<S::ft, S::threads>(a, lds, tileF, tileT, S::tt, tid);
        __syncthreads();
    }
    // (one copy of the epilogue's code for all blocks of tokens: unrolled it is no faster, and NTB times as long)
#pragma nounroll
    for (int tb = 0; tb < NTB; ++tb) {
        float y[4][16];
#define TPQ_TAKE(TB)                                                                        \
    if (TB < NTB && tb == TB) {                                                             \
        _Pragma("unroll") for (int fb = 0; fb < 4; ++fb)                                    \
            _Pragma("unroll") for (int v = 0; v < 16; ++v) y[fb][v] = acc[fb][TB < NTB ? TB : 0][v]; \
    }
        TPQ_TAKE(0)
        else TPQ_TAKE(1)
        else TPQ_TAKE(2)
        else TPQ_TAKE(3)
#undef TPQ_TAKE
#pragma unroll
        for (int fb = 0; fb < 4; ++fb)
#pragma unroll
            for (int v = 0; v < 16; ++v) y[fb][v] = round_via_bf16(y[fb][v]);
        const uint32_t tslot = 32u * (NTB * wt + tb) + row;
        const int64_t t = tileT + tslot;
        const bool t_ok = t < a.T;
        tile_epilogue<G>(a, y, ragged, F0, t_ok ? t : 0, t_ok, h, reinterpret_cast<float *>(lds), wf, tslot);
    }
}

// Few tokens: a workgroup has the G features of one group and 16 NTB tokens, and its 8 waves share K: wave w takes
// the stages of 32 k that are w modulo their number, through a ring in LDS of its own, so that nothing waits for a barrier and
// all of a short K is on its way at once.  The partial sums meet in LDS, where all threads share the epilogue.  Bound by what a
// compute unit can have outstanding to memory; E / G of them hold a group each.  In the tiles below one wave does the
// products and the epilogue of 16 tokens by itself, at E / 128 units whatever G, and a stage costs it 0.19 us from barrier to barrier.
// (Fragments loaded straight into registers, 16 rows by 64 bytes an instruction with neighbouring lanes in different rows:
// 41 bytes/ns a compute unit, where four lanes to a row, as here, reach twice that.)
// Stages taken in pairs by a wave, so that it has both halves of a line, are 6 to 14 % slower.
// E = 5120, G = 128, T = 16, weights in the L2s (in the memory-side cache): K = 640 8.8 -> 4.2 us (9.0 -> 6.0), K = 1728 15.3 -> 6.5 (15.1 -> 10.8); T = 64,
// K = 1728 15.6 -> 7.2 (16.0 -> 9.3): more tokens are more workgroups, until the chip is full (launch_tiles()).
template <int G, int NTB>
struct FewShape {
    static constexpr int waves = 8, threads = 64 * waves;
    static constexpr int FW = G == 256 ? 2 : 1, KW = waves / FW; // waves across features and k
    static constexpr int FB = G / (16 * FW);                     // blocks of 16 features of a wave
    static constexpr int nl = FB + NTB, stage = nl * 1024;       // loads and LDS bytes of a stage: 16 rows of 64 bytes each
    static constexpr int fit = 163840 / waves / stage, ring = fit < 4 ? fit : 4;
    static constexpr int pitch = G + 4;                          // floats of a token's row of partial sums
    static constexpr int sums = KW * 16 * pitch * 4, lds = sums > waves * ring * stage ? sums : waves * ring * stage;
    static_assert(ring >= 2 && lds <= 163840 && (ring - 1) * nl <= 63, "the ring fits, its waits can be counted");
};

template <int G, int NTB>
__global__ __launch_bounds__((FewShape<G, NTB>::threads)) void k_gemm_few(GemmArgs a, uint32_t tiles_t)
{
    typedef FewShape<G, NTB> S;
    constexpr int FB = S::FB, NL = S::nl;
    extern __shared__ u32x4 smem_gemm[];
    float *const part = reinterpret_cast<float *>(smem_gemm);  // [k share][token of 16][pitch], once the ring is done with
    const uint32_t tid = threadIdx.x, ln = tid & 63u;
    const uint32_t wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const uint32_t wf = wave % S::FW, wk = wave / S::FW;
    // (a group's workgroups one after the other on one XCD: its weights come from memory once)
    const uint32_t id = xcd_contiguous_index(blockIdx.x, gridDim.x);
    const uint32_t gi = id / tiles_t, F0 = gi * static_cast<uint32_t>(G);
    if (F0 >= static_cast<uint32_t>(a.E)) return;  // (the grid is rounded up to a multiple of 8)
    const int T0 = 16 * NTB * static_cast<int>(id - gi * tiles_t);
    const int K = a.K, T = static_cast<int>(a.T);

    // a load instruction fills 16 rows of 64 bytes, four lanes a row; rows past the last are the last again, and a stage that
    // would leave the row starts earlier (what it has twice is multiplied by zero): every load is in bounds and unconditional
    const uint32_t prow = ln / 4u;
    const int pk = static_cast<int>((ln % 4u) ^ ((prow >> 1) & 3u)) * 8, pkc = min(pk, K - 8);
    uint32_t voff[NL];
#pragma unroll
    for (int f = 0; f < FB; ++f)
        voff[f] = 2u * (min(F0 + (wf * FB + f) * 16u + prow, static_cast<uint32_t>(a.E) - 1u) * static_cast<uint32_t>(K) + pkc);
#pragma unroll
    for (int t = 0; t < NTB; ++t)
        voff[FB + t] = 2u * (static_cast<uint32_t>(min(T0 + 16 * t + static_cast<int>(prow), T - 1)) * static_cast<uint32_t>(a.ldX) + pkc);
    const uint64_t pa = reinterpret_cast<uint64_t>(a.Wp), pb = reinterpret_cast<uint64_t>(a.X);
    const u32x4 ra = {static_cast<uint32_t>(pa), static_cast<uint32_t>(pa >> 32),
                      static_cast<uint32_t>(static_cast<int64_t>(a.E) * K * 2), 0x00020000u};
    const u32x4 rb = {static_cast<uint32_t>(pb), static_cast<uint32_t>(pb >> 32),
                      static_cast<uint32_t>(((a.T - 1) * a.ldX + K) * 2), 0x00020000u};
    uint8_t *const ring = reinterpret_cast<uint8_t *>(smem_gemm) + wave * (S::ring * S::stage);
    const uint32_t lds0 = static_cast<uint32_t>(reinterpret_cast<uintptr_t>((__attribute__((address_space(3))) uint8_t *)ring));
    const int k_last = max(K - kTileBK, 0), all = (K + kTileBK - 1) / kTileBK;
    const int mine = (all - static_cast<int>(wk) + S::KW - 1) / S::KW;  // this wave's stages (at most 0 where K is short)
    auto stage_k = [&](int i) { return kTileBK * (static_cast<int>(wk) + i * S::KW); };
    auto dma = [&](int i, uint32_t buf) __attribute__((always_inline)) {
        const uint32_t kb2 = static_cast<uint32_t>(2 * min(stage_k(i), k_last));
#pragma unroll
        for (int l = 0; l < NL; ++l) {
            const uint32_t m = lds0 + buf * S::stage + 1024u * l;
            if (l < FB)
                asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tbuffer_load_dwordx4 %1, %2, %3 offen lds" ::"s"(m), "v"(voff[l]), "s"(ra), "s"(kb2) : "memory");
            else
                asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tbuffer_load_dwordx4 %1, %2, %3 offen lds" ::"s"(m), "v"(voff[l]), "s"(rb), "s"(kb2) : "memory");
        }
    };

    typedef float f32x4_t __attribute__((ext_vector_type(4)));
    f32x4_t acc[FB][NTB];
#pragma unroll
    for (int f = 0; f < FB; ++f)
#pragma unroll
        for (int t = 0; t < NTB; ++t) acc[f][t] = f32x4_t{0.f, 0.f, 0.f, 0.f};
    const uint32_t row = ln & 15u, kq = ln >> 4;
    const uint32_t at = row * 64u + ((kq ^ ((row >> 1) & 3u)) * 16u);
#pragma unroll
    for (int i = 0; i < S::ring; ++i)
        if (i < mine) dma(i, i);
    uint32_t buf = 0;
    for (int i = 0; i < mine; ++i) {
        // the stages behind this one are on their way: as many as the ring holds, fewer at the end
        const int behind = mine - 1 - i;
        if (behind >= S::ring - 1)
            asm volatile("s_waitcnt vmcnt(%0)" ::"n"((S::ring - 1) * NL) : "memory");
        else if (S::ring > 3 && behind == 2)
            asm volatile("s_waitcnt vmcnt(%0)" ::"n"(2 * NL) : "memory");
        else if (S::ring > 2 && behind == 1)
            asm volatile("s_waitcnt vmcnt(%0)" ::"n"(NL) : "memory");
        else
            asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
        const uint8_t *st = ring + buf * S::stage + at;
        u32x4 w[FB], x[NTB];
#pragma unroll
        for (int t = 0; t < NTB; ++t) x[t] = *reinterpret_cast<const u32x4 *>(st + 1024 * (FB + t));
#pragma unroll
        for (int f = 0; f < FB; ++f) w[f] = *reinterpret_cast<const u32x4 *>(st + 1024 * f);
        if (i + S::ring < mine) {  // the buffer is free once its fragments are in registers
            asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
            dma(i + S::ring, buf);
        }
        const int k = min(stage_k(i), k_last) + 8 * static_cast<int>(kq);
        const bool in = k >= stage_k(i) && k < K;
#pragma unroll
        for (int t = 0; t < NTB; ++t) x[t] = in ? x[t] : u32x4{0u, 0u, 0u, 0u};
#pragma unroll
        for (int f = 0; f < FB; ++f)
#pragma unroll
            for (int t = 0; t < NTB; ++t)
                acc[f][t] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8_t, w[f]),
                                                                    __builtin_bit_cast(bf16x8_t, x[t]), acc[f][t], 0, 0, 0);
        buf = buf + 1u == S::ring ? 0u : buf + 1u;
    }
    __syncthreads();  // (every wave has taken its last fragments)

    // ---- 16 tokens at a time: the shares meet, then G / 4 lanes have a token's group, 4 features each
    constexpr uint32_t LPT = G / 4;  // lanes of a token
    const int n_tb = (T - T0 + 15) / 16;
    const bool whole = F0 + G <= static_cast<uint32_t>(a.r);
#pragma unroll
    for (int t0 = 0; t0 < NTB; ++t0) {
        if (t0 >= n_tb) break;
        if (t0) __syncthreads();
#pragma unroll
        for (int f = 0; f < FB; ++f)
            *reinterpret_cast<f32x4_t *>(part + (wk * 16u + row) * S::pitch + (wf * FB + f) * 16u + 4u * kq) = acc[f][t0];
        __syncthreads();
#pragma unroll
        for (uint32_t i0 = 0; i0 < 16u * LPT; i0 += S::threads) {
            const uint32_t i = i0 + tid;
            if (16u * LPT < S::threads && i >= 16u * LPT) break;  // (whole waves)
            const uint32_t tok = i / LPT, q = i % LPT, n0 = F0 + 4u * q;
            f32x4_t p[S::KW];
#pragma unroll
            for (int w = 0; w < S::KW; ++w) p[w] = *reinterpret_cast<const f32x4_t *>(part + (w * 16u + tok) * S::pitch + 4u * q);
            float y[4];
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                float v = p[0][e];
#pragma unroll
                for (int w = 1; w < S::KW; ++w) v += p[w][e];
                y[e] = round_via_bf16(v);
            }
            const int64_t t = T0 + 16 * t0 + static_cast<int>(tok);
            const bool t_ok = t < a.T;
            if (a.Ymsg && t_ok && n0 < static_cast<uint32_t>(a.E))
                *reinterpret_cast<uint2 *>(a.Ymsg + t * a.ldYm + n0) = make_uint2(
                    (__float_as_uint(y[0]) >> 16) | __float_as_uint(y[1]), (__float_as_uint(y[2]) >> 16) | __float_as_uint(y[3]));
            const int live = whole ? 4 : a.r - static_cast<int>(n0);  // quantised features from n0 on
            if (!whole && t_ok) {
                uint16_t *out = reinterpret_cast<uint16_t *>(a.outl + t * a.pitch_outl);
#pragma unroll
                for (int e = 0; e < 4; ++e)
                    if (e >= live && n0 + e < static_cast<uint32_t>(a.E)) out[n0 + e - a.r] = static_cast<uint16_t>(__float_as_uint(y[e]) >> 16);
            }
            if (F0 >= static_cast<uint32_t>(a.r)) continue;  // (no quantised feature in the workgroup)
            constexpr float kBig = 3.3895314e38f;
            float mn = kBig, mx = -kBig;
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                mn = fminf(mn, e < live ? y[e] : kBig);
                mx = fmaxf(mx, e < live ? y[e] : -kBig);
            }
            group_minmax<LPT == 64 ? 32 : static_cast<int>(LPT)>(mn, mx);
            if (LPT == 64) {
                mn = fminf(mn, __shfl_xor(mn, 32, 64));
                mx = fmaxf(mx, __shfl_xor(mx, 32, 64));
            }
            mn = mn + 0.0f;
            const float s32 = div_by_15(mx - mn);
            const uint32_t sb = pack_bf16x2(s32, s32) & 0xFFFFu;
            const float sc = bf16_bits_to_f32(sb);
            const bool constant = sc < 1e-30f;
            const float inv = constant ? 0.0f : reciprocal_of_scale(sc);
            if (q == 0 && t_ok) {
                reinterpret_cast<uint16_t *>(a.scale + t * a.pitch_meta)[gi] = static_cast<uint16_t>(constant ? 0u : sb);
                reinterpret_cast<uint16_t *>(a.zero + t * a.pitch_meta)[gi] = static_cast<uint16_t>(__float_as_uint(mn) >> 16);
            }
            float pr[4];
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const float df = (e < live ? y[e] : mn) - mn;
                pr[e] = df * inv;
            }
            uint32_t w = __builtin_amdgcn_cvt_pk_u8_f32(pr[1], 0u, 0u);
            w = __builtin_amdgcn_cvt_pk_u8_f32(pr[0], 1u, w);
            w = __builtin_amdgcn_cvt_pk_u8_f32(pr[3], 2u, w);
            w = __builtin_amdgcn_cvt_pk_u8_f32(pr[2], 3u, w);
            w = (w << 12) | w;
            w = __builtin_amdgcn_perm(w, w, 0x0C0C0301u);  // the four codes in the low half
            const uint32_t other = __builtin_amdgcn_update_dpp(0u, w, 0xB1, 0xF, 0xF, true);
            if (!(q & 1u) && live > 0 && t_ok)
                *reinterpret_cast<uint32_t *>(a.codes + t * a.pitch_codes + n0 / 2u) = w | (other << 16);
        }
    }
}

// the kernel may use more LDS than the default limit: allowed once per device
template <typename Kernel>
static hipError_t allow_lds(Kernel kernel, int bytes, std::atomic<uint64_t> &allowed)
{
    int dev = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return e;
    const uint64_t bit = dev < 64 ? 1ull << dev : 0ull;
    if (!(allowed.load(std::memory_order_relaxed) & bit)) {
        e = hipFuncSetAttribute(reinterpret_cast<const void *>(kernel), hipFuncAttributeMaxDynamicSharedMemorySize, bytes);
        if (e != hipSuccess) return e;
        allowed.fetch_or(bit, std::memory_order_relaxed);
    }
    return hipSuccess;
}

template <int G, int NTB>
static int launch_few_g(const GemmArgs &a, hipStream_t s)
{
    typedef FewShape<G, NTB> S;
    const auto kernel = &k_gemm_few<G, NTB>;
    static std::atomic<uint64_t> allowed;
    const hipError_t e = S::lds > 65536 ? allow_lds(kernel, S::lds, allowed) : hipSuccess;
    if (e != hipSuccess) return hip_result(e);
    const int64_t tiles_t = (a.T + 16 * NTB - 1) / (16 * NTB), blocks = ((a.E + G - 1) / G * tiles_t + 7) / 8 * 8;
    if (blocks * S::threads >= (1ll << 32)) return TPQ_ERR_SHAPE;
    launch_kernel(kernel, dim3(static_cast<unsigned>(blocks)), dim3(S::threads), static_cast<size_t>(S::lds), s, a,
                  static_cast<uint32_t>(tiles_t));
    return hip_result(hipGetLastError());
}

template <int G, int FW, int TW, int NTB>
static int launch_tile_g(const GemmArgs &a, hipStream_t s)
{
    typedef TileShape<FW, TW, NTB> S;
    const auto kernel = &k_gemm_tile<G, FW, TW, NTB>;
    const int64_t tiles_f = (a.E + S::ft - 1) / S::ft, tiles_t = (a.T + S::tt - 1) / S::tt;
    const int64_t blocks = (tiles_f * tiles_t + 7) / 8 * 8;  // (a multiple of 8 for the XCD order)
    if (blocks * S::threads >= (1ll << 32)) return TPQ_ERR_SHAPE;
    static std::atomic<uint64_t> allowed;
    const hipError_t e = allow_lds(kernel, S::lds, allowed);
    if (e != hipSuccess) return hip_result(e);
    launch_kernel(kernel, dim3(static_cast<unsigned>(blocks)), dim3(S::threads), static_cast<size_t>(S::lds), s, a,
                  static_cast<uint32_t>(tiles_t));
    return hip_result(hipGetLastError());
}

template <int FW, int TW, int NTB>
static int launch_tile(const GemmArgs &a, hipStream_t s)
{
    switch (a.G) {
    case 32: return launch_tile_g<32, FW, TW, NTB>(a, s);
    case 64: return launch_tile_g<64, FW, TW, NTB>(a, s);
    case 128: return launch_tile_g<128, FW, TW, NTB>(a, s);
    case 256:
        if constexpr (FW == 2) return launch_tile_g<256, FW, TW, NTB>(a, s);
        return TPQ_ERR_UNSUPPORTED;
    default: return TPQ_ERR_UNSUPPORTED;
    }
}

// The tile: the one whose rounds over the chip cost least.  A compute unit holds one workgroup, so a launch
// takes ceil(tiles / compute units) rounds; a round of a tile costs what the table says, measured back to back at
// K = 1728 (and in the same ratios at K = 640; at K = 128 the ends are most of it, and 4096 x 2048 would be 6 % faster in
// smaller tiles), E = 5120, in us of a launch of one round: 128 features x 64 tokens
// 16.3, 128 x 128 17.5, 256 x 64 17.7 (the loads' time: more tokens are free), 256 x 128 24, 256 x 192 31, 256 x 256
// 39 (the products' time, and 8 to 10 us of ends whatever the tile).  Where a smaller tile needs no further round it
// wins: 512 tokens 18.7 us at 128 x 128 against 23.7 at 256 x 128; 1024 tokens 25.6 at 256 x 128 against 33.9
// (two rounds) and 31.7 (256 x 192); 2048 tokens 37.5 at 256 x 192 against 49 and 54 (two and three rounds)
// and 44 (256 x 256).
//
// Few tokens: k_gemm_few where its estimate is 5 % below the tile's.  Both estimates are fits to 3400 launches (E 128 .. 16384, K 16 .. 14400, 1 to 1500
// tokens) whose weights came from the memory-side cache, as a layer's do that ran a few layers ago: ns of a launch = ends + rounds * (round + slope * K
// / 1000), the slope larger where an XCD's workgroups read more than its L2 holds (far) and smaller where several have the same weights
// (shared); k_gemm_few besides not under 3.95 us, nor under what all units get from their L2s together.  Half of the launches are within 2 to 14 % of
// their fit, nine of ten within 30 %.  Of 1000 launches that the fits have not seen, the form taken is more than 5 % slower than the tile for 5 to 8 (32 before,
// by estimates from weights in L2), and 0.6 % off the fastest form in the mean (1.2 % before); for 24 (42) with weights from memory, where a unit's
// one group is bound by the lines it can have outstanding in either form and the tile has a line's halves together.
// Tile / 16 / 32 tokens a workgroup, us, weights in the memory-side cache (and in the L2s): E = 5120, T = 16, K = 640 9.0 / 6.0 / 6.1 (8.8 / 4.2 / 4.7) with G = 128,
// 10.0 / 9.5 / 9.5 (9.4 / 6.1 / 6.5) with 256; K = 1728 15.1 / 10.8 / 10.8 (15.3 / 6.5 / 7.1), and 16.8 / 18.8 / 19.2 (16.6 / 10.1 / 11.4) with 256; T = 64, K = 1728 16.0 / 9.3 / 11.8
// (15.6 / 7.2 / 8.3); E = 8192, K = 3584, T = 16 25.8 / 20.0 / 20.4, and 30.2 / 37.6 / 38.2 with 256.
static int launch_tiles(const GemmArgs &a, hipStream_t s)
{
    struct Tile {
        int ft, tt, cost;
        int ends, round, slope, far;  // the estimate; slope 0: none, k_gemm_few is never faster
        int (*launch)(const GemmArgs &, hipStream_t);
    };
    static const Tile tiles[] = {
        {128, 64, 16, 2960, 2420, 6030, 150, launch_tile<1, 2, 1>},    {128, 128, 17, 5000, 1470, 8140, 0, launch_tile<1, 4, 1>},
        {256, 64, 18, 1370, 4240, 8410, 2050, launch_tile<2, 2, 1>},   {256, 128, 24, 1990, 7440, 11280, 1770, launch_tile<2, 2, 2>},
        {256, 192, 31, 6500, 9580, 11990, 5380, launch_tile<2, 2, 3>}, {256, 256, 39, 0, 0, 0, 0, launch_tile<2, 2, 4>},
    };
    struct Few {
        int G, tt;
        int ends, round, slope, far, shared, chip, mb;  // shared: per mille of the slope saved where a group's workgroups are many; all units together: chip ns, and mb ns a MB
        int (*launch)(const GemmArgs &, hipStream_t);
    };
    static const Few fews[] = {
        {32, 16, 1240, 1220, 1220, 470, 41, 3040, 72, launch_few_g<32, 1>},     {32, 32, 800, 1930, 1470, 640, 0, 2880, 70, launch_few_g<32, 2>},
        {32, 64, 0, 3180, 2000, 940, 0, 4030, 50, launch_few_g<32, 4>},         {64, 16, 1030, 1360, 2370, 660, 101, 3450, 44, launch_few_g<64, 1>},
        {64, 32, 170, 2470, 2610, 640, 0, 3690, 57, launch_few_g<64, 2>},       {64, 64, 0, 3630, 2850, 1260, 0, 4150, 73, launch_few_g<64, 4>},
        {128, 16, 700, 1820, 4550, 1220, 137, 2900, 79, launch_few_g<128, 1>},  {128, 32, 0, 3040, 4800, 1180, 0, 4070, 80, launch_few_g<128, 2>},
        {256, 16, 440, 2510, 8820, 3470, 123, 3740, 65, launch_few_g<256, 1>},  {256, 32, 0, 3930, 9320, 3120, 0, 5130, 82, launch_few_g<256, 2>},
    };
    int cus = 0;
    const hipError_t e = compute_units_of_current_device(&cus);
    if (e != hipSuccess) return hip_result(e);
    const int64_t K = a.K;
    const Tile *best = nullptr;
    int64_t least = 0, rounds = 0;
    for (const Tile &t : tiles) {
        if (a.G > t.ft) continue;  // a group lies inside a tile
        const int64_t n = static_cast<int64_t>((a.E + t.ft - 1) / t.ft) * ((a.T + t.tt - 1) / t.tt);
        const int64_t cost = (n + cus - 1) / cus * t.cost;
        if (!best || cost < least) {
            best = &t;
            least = cost;
            rounds = (n + cus - 1) / cus;
        }
    }
    if (!best->slope) return best->launch(a, s);
    // ns per 1000 k: of the XCD's contiguous share of the workgroups, tokens fastest, how many features' weights; from 3 MB on beyond its L2
    const auto slope = [&](int64_t features, int64_t tokens, int near, int far, int shared) {
        const int64_t nf = (a.E + features - 1) / features, nt = (a.T + tokens - 1) / tokens, share = (nf * nt + 7) / 8;
        const int64_t bytes = 2 * K * (std::min(nf, (share + nt - 2) / nt + 1) * features + a.T);
        const int64_t s0 = near + far * std::min<int64_t>(std::max<int64_t>((bytes - 3000000) / 2000, 0), 1000) / 1000;
        return s0 - s0 * shared / 1000 * (nt - 1) / nt;
    };
    int64_t ns = 95 * (best->ends + rounds * (best->round + slope(best->ft, best->tt, best->slope, best->far, 0) * K / 1000)) / 100;
    const Few *few = nullptr;
    for (const Few &f : fews) {
        if (f.G != a.G) continue;
        const int64_t n = static_cast<int64_t>((a.E + f.G - 1) / f.G) * ((a.T + f.tt - 1) / f.tt);
        const int64_t unit = f.ends + (n + cus - 1) / cus * (f.round + slope(f.G, f.tt, f.slope, f.far, f.shared) * K / 1000);
        const int64_t all = std::max<int64_t>(3950, f.chip + n * (f.G + f.tt) * K * 2 / 1000 * f.mb / 1000);
        if (std::max(unit, all) < ns) {
            few = &f;
            ns = std::max(unit, all);
        }
    }
    return few ? few->launch(a, s) : best->launch(a, s);
}

int launch_gemm_weights(const tpq_layout *L, const void *plan, const uint16_t *Wt, int64_t ldW, int K,
                        uint16_t *Wp, hipStream_t s)
{
    const PlanOffsets o = plan_offsets(L->k, L->r, L->G);
    k_gemm_weights<<<L->E, 256, 0, s>>>(static_cast<const uint8_t *>(plan), L->E, L->k, L->G, L->r, o.idx, o.src,
                                        Wt, ldW, K, Wp);
    return hip_result(hipGetLastError());
}

int launch_gemm_encode(const tpq_layout *L, const uint16_t *X, int64_t T, int64_t ldX, int K,
                       const uint16_t *Wp, uint8_t *codes, uint16_t *scale, uint16_t *zero,
                       uint16_t *outl, uint16_t *Ymsg, int64_t ldYm, hipStream_t s)
{
    GemmArgs a;
    a.X = X;
    a.ldX = ldX;
    a.T = T;
    a.Wp = Wp;
    a.K = K;
    a.E = L->E;
    a.k = L->k;
    a.G = L->G;
    a.r = L->r;
    a.ng = L->ng;
    a.codes = codes;
    a.scale = reinterpret_cast<uint8_t *>(scale);
    a.zero = reinterpret_cast<uint8_t *>(zero);
    a.outl = reinterpret_cast<uint8_t *>(outl);
    a.pitch_codes = L->pitch_codes;
    a.pitch_meta = L->pitch_meta;
    a.pitch_outl = L->pitch_outl;
    a.Ymsg = Ymsg;
    a.ldYm = ldYm;
    return launch_tiles(a, s);
}

}  // namespace tpq
