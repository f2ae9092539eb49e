// tpq_decode_reduce kernel: dequantise the N devices' messages and add them
// (paper Sec. 2, decompression D^(i) and the sum over devices; Fig. 2 caption),
// selected features scattered back to their original columns.
#include <type_traits>

#include "tpq_device.h"
#include "tpq_internal.h"

namespace tpq {

// A word's 8 codes as floats.  One code per byte; the bytes 0 .. 15 read as FP8 (E4M3) are the codes times 2^-9 (subnormals
// and the first binade have the same spacing), so the scaled pair conversion turns two codes into floats at once.
__device__ __forceinline__ void codes8(float (&c)[8], uint32_t w)
{
    const uint32_t lo = w & 0x0F0F0F0Fu, hi = (w >> 4) & 0x0F0F0F0Fu;
    const f32x2 c02 = __builtin_amdgcn_cvt_scalef32_pk_f32_fp8(lo, 512.0f, false);
    const f32x2 c46 = __builtin_amdgcn_cvt_scalef32_pk_f32_fp8(lo, 512.0f, true);
    const f32x2 c13 = __builtin_amdgcn_cvt_scalef32_pk_f32_fp8(hi, 512.0f, false);
    const f32x2 c57 = __builtin_amdgcn_cvt_scalef32_pk_f32_fp8(hi, 512.0f, true);
    c[0] = c02.x; c[1] = c13.x; c[2] = c02.y; c[3] = c13.y;
    c[4] = c46.x; c[5] = c57.x; c[6] = c46.y; c[7] = c57.y;
}

// ... -> code * scale + zero (the product is exact)
__device__ __forceinline__ void dequantise8(float (&x)[8], uint32_t w, float sc, float ze)
{
    float c[8];
    codes8(c, w);
#pragma unroll
    for (int e = 0; e < 8; ++e) x[e] = __builtin_fmaf(c[e], sc, ze);
}

// The 8 B-bit fields of a 64-bit word as floats: field e at bits B*e .. B*e + B - 1.
template <int B>
__device__ __forceinline__ void unpack_codes(uint64_t w, float (&c)[8])
{
#pragma unroll
    for (int e = 0; e < 8; ++e)
        c[e] = static_cast<float>(static_cast<uint32_t>(w >> (B * e)) & ((1u << B) - 1u));
}

// ... less half their range: field - 2^(B - 1) as a float.
template <int B>
__device__ __forceinline__ void unpack_signed(uint64_t w, float (&c)[8])
{
    uint64_t half = 0;
#pragma unroll
    for (int e = 0; e < 8; ++e) half |= 1ull << (B * e + B - 1);
    w ^= half;
#pragma unroll
    for (int e = 0; e < 8; ++e)
        c[e] = static_cast<float>(static_cast<int32_t>(static_cast<uint32_t>(w >> (B * e)) << (32 - B)) >> (32 - B));
}

// acc <- acc (+) x for 8 features at once, in the requested arithmetic.  In the bf16 chain acc is the last sum before its
// rounding: term and sum are rounded by one pair conversion and added by one dot product with (1, 1), which takes -0 + -0 for +0;
// without DOT by an addition.  Finished by round8().
template <int ACC, bool DOT = true>
__device__ __forceinline__ void accumulate8(float (&acc)[8], const float (&x)[8], bool first)
{
    if (first) {
#pragma unroll
        for (int e = 0; e < 8; ++e) acc[e] = x[e];
    } else if (ACC == TPQ_ACC_BF16 && DOT) {
        bf16_chain8(acc, x);
    } else {
#pragma unroll
        for (int e = 0; e < 8; ++e)
            acc[e] = ACC == TPQ_ACC_BF16 ? round_via_bf16(acc[e]) + round_via_bf16(x[e]) : acc[e] + x[e];
    }
}

template <int ACC>
__device__ __forceinline__ void round8(float (&acc)[8])
{
    if (ACC == TPQ_ACC_BF16) {
#pragma unroll
        for (int e = 0; e < 8; ++e) acc[e] = round_via_bf16(acc[e]);
    }
}

// The literal bf16 chain by additions, a rank at a time, for the sums that bf16_chain8() gets wrong: those that are -0.  They are only where every
// term is: a zero point of -0 and a scale with its sign set (less than 0, or -0) in every message.  The encoder sends neither, so
// callers come here only where a lane sees that sign in the first rank's message.
template <bool GEN>
__device__ __forceinline__ void exact_chain(float (&acc)[8], uint32_t N, uint32_t bits, const RankPtrs &codesp, const RankPtrs &scalep,
                                            const RankPtrs &zerop, uint32_t off_codes, uint32_t off_meta)
{
#pragma nounroll
    for (uint32_t i = 0; i < N; ++i) {
        const uint8_t *pc = static_cast<const uint8_t *>(codesp.p[i]) + off_codes;
        const uint64_t w = GEN ? *reinterpret_cast<const u64_a1 *>(pc) : *reinterpret_cast<const uint32_t *>(pc);
        const float sc = bf16_bits_to_f32(*reinterpret_cast<const uint16_t *>(static_cast<const uint8_t *>(scalep.p[i]) + off_meta));
        const float ze = bf16_bits_to_f32(*reinterpret_cast<const uint16_t *>(static_cast<const uint8_t *>(zerop.p[i]) + off_meta));
        float x[8];
#pragma unroll
        for (uint32_t e = 0; e < 8; ++e)
            x[e] = __builtin_fmaf(static_cast<float>(static_cast<uint32_t>(w >> (bits * e)) & ((1u << bits) - 1u)), sc, ze);
        accumulate8<TPQ_ACC_BF16, false>(acc, x, i == 0u);
    }
}

// ---------------------------------------------------------------------------
// Stores of one pass and row.  The wave parks its 512 sums in LDS in compacted order
// (8 per lane), then lane s takes the pass's s-th store entry from the plan: a block of
// 8 consecutive features that go to 8 consecutive columns -- read back from LDS at
// whatever feature offset the block starts (two aligned 16-byte reads and a funnel
// shift), written with one 128-bit store (two for fp32 output) -- or, for the few
// features of runs shorter than 8, a single feature.  Selected columns cut the stream of
// features into runs; blocks follow the runs, so no store is split feature by feature.
// st: this wave's staging area (64 x 16 bytes for bf16 output, 128 x 16 for fp32).
// e0, e1: the entries of slots lane and 64 + lane (loaded early); further entries are
// read here.  All 64 lanes must call.
// ---------------------------------------------------------------------------
template <int OUT>
__device__ __forceinline__ void store_pass(u32x4 *st, const float (&acc)[8], uint8_t *out_row,
                                           uint32_t lane, const uint32_t *entries, uint32_t nb,
                                           uint32_t nall, uint32_t e0, uint32_t e1)
{
    if (OUT == TPQ_OUT_FP32) {
        st[2u * lane] = u32x4{__float_as_uint(acc[0]), __float_as_uint(acc[1]), __float_as_uint(acc[2]),
                              __float_as_uint(acc[3])};
        st[2u * lane + 1u] = u32x4{__float_as_uint(acc[4]), __float_as_uint(acc[5]),
                                   __float_as_uint(acc[6]), __float_as_uint(acc[7])};
    } else {
        st[lane] = u32x4{pack_bf16x2(acc[0], acc[1]), pack_bf16x2(acc[2], acc[3]),
                         pack_bf16x2(acc[4], acc[5]), pack_bf16x2(acc[6], acc[7])};
    }
    wave_lds_fence();
    for (uint32_t s0 = 0; s0 < nall; s0 += 64) {
        const uint32_t slot = s0 + lane;
        uint32_t e = s0 == 0 ? e0 : e1;
        if (s0 >= 128) e = slot < nall ? entries[slot] : 0u;
        const uint32_t col = e & 0xFFFFu, at = (e >> 16) & 0x1FFu;
        if (slot < nb) {
            if (OUT == TPQ_OUT_FP32) {
                // 8 dwords from dword `at` on: three aligned reads, shift by at % 4 dwords
                const uint32_t q = at >> 2;
                const u32x4 A = st[q], B = st[min(q + 1u, 127u)], C = st[min(q + 2u, 127u)];
                // (selects between named values: an indexed array here ends up in memory)
                const bool s2 = (at & 2u) != 0, s1 = (at & 1u) != 0;
#define TPQ_SEL(c, hi, lo) ((c) ? (hi) : (lo))
                const uint32_t u0 = TPQ_SEL(s2, A.z, A.x), u1 = TPQ_SEL(s2, A.w, A.y), u2 = TPQ_SEL(s2, B.x, A.z),
                               u3 = TPQ_SEL(s2, B.y, A.w), u4 = TPQ_SEL(s2, B.z, B.x), u5 = TPQ_SEL(s2, B.w, B.y),
                               u6 = TPQ_SEL(s2, C.x, B.z), u7 = TPQ_SEL(s2, C.y, B.w), u8 = TPQ_SEL(s2, C.z, C.x);
                const uint32_t o[8] = {TPQ_SEL(s1, u1, u0), TPQ_SEL(s1, u2, u1), TPQ_SEL(s1, u3, u2),
                                       TPQ_SEL(s1, u4, u3), TPQ_SEL(s1, u5, u4), TPQ_SEL(s1, u6, u5),
                                       TPQ_SEL(s1, u7, u6), TPQ_SEL(s1, u8, u7)};
                __builtin_nontemporal_store(u32x4{o[0], o[1], o[2], o[3]},
                                            reinterpret_cast<u32x4_a4 *>(out_row + 4u * col));
                __builtin_nontemporal_store(u32x4{o[4], o[5], o[6], o[7]},
                                            reinterpret_cast<u32x4_a4 *>(out_row + 4u * col + 16u));
            } else {
                // 8 half-words from half-word `at` on: two aligned reads, shift by at % 8
                const uint32_t q = at >> 3;
                const u32x4 A = st[q], B = st[min(q + 1u, 63u)];
                const bool s2 = (at & 4u) != 0, s1 = (at & 2u) != 0;
                const uint32_t sh = (at & 1u) << 4;
                const uint32_t u0 = TPQ_SEL(s2, A.z, A.x), u1 = TPQ_SEL(s2, A.w, A.y), u2 = TPQ_SEL(s2, B.x, A.z),
                               u3 = TPQ_SEL(s2, B.y, A.w), u4 = TPQ_SEL(s2, B.z, B.x), u5 = TPQ_SEL(s2, B.w, B.y);
                const uint32_t v0 = TPQ_SEL(s1, u1, u0), v1 = TPQ_SEL(s1, u2, u1), v2 = TPQ_SEL(s1, u3, u2),
                               v3 = TPQ_SEL(s1, u4, u3), v4 = TPQ_SEL(s1, u5, u4);
#undef TPQ_SEL
                const uint32_t o[4] = {__builtin_amdgcn_alignbit(v1, v0, sh), __builtin_amdgcn_alignbit(v2, v1, sh),
                                       __builtin_amdgcn_alignbit(v3, v2, sh), __builtin_amdgcn_alignbit(v4, v3, sh)};
                __builtin_nontemporal_store(u32x4{o[0], o[1], o[2], o[3]},
                                            reinterpret_cast<u32x4_a2 *>(out_row + 2u * col));
            }
        } else if (slot < nall) {
            const uint32_t *stw = reinterpret_cast<const uint32_t *>(st);
            if (OUT == TPQ_OUT_FP32) {
                *reinterpret_cast<uint32_t *>(out_row + 4u * col) = stw[at];
            } else {
                const uint32_t w = stw[at >> 1];
                *reinterpret_cast<uint16_t *>(out_row + 2u * col) =
                    static_cast<uint16_t>((at & 1u) ? (w >> 16) : (w & 0xFFFFu));
            }
        }
    }
    // A later call's staging writes follow these reads in program order, and a wave's LDS
    // operations execute in order: nothing to wait for (a fence here would also hold the
    // wave until its global stores have completed).
    __builtin_amdgcn_wave_barrier();
}

// Before a batch's loads and behind each rank's.  Else the compiler takes the first loads that two batch sizes have in common ahead
// of the branch between them, leaves the others behind a wait for those, and moves the last rank's behind the others' arithmetic.
#define TPQ_LOADS_STAY(NB) asm volatile("; %0 ranks" ::"n"(NB) : "memory")

// one more term of the accumulation (fp32 add; rounded to bf16 in the literal bf16 chain)
template <int ACC>
__device__ __forceinline__ float add_term(float acc, float x)
{
    const float s = acc + x;
    return ACC == TPQ_ACC_BF16 ? round_via_bf16(s) : s;
}

// A wave's sums by column: 512 columns of its pass as fp32, 7 more that a chunk across the pass's
// end may touch, and one place for features of other passes.
constexpr uint32_t kRowQuads = 130, kRowNowhere = 519;

// The features of a chunk -> their columns.  cols: the chunk's 8 columns (16 bits each), col0: the pass's first.
__device__ __forceinline__ void scatter_chunk(float *row, const float (&x)[8], const u32x4 &cols, uint32_t col0, bool whole)
{
    typedef unsigned short u16x2 __attribute__((ext_vector_type(2)));
    const uint32_t first = cols.x & 0xFFFFu, at = first - col0;
    if (whole && (cols.w >> 16) - first == 7u && at < 512u) {  // 8 neighbours: two stores
        *reinterpret_cast<u32x4_a4 *>(row + at) =
            u32x4{__float_as_uint(x[0]), __float_as_uint(x[1]), __float_as_uint(x[2]), __float_as_uint(x[3])};
        *reinterpret_cast<u32x4_a4 *>(row + at + 4u) =
            u32x4{__float_as_uint(x[4]), __float_as_uint(x[5]), __float_as_uint(x[6]), __float_as_uint(x[7])};
    } else {
        // feature by feature, the last first: positions past the row's last feature name its column
        // too, and its own value has to be the one that stays
        const uint32_t cw[4] = {cols.x, cols.y, cols.z, cols.w};
        const unsigned short c16 = static_cast<unsigned short>(col0);
#pragma unroll
        for (int w = 3; w >= 0; --w) {
            const u16x2 d2 = __builtin_elementwise_min(__builtin_bit_cast(u16x2, cw[w]) - u16x2{c16, c16},
                                                       u16x2{kRowNowhere, kRowNowhere});
            const uint32_t d = __builtin_bit_cast(uint32_t, d2);
            row[d >> 16] = x[2 * w + 1];
            row[d & 0xFFFFu] = x[2 * w];
        }
    }
}

// v holds four ranks' values of 16 columns, a row of 16 lanes each: acc <- acc (+) rank 4 rq (+) .. in every row
template <int ACC>
__device__ __forceinline__ void add_quad(float &acc, uint32_t v, uint32_t rq, uint32_t N)
{
    const auto a = __builtin_amdgcn_permlane16_swap(v, v, false, false);
    const uint32_t even = a[0], odd = a[1];
    const auto b = __builtin_amdgcn_permlane32_swap(even, even, false, false);
    const auto c = __builtin_amdgcn_permlane32_swap(odd, odd, false, false);
    const float x[4] = {bf16_bits_to_f32(b[0]), bf16_bits_to_f32(c[0]), bf16_bits_to_f32(b[1]), bf16_bits_to_f32(c[1])};
    const uint32_t left = N - 4u * rq;  // (uniform, 1 or more)
    acc = rq == 0u ? x[0] : add_term<ACC>(acc, x[0]);
    if (left >= 4u) {
        acc = add_term<ACC>(add_term<ACC>(add_term<ACC>(acc, x[1]), x[2]), x[3]);
    } else {
        if (left > 1u) acc = add_term<ACC>(acc, x[1]);
        if (left > 2u) acc = add_term<ACC>(acc, x[2]);
    }
}

// ---------------------------------------------------------------------------
// One wavefront handles one column pass of one output row: up to 64 blocks of 8 columns, the chunks (up to
// 64, one per lane) whose features lie there, and the selected features between them.  Waves
// are independent (no barrier; LDS only as each wave's private row of sums), so a CU always holds
// waves in every phase and loads, arithmetic and stores overlap.
//
// Every lane issues its loads at once -- one 32-bit word of codes (8 features) per rank, the group's scale
// and zero per rank, the columns of its 8 features, the selected features' values (four ranks of
// 16 columns per load) -- then dequantises (code * scale + zero: one FMA, the product is exact) and
// accumulates in ascending rank order.  The sums meet in LDS in column order, where a lane takes 8
// neighbouring columns, adds the epilogue's terms and stores them: one aligned 128-bit store (two for fp32
// output) per lane, every line of the output written whole, by one wave, once.
// Why by columns: as passes of 512 compacted features the sums left in runs between selected columns -- 2-byte
// aligned stores, a second, nearly empty round of them per pass, the epilogue's operands loaded the same way,
// and waves of their own for the selected features.  Kernel times, before and now (T = 2048, E = 5120, k = 80, N = 8
// unless said): with residual and bias 25.3 -> 19.9 us (fp32), 29.6 -> 23.7 (bf16 chain); without 17.5 -> 17.2; 16384 x
// 8192, k = 341, N = 16, fp32 output 480 -> 420; 6 bits, 1777 x 5000, N = 5 22.8 -> 21.3.  Bound by what a compute unit has
// outstanding to memory, a wave's chain of loads at small sizes, and by instruction issue in the bf16 chain.  Eight waves per SIMD.
// Ranks come in batches with code of their own for 1 to 8 (2, 4, 6 and 8 where that code is long: other code widths, LANES).
// As batches of 8 whatever was left, the loads of ranks that are not there were issued too (the last rank's again), and the
// compiler put a rank's loads behind the others' arithmetic, a second wait for memory.  Kernel times at T = 2048, E = 5120, k = 80, fp32 / bf16 chain,
// before -> now: N = 2 13.4 -> 11.2 / 13.5 -> 11.6 us, N = 3 13.8 -> 11.8 / 14.4 -> 12.4, N = 5, 6 bits 19.7 -> 17.8 / 19.9 -> 17.9,
// N = 8 16.7 -> 16.2 / 20.7 -> 18.4, with fp32 output 20.2 -> 20.0 / 22.6 -> 21.1, with residual and bias 19.3 -> 19.4 / 23.1 -> 21.6; N = 12, k = 20, 5 bits (rows) 41.3 -> 34.4 / 41.9 -> 34.8; N = 12, 4096 rows, k = 200
// 45.3 -> 39.8 / 52.7 -> 45.8.
// grid: (row, pass) pairs, 4 per workgroup, workgroups rounded up to a multiple of 8.
// ---------------------------------------------------------------------------
//
// GEN selects code widths other than 4 bits (Sec. 4, the experiment that varies the bits
// of the quantised features): a chunk's 8 codes are b bytes at byte chunk * b of the row,
// fetched with one 64-bit load at that byte (the row's pitch leaves room behind the last).
//
// FUSED adds the block's epilogue (Sec. 2: the sum over the devices plus the bias): an addend row and / or the
// bias as two more terms of the accumulation.
// LANES: how the selected features come.  Without it (8 ranks at most, few selected features): four ranks of 16 columns
// per load, a rank's row of lanes with its own pointer.  The pointers are fetched ahead of everything, and the first 16
// columns (mostly all there are) behind the first messages: picked from scalar registers the pointers cost 40 instructions a
// wave, and fetched behind the messages' loads a second wait for all of those (18.7 and 21.5 us at T = 2048, E = 5120, N = 8).
// With it: a lane per column, 64 of them loaded and added with every 8 ranks' messages; 8 loads and 3 registers more (seven waves per
// SIMD), but nothing waits for pointers behind the messages, and 17 or more columns are no path of their own.  Kernel
// times without / with / as rows (k_decode_rows), bf16 output: N = 4, k = 80 14.8 / 16.0 / 16.0 us; N = 8, k = 80 16.4 / 16.4 / 16.8; N = 8, k = 213
// 18.8 / 16.5 / 21.7; N = 64, 64 rows 14.5 / 11.8 / 10.1.
template <int LPG, int ACC, int OUT, bool GEN, bool FUSED, bool LANES>
__global__ __launch_bounds__(256, (GEN ? 7 : 8) - LANES) void k_decode_pass(DecodeArgs a, RankPtrs codesp, RankPtrs scalep,
                                                     RankPtrs zerop, RankPtrs outlp)
{
    // Nothing is stored unless the header says that the plan is good; the loads do not wait for that
    // answer (whatever the plan's tables hold, they are kept inside the plan, the messages and the
    // addend).
    const uint32_t lane = threadIdx.x & 63u;
    const uint32_t wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    // Each XCD works through one contiguous range of (row, pass) pairs, a row's passes one after
    // the other: the lines two neighbouring waves share (a row's scales and zeros, the ends of their code
    // ranges) then meet in one L2, close in time.
    const uint32_t E = static_cast<uint32_t>(a.E), k = static_cast<uint32_t>(a.k);
    const uint32_t passes = static_cast<uint32_t>(a.cpasses);
    const uint32_t pair = xcd_contiguous_index(blockIdx.x, gridDim.x) * 4u + wave;
    const uint32_t stride = static_cast<uint32_t>(a.cpass_stride);
    // (by multiplication: exact below 2^32 / stride, which the host keeps)
    const uint32_t t = stride == 1u ? pair : __umulhi(pair, a.cpass_magic), task = pair - t * stride;
    if (t >= static_cast<uint32_t>(a.T) || task >= passes) return;  // (the grid is rounded up to 8 blocks of 4)

    constexpr uint32_t OB = OUT == TPQ_OUT_FP32 ? 4u : 2u;  // bytes per output value
    const uint32_t N = static_cast<uint32_t>(a.n_ranks);
    const uint32_t ng = static_cast<uint32_t>(a.ng);
    const uint32_t chunks = static_cast<uint32_t>(a.chunks);
    const uint4 cp = reinterpret_cast<const uint4 *>(a.plan + a.off_cpass)[task];
    const uint32_t n_blk = min(cp.x >> 16, 64u), blk0 = min(cp.x & 0xFFFFu, E / 8u - 1u), col0 = 8u * blk0;
    const uint32_t n_sel = min(cp.z >> 16, k), s0 = min(cp.z & 0xFFFFu, k);
    const uint32_t n_chunk = cp.y >> 16;
    // (one word, made here, where the header has come with the pass: kept for later it is seven registers)
    const PlanHeader *ph = reinterpret_cast<const PlanHeader *>(a.plan);
    uint32_t refuse = (ph->magic ^ kPlanMagic) | static_cast<uint32_t>((ph->status ^ kPlanOk) | (ph->E ^ a.E) | (ph->k ^ a.k) | (ph->G ^ a.G));
    asm volatile("" : "+s"(refuse));

    // (The host fills the table up to a multiple of 8 with the first pointer, and passes the codes' pointers at a
    // pitch of 0 where there are no selected features; nobody looks at what is read then.)
    const int32_t *idx = reinterpret_cast<const int32_t *>(a.plan + a.off_idx);
    const uint32_t off_outl = t * static_cast<uint32_t>(a.pitch_outl);
    const uint32_t sel_at = min(s0 + (LANES ? lane : lane & 15u), max(k, 1u) - 1u), off_sel = off_outl + 2u * sel_at;
    const void *sel_p0 = nullptr, *sel_p1 = nullptr;
    if constexpr (!LANES) {
        const void *const *po = outlp.p + (lane >> 4);
        sel_p0 = po[0];
        sel_p1 = po[4];
    }
    auto load_sel = [&](const void *p) __attribute__((always_inline)) {
        return static_cast<uint32_t>(*reinterpret_cast<const uint16_t *>(static_cast<const uint8_t *>(p) + off_sel));
    };
    uint32_t sel_col = 0u, sel_v0 = 0u, sel_v1 = 0u;
    float sel = 0.0f;

    // One 32-bit byte offset per section serves every rank (the host keeps
    // T * pitch below 2^31 per launch): the rank only changes the scalar base.
    const uint32_t chunk = min((cp.y & 0xFFFFu) + min(lane, max(n_chunk, 1u) - 1u), max(chunks, 1u) - 1u);
    const uint32_t g = min(chunk / LPG, max(ng, 1u) - 1u);
    const uint32_t off_codes = t * static_cast<uint32_t>(a.pitch_codes) +
                               (GEN ? static_cast<uint32_t>(a.bits) : 4u) * chunk;
    const uint32_t off_meta = t * static_cast<uint32_t>(a.pitch_meta) + 2u * g;
    const bool quant = n_chunk > 0 && chunks > 0;
    const u32x4 cols = reinterpret_cast<const u32x4 *>(a.plan + a.off_src)[chunk];  // (in the plan also where there is none)
    float acc[8];
    uint64_t signs = 0u;  // bf16 chain: the lanes that see a sign in the first rank's scale (exact_chain())

    // NB ranks at a time: all loads first, then the arithmetic, a rank's as soon as its loads are there.  left: ranks from i0
    // on, NB or one less (GEN, LANES; the host fills the pointer tables up to an even number).
    // (the code width is a compile-time constant inside: one copy of the loop per width)
    auto batch = [&](uint32_t i0, uint32_t left, auto size_tag, auto bits_tag, auto first_tag, auto order_tag) __attribute__((always_inline)) {
        constexpr int NB = decltype(size_tag)::value;
        constexpr int BITS = decltype(bits_tag)::value;
        constexpr bool FIRST = decltype(first_tag)::value;
        constexpr bool ORDER = decltype(order_tag)::value;
        uint32_t w[NB], sb[NB], zb[NB];
        uint64_t wq[NB];  // GEN
        // (a base of this branch's own: else all sizes' pointers are loaded ahead of the branch, and spill where registers are
        // short: N = 8, bf16 chain 18.3 -> 24.5 us, fp32 with fp32 output 20.0 -> 25.2.  In fp32 with bf16 output they nearly fit, and
        // that is faster: with residual and bias 19.4 against 19.8)
        uint32_t base = i0;
        if constexpr (ACC == TPQ_ACC_BF16 || OUT == TPQ_OUT_FP32 || GEN || LANES) asm volatile("" : "+s"(base));
        const void *const *pc = codesp.p + base;
        const void *const *ps = scalep.p + base;
        const void *const *pz = zerop.p + base;
        uint32_t oc = off_codes, om = off_meta;
        if constexpr (ORDER) TPQ_LOADS_STAY(NB);
        // (offsets of this branch's own: a base per rank beside them in one load instruction, no 64-bit sums.  Batches without an
        // order share theirs: N = 64, 64 rows, fp32 output 12.5 -> 11.1 us)
        if constexpr (ORDER) asm volatile("" : "+v"(oc), "+v"(om));
        uint32_t vb[NB];  // LANES
        if constexpr (LANES) {
#pragma unroll
            for (int j = 0; j < NB; ++j) vb[j] = load_sel((outlp.p + base)[j]);
        }
#pragma unroll
        for (int j = 0; j < NB; ++j) {
            if constexpr (GEN)
                wq[j] = __builtin_nontemporal_load(reinterpret_cast<const u64_a1 *>(
                    static_cast<const uint8_t *>(pc[j]) + oc));
            else
                w[j] = __builtin_nontemporal_load(reinterpret_cast<const uint32_t *>(
                    static_cast<const uint8_t *>(pc[j]) + oc));
            sb[j] = *reinterpret_cast<const uint16_t *>(static_cast<const uint8_t *>(ps[j]) + om);
            zb[j] = *reinterpret_cast<const uint16_t *>(static_cast<const uint8_t *>(pz[j]) + om);
            if constexpr (ORDER) TPQ_LOADS_STAY(NB);
        }
        if constexpr (FIRST && !LANES) {
            __builtin_amdgcn_sched_barrier(0);  // (else the wait for their pointers comes before the messages' loads)
            sel_v0 = load_sel(sel_p0);
            sel_v1 = load_sel(sel_p1);
            sel_col = static_cast<uint32_t>(idx[sel_at]);
        }
        if constexpr (LANES) {
#pragma unroll
            for (int j = 0; j < NB; ++j) {
                const float v = bf16_bits_to_f32(vb[j]);
                if (j < NB - 1 || left == NB) sel = FIRST && j == 0 ? v : add_term<ACC>(sel, v);  // uniform
            }
        }
#pragma unroll
        for (int j = 0; j < NB; ++j) {
            if ((!GEN && !LANES) || j < NB - 1 || left == NB) {  // uniform
                const float sc = bf16_bits_to_f32(sb[j]), ze = bf16_bits_to_f32(zb[j]);
                float x[8];
                if constexpr (GEN) {
                    float c[8];
                    unpack_codes<BITS>(wq[j], c);
#pragma unroll
                    for (int e = 0; e < 8; ++e) x[e] = __builtin_fmaf(c[e], sc, ze);  // product exact
                } else {
                    dequantise8(x, w[j], sc, ze);
                }
                if (ACC == TPQ_ACC_BF16 && FIRST && j == 0) signs = __builtin_amdgcn_ballot_w64(sb[j] >= 0x8000u);
                accumulate8<ACC>(acc, x, FIRST && j == 0);
            }
        }
    };
    auto size = [&](uint32_t i0, uint32_t left, auto size_tag, auto bits_tag, auto first_tag) __attribute__((always_inline)) {
        constexpr int NB = decltype(size_tag)::value;
        if constexpr (!GEN && !LANES) {
            if (left < NB) {
                batch(i0, left, std::integral_constant<int, NB - 1>{}, bits_tag, first_tag, std::true_type{});
                return;
            }
        }
        batch(i0, left, size_tag, bits_tag, first_tag, std::true_type{});
    };
    // ranks i0 .. N - 1, at most 8
    auto some = [&](uint32_t i0, auto bits_tag, auto first_tag) __attribute__((always_inline)) {
        const uint32_t left = N - i0;
        if (left > 6u) size(i0, left, std::integral_constant<int, 8>{}, bits_tag, first_tag);
        else if (left > 4u) size(i0, left, std::integral_constant<int, 6>{}, bits_tag, first_tag);
        else if (left > 2u) size(i0, left, std::integral_constant<int, 4>{}, bits_tag, first_tag);
        else size(i0, left, std::integral_constant<int, 2>{}, bits_tag, first_tag);
    };
    auto run = [&](auto bits_tag) __attribute__((always_inline)) {
        // (the first batch is code of its own: it starts the sums and fetches the selected features)
        if constexpr (!LANES) {
            some(0, bits_tag, std::true_type{});  // 8 ranks at most
        } else {
            if (N <= 8u) {
                some(0, bits_tag, std::true_type{});
            } else {
                // in fp32 the compiler may load the next ranks ahead of a batch's arithmetic (held back, N = 16, 8192 x 8192, fp32
                // output takes 241 us instead of 218); in the bf16 chain that costs more than it gives (N = 12, 4096 x 5120
                // 46.1 against 43.8).  Except from the second batch on at other code widths, where few rows of many ranks wait for the chain
                // of batches (N = 32, 81 rows of 4608, 5 bits, fp32 output 10.9 -> 9.4 us; many rows, N = 64, 245 x 5120, 6 bits 32.8 -> 33.8)
                const std::integral_constant<int, 8> eight;
                const std::integral_constant<bool, ACC == TPQ_ACC_BF16> order;
                const std::integral_constant<bool, ACC == TPQ_ACC_BF16 && !GEN> later;
                batch(0, 8u, eight, bits_tag, std::true_type{}, order);
                if (ACC == TPQ_ACC_BF16 && signs) return;  // (begun again below)
                uint32_t i0 = 8;
                if constexpr (GEN) {
                    for (; i0 + 8 <= N; i0 += 8) batch(i0, 8u, eight, bits_tag, std::false_type{}, later);
                    if (i0 < N) some(i0, bits_tag, std::false_type{});
                } else {  // (the last 8 outside of the loop: N = 16 220 us instead of 230; at other code widths that would spill)
                    for (; i0 + 8 < N; i0 += 8) batch(i0, 8u, eight, bits_tag, std::false_type{}, order);
                    if (i0 + 8 == N)
                        batch(i0, 8u, eight, bits_tag, std::false_type{}, order);
                    else
                        some(i0, bits_tag, std::false_type{});
                }
            }
        }
    };
    __shared__ u32x4 rows[4 * kRowQuads];
    float *const row = reinterpret_cast<float *>(rows + wave * kRowQuads);
    if (quant) {
        if constexpr (GEN) {
            switch (a.bits) {
            case 2: run(std::integral_constant<int, 2>{}); break;
            case 3: run(std::integral_constant<int, 3>{}); break;
            case 5: run(std::integral_constant<int, 5>{}); break;
            case 6: run(std::integral_constant<int, 6>{}); break;
            default: run(std::integral_constant<int, 8>{}); break;
            }
        } else {
            run(std::integral_constant<int, 4>{});
        }
        if (ACC == TPQ_ACC_BF16 && signs) {
            exact_chain<GEN>(acc, N, GEN ? static_cast<uint32_t>(a.bits) : 4u, codesp, scalep, zerop, off_codes, off_meta);
            if constexpr (LANES) {
#pragma nounroll
                for (uint32_t i = 0; i < N; ++i) {
                    const float v = bf16_bits_to_f32(load_sel(outlp.p[i]));
                    sel = i == 0u ? v : add_term<ACC>(sel, v);
                }
            }
        }
        round8<ACC>(acc);
        scatter_chunk(row, acc, cols, col0, chunk < static_cast<uint32_t>(a.r) >> 3);
    }
    if (refuse) return;

    // ---- selected features ----------------------------------------------------------------
    uint32_t done = 0u;
    if constexpr (LANES) {
        if (quant) {
            if (lane < n_sel) row[min(static_cast<uint32_t>(idx[sel_at]) - col0, kRowNowhere)] = sel;
            done = 64u;
        }
    } else if (quant && n_sel <= 16u) {
        if (n_sel > 0) {
            float v = 0.0f;
            add_quad<ACC>(v, sel_v0, 0u, N);
            if (N > 4u) add_quad<ACC>(v, sel_v1, 1u, N);
            if (lane < n_sel) row[min(sel_col - col0, kRowNowhere)] = v;
        }
        done = n_sel;
    }
    for (uint32_t p0 = done; p0 < n_sel; p0 += 64) {  // those that are left: a lane per column
        const uint32_t p = min(s0 + p0 + lane, k - 1u);
        float v = 0.0f;
        for (uint32_t i0 = 0; i0 < N; i0 += 8) {
            uint32_t b[8];
#pragma unroll
            for (int jj = 0; jj < 8; ++jj)
                b[jj] = reinterpret_cast<const uint16_t *>(
                    static_cast<const uint8_t *>(outlp.p[min(i0 + jj, N - 1u)]) + off_outl)[p];
#pragma unroll
            for (int jj = 0; jj < 8; ++jj)
                if (i0 + jj < N) v = i0 + jj == 0 ? bf16_bits_to_f32(b[jj]) : add_term<ACC>(v, bf16_bits_to_f32(b[jj]));
        }
        if (p0 + lane < n_sel) row[min(static_cast<uint32_t>(idx[p]) - col0, kRowNowhere)] = v;
    }
    wave_lds_fence();

    // ---- a lane's columns: the epilogue's terms, the store --------------------------------
    uint8_t *const out = static_cast<uint8_t *>(a.out) + (static_cast<int64_t>(t) * a.ldOut + col0) * OB;
    const uint8_t *addend = nullptr, *bias = nullptr;
    if constexpr (FUSED) {
        if (a.addend) addend = a.addend + (static_cast<int64_t>(t) * a.ldAdd + col0) * 2;
        if (a.bias) bias = a.bias + 2u * col0;
    }
    if (OUT == TPQ_OUT_FP32) {
#pragma unroll
        for (int h = 0; h < 2; ++h) {  // 4 columns per lane and store: neighbouring lanes', neighbouring quads
            const uint32_t q = 64u * h + lane;
            if (q < 2u * n_blk) {
                const u32x4 y = rows[wave * kRowQuads + q];
                float f[4] = {__uint_as_float(y.x), __uint_as_float(y.y), __uint_as_float(y.z), __uint_as_float(y.w)};
                if constexpr (FUSED) {
                    typedef uint32_t u32x2_a2 __attribute__((ext_vector_type(2), aligned(2)));
#define TPQ_ADD4(src)                                                           \
    {                                                                           \
        const u32x2_a2 z = *reinterpret_cast<const u32x2_a2 *>((src) + 8u * q); \
        f[0] = add_term<ACC>(f[0], bf16_lo_to_f32(z.x));                        \
        f[1] = add_term<ACC>(f[1], bf16_hi_to_f32(z.x));                        \
        f[2] = add_term<ACC>(f[2], bf16_lo_to_f32(z.y));                        \
        f[3] = add_term<ACC>(f[3], bf16_hi_to_f32(z.y));                        \
    }
                    if (addend) TPQ_ADD4(addend)
                    if (bias) TPQ_ADD4(bias)
#undef TPQ_ADD4
                }
                __builtin_nontemporal_store(u32x4{__float_as_uint(f[0]), __float_as_uint(f[1]), __float_as_uint(f[2]),
                                                  __float_as_uint(f[3])},
                                            reinterpret_cast<u32x4 *>(out + 16u * q));
            }
        }
    } else if (lane < n_blk) {
        const u32x4 y0 = rows[wave * kRowQuads + 2u * lane], y1 = rows[wave * kRowQuads + 2u * lane + 1u];
        float f[8] = {__uint_as_float(y0.x), __uint_as_float(y0.y), __uint_as_float(y0.z), __uint_as_float(y0.w),
                      __uint_as_float(y1.x), __uint_as_float(y1.y), __uint_as_float(y1.z), __uint_as_float(y1.w)};
        if constexpr (FUSED) {
#define TPQ_ADD8(src)                                                                 \
    {                                                                                 \
        const u32x4 z = *reinterpret_cast<const u32x4_a2 *>((src) + 16u * lane);      \
        f[0] = add_term<ACC>(f[0], bf16_lo_to_f32(z.x)); f[1] = add_term<ACC>(f[1], bf16_hi_to_f32(z.x)); \
        f[2] = add_term<ACC>(f[2], bf16_lo_to_f32(z.y)); f[3] = add_term<ACC>(f[3], bf16_hi_to_f32(z.y)); \
        f[4] = add_term<ACC>(f[4], bf16_lo_to_f32(z.z)); f[5] = add_term<ACC>(f[5], bf16_hi_to_f32(z.z)); \
        f[6] = add_term<ACC>(f[6], bf16_lo_to_f32(z.w)); f[7] = add_term<ACC>(f[7], bf16_hi_to_f32(z.w)); \
    }
            if (addend) TPQ_ADD8(addend)
            if (bias) TPQ_ADD8(bias)
#undef TPQ_ADD8
        }
        __builtin_nontemporal_store(
            u32x4{pack_bf16x2(f[0], f[1]), pack_bf16x2(f[2], f[3]), pack_bf16x2(f[4], f[5]), pack_bf16x2(f[6], f[7])},
            reinterpret_cast<u32x4 *>(out + 16u * lane));
    }
}

// ---------------------------------------------------------------------------
// The same sums by passes of 512 compacted features, selected features in waves of their own: for more than 8 ranks, bf16
// output and no epilogue, or 8 ranks' wide codes (decode_form()).  With that many ranks the loads are what counts: a pass's codes are two whole lines
// per rank (a column pass's lie across three), and the selected features' lines are asked for once a row instead of in every
// pass, so that the L2 gets 10.3 million requests where column passes make 12.4 (N = 16, 8192 x 8192, k = 128).  Kernel
// times, rows / column passes (LANES): that 166 / 193 us; N = 12, 8192 x 5120, k = 80 85.7 / 91.7; N = 16, 8192 x 5120 100 / 116;
// N = 64, 64 x 5120 10.1 / 11.8.  But the sums leave at 2-byte alignment between selected columns, so that column passes win
// with more of those (N = 16, 8192 x 5120, k = 213 133 / 118), with fp32 output and with an epilogue.
// grid: (row, group of 4 waves) pairs, rounded up to a multiple of 8.
// ---------------------------------------------------------------------------
template <int LPG, int ACC, bool GEN>
__global__ __launch_bounds__(256) void k_decode_rows(DecodeArgs a, RankPtrs codesp, RankPtrs scalep,
                                                     RankPtrs zerop, RankPtrs outlp)
{
    // Nothing is stored unless the header says that the plan is good; the pass waves'
    // loads do not wait for that answer (the message sections do not depend on the plan,
    // and reads of the plan's tables are kept inside the plan buffer whatever it holds).
    const bool bad = plan_header_bad(a.plan, a.E, a.k, a.G);
    const uint32_t lane = threadIdx.x & 63u;
    const uint32_t wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const uint32_t passes = static_cast<uint32_t>(a.chunks_padded) >> 6;
    // Each XCD works through one contiguous range of (row, wave group) pairs, a row's
    // groups one after the other: the lines two neighbouring waves share (a row's scales
    // and zeros, the ends of their code ranges, the output lines at a pass boundary)
    // then meet in one L2, close in time.
    const uint32_t ny = (passes + ((static_cast<uint32_t>(a.k) + 63u) >> 6) + 3u) >> 2;
    const uint32_t logical = xcd_contiguous_index(blockIdx.x, gridDim.x);
    const uint32_t t = logical / ny;
    if (t >= static_cast<uint32_t>(a.T)) return;  // (the grid is rounded up to 8 blocks)
    const uint32_t task = (logical - t * ny) * 4u + wave;

    constexpr int OUT = TPQ_OUT_BF16;
    constexpr uint32_t OB = 2u;  // bytes per output value
    const uint32_t N = static_cast<uint32_t>(a.n_ranks);
    const uint32_t ng = static_cast<uint32_t>(a.ng);
    const uint32_t chunks = static_cast<uint32_t>(a.chunks);
    uint8_t *const out_row = static_cast<uint8_t *>(a.out) + static_cast<int64_t>(t) * a.ldOut * OB;

    if (task >= passes) {
        // ---- selected features ------------------------------------------------------
        const uint32_t p = (task - passes) * 64u + lane;
        if (bad || p >= static_cast<uint32_t>(a.k)) return;
        const int32_t *idx = reinterpret_cast<const int32_t *>(a.plan + a.off_idx);
        const uint32_t off_outl = t * static_cast<uint32_t>(a.pitch_outl);
        const uint32_t j = static_cast<uint32_t>(idx[p]);
        float acc = 0.f;
        for (uint32_t i0 = 0; i0 < N; i0 += 8) {
            uint32_t v[8];
#pragma unroll
            for (int jj = 0; jj < 8; ++jj)
                v[jj] = reinterpret_cast<const uint16_t *>(
                    static_cast<const uint8_t *>(outlp.p[min(i0 + jj, N - 1u)]) + off_outl)[p];
#pragma unroll
            for (int jj = 0; jj < 8; ++jj) {
                if (i0 + jj < N) {
                    const float x = bf16_bits_to_f32(v[jj]);
                    if (i0 + jj == 0) {
                        acc = x;
                    } else {
                        acc = acc + x;
                        if (ACC == TPQ_ACC_BF16) acc = round_via_bf16(acc);
                    }
                }
            }
        }
        *reinterpret_cast<uint16_t *>(out_row + 2u * j) = static_cast<uint16_t>(pack_bf16x2(acc, acc));
        return;
    }

    // ---- one pass of quantised features ---------------------------------------------
    const uint32_t chunk = task * 64u + lane;
    const uint32_t g = min(chunk / LPG, ng - 1u);
    // the pass's store entries: where they start, blocks, blocks + narrow entries
    const uint4 sp = reinterpret_cast<const uint4 *>(a.plan + a.off_spass)[task];
    const uint32_t first = min(sp.x, static_cast<uint32_t>(a.sblk_cap));
    const uint32_t *entries = reinterpret_cast<const uint32_t *>(a.plan + a.off_sblk) + first;
    const uint32_t nall = min(sp.y + sp.z, static_cast<uint32_t>(a.sblk_cap) - first), nb = min(sp.y, nall);
    const uint32_t e0 = lane < nall ? entries[lane] : 0u;
    const uint32_t e1 = 64u + lane < nall ? entries[64u + lane] : 0u;
    // One 32-bit byte offset per section serves every rank (the host keeps
    // T * pitch below 2^31 per launch): the rank only changes the scalar base.
    const uint32_t off_codes = t * static_cast<uint32_t>(a.pitch_codes) +
                               (GEN ? static_cast<uint32_t>(a.bits) : 4u) * min(chunk, chunks - 1u);
    const uint32_t off_meta = t * static_cast<uint32_t>(a.pitch_meta) + 2u * g;
    float acc[8];
    uint32_t sign = 0u;  // bf16 chain: of the first rank's scale (exact_chain())

    // NB ranks at a time, as in k_decode_pass; FULL: 8, and the compiler may load the next ones ahead of a batch's arithmetic
    // (held back, N = 64, 64 rows takes 12.0 us instead of 10.2)
    auto batch = [&](uint32_t i0, uint32_t left, auto size_tag, auto bits_tag, auto full_tag) __attribute__((always_inline)) {
        constexpr int NB = decltype(size_tag)::value;
        constexpr int BITS = decltype(bits_tag)::value;
        constexpr bool FULL = decltype(full_tag)::value;
        uint32_t w[NB], sb[NB], zb[NB];
        uint64_t wq[NB];  // GEN
        const void *const *pc = codesp.p + i0;
        const void *const *ps = scalep.p + i0;
        const void *const *pz = zerop.p + i0;
        uint32_t oc = off_codes, om = off_meta;
        if constexpr (!FULL) {
            TPQ_LOADS_STAY(NB);
            asm volatile("" : "+v"(oc), "+v"(om));
        }
#pragma unroll
        for (int j = 0; j < NB; ++j) {
            if constexpr (GEN)
                wq[j] = __builtin_nontemporal_load(reinterpret_cast<const u64_a1 *>(
                    static_cast<const uint8_t *>(pc[j]) + oc));
            else
                w[j] = __builtin_nontemporal_load(reinterpret_cast<const uint32_t *>(
                    static_cast<const uint8_t *>(pc[j]) + oc));
            sb[j] = *reinterpret_cast<const uint16_t *>(static_cast<const uint8_t *>(ps[j]) + om);
            zb[j] = *reinterpret_cast<const uint16_t *>(static_cast<const uint8_t *>(pz[j]) + om);
        }
        if constexpr (!FULL) TPQ_LOADS_STAY(NB);
#pragma unroll
        for (int j = 0; j < NB; ++j) {
            if (FULL || j < NB - 1 || left == NB) {  // uniform
                const float sc = bf16_bits_to_f32(sb[j]), ze = bf16_bits_to_f32(zb[j]);
                float x[8];
                if constexpr (GEN) {
                    float c[8];
                    unpack_codes<BITS>(wq[j], c);
#pragma unroll
                    for (int e = 0; e < 8; ++e) x[e] = __builtin_fmaf(c[e], sc, ze);  // product exact
                } else {
                    dequantise8(x, w[j], sc, ze);
                }
                if (ACC == TPQ_ACC_BF16 && FULL && i0 + j == 0) sign = sb[j];
                accumulate8<ACC>(acc, x, FULL && i0 + j == 0);
            }
        }
    };
    auto run = [&](auto bits_tag) __attribute__((always_inline)) {  // (8 ranks or more)
        const std::integral_constant<int, 8> eight;
        uint32_t i0 = 0;
        for (; i0 + 8 <= N; i0 += 8) batch(i0, 8u, eight, bits_tag, std::true_type{});
        const uint32_t left = N - i0;
        if (left > 6u) batch(i0, left, eight, bits_tag, std::false_type{});
        else if (left > 4u) batch(i0, left, std::integral_constant<int, 6>{}, bits_tag, std::false_type{});
        else if (left > 2u) batch(i0, left, std::integral_constant<int, 4>{}, bits_tag, std::false_type{});
        else if (left > 0u) batch(i0, left, std::integral_constant<int, 2>{}, bits_tag, std::false_type{});
    };
    if constexpr (GEN) {
        switch (a.bits) {
        case 2: run(std::integral_constant<int, 2>{}); break;
        case 3: run(std::integral_constant<int, 3>{}); break;
        case 5: run(std::integral_constant<int, 5>{}); break;
        case 6: run(std::integral_constant<int, 6>{}); break;
        default: run(std::integral_constant<int, 8>{}); break;
        }
    } else {
        run(std::integral_constant<int, 4>{});
    }
    if (ACC == TPQ_ACC_BF16 && __builtin_amdgcn_ballot_w64(sign >= 0x8000u))
        exact_chain<GEN>(acc, N, GEN ? static_cast<uint32_t>(a.bits) : 4u, codesp, scalep, zerop, off_codes, off_meta);
    round8<ACC>(acc);
    if (bad) return;
    __shared__ u32x4 stage[4 * 64];
    store_pass<OUT>(stage + wave * 64u, acc, out_row, lane, entries, nb, nall, e0, e1);
}

// ---------------------------------------------------------------------------
// Static symmetric mode (Sec. 3): no scale / zero sections; a feature's value is
// (nibble - 8) * step, the steps of (device, feature) read from a table in compacted
// order (8 per chunk and device: two 128-bit loads that the L2 serves).  Same wave
// roles, loads, accumulation order and stores as k_decode_pass, but a wave takes R
// consecutive rows: the rows share the step loads, which otherwise outnumber the code
// loads two to one.  Rows past the end are read as the last row and not stored.
// grid: (block of R rows, group of 4 waves) pairs, rounded up to a multiple of 8.
// ---------------------------------------------------------------------------
template <int ACC, int OUT, int R, bool GEN>
__global__ __launch_bounds__(256) void k_decode_static(DecodeArgs a, RankPtrs codesp, RankPtrs outlp)
{
    const bool bad = plan_header_bad(a.plan, a.E, a.k, a.G);  // checked before any store
    const uint32_t lane = threadIdx.x & 63u;
    const uint32_t wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const uint32_t passes = static_cast<uint32_t>(a.chunks_padded) >> 6;
    // (row block, wave group) pairs over the XCDs as in k_decode_pass
    const uint32_t ny = (passes + ((static_cast<uint32_t>(a.k) + 63u) >> 6) + 3u) >> 2;
    const uint32_t logical = xcd_contiguous_index(blockIdx.x, gridDim.x);
    const uint32_t rb = logical / ny;
    if (rb * static_cast<uint32_t>(R) >= static_cast<uint32_t>(a.T)) return;  // (grid rounded up to 8)
    const uint32_t task = (logical - rb * ny) * 4u + wave;

    constexpr uint32_t OB = OUT == TPQ_OUT_FP32 ? 4u : 2u;  // bytes per output value
    const uint32_t N = static_cast<uint32_t>(a.n_ranks);
    const uint32_t chunks = static_cast<uint32_t>(a.chunks);
    // the wave's rows; rows past the end are read as the last row and not stored
    const uint32_t t0 = rb * static_cast<uint32_t>(R);
    const uint32_t n_rows = min(static_cast<uint32_t>(R), static_cast<uint32_t>(a.T) - t0);
    uint32_t tr[R];
    uint8_t *out_row[R];
#pragma unroll
    for (int rr = 0; rr < R; ++rr) {
        tr[rr] = t0 + min(static_cast<uint32_t>(rr), n_rows - 1u);
        out_row[rr] = static_cast<uint8_t *>(a.out) + static_cast<int64_t>(tr[rr]) * a.ldOut * OB;
    }

    if (task >= passes) {
        // ---- selected features ------------------------------------------------------
        const uint32_t p = (task - passes) * 64u + lane;
        if (bad || p >= static_cast<uint32_t>(a.k)) return;
        const int32_t *idx = reinterpret_cast<const int32_t *>(a.plan + a.off_idx);
        const uint32_t j = static_cast<uint32_t>(idx[p]);
        float acc[R];
#pragma unroll
        for (int rr = 0; rr < R; ++rr) acc[rr] = 0.f;
        for (uint32_t i0 = 0; i0 < N; i0 += 8) {
            uint32_t v[R][8];
#pragma unroll
            for (int rr = 0; rr < R; ++rr)
#pragma unroll
                for (int jj = 0; jj < 8; ++jj)
                    v[rr][jj] = reinterpret_cast<const uint16_t *>(
                        static_cast<const uint8_t *>(outlp.p[min(i0 + jj, N - 1u)]) +
                        tr[rr] * static_cast<uint32_t>(a.pitch_outl))[p];
#pragma unroll
            for (int rr = 0; rr < R; ++rr)
#pragma unroll
                for (int jj = 0; jj < 8; ++jj) {
                    if (i0 + jj < N) {
                        const float x = bf16_bits_to_f32(v[rr][jj]);
                        if (i0 + jj == 0) {
                            acc[rr] = x;
                        } else {
                            acc[rr] = acc[rr] + x;
                            if (ACC == TPQ_ACC_BF16) acc[rr] = round_via_bf16(acc[rr]);
                        }
                    }
                }
        }
#pragma unroll
        for (int rr = 0; rr < R; ++rr) {
            if (static_cast<uint32_t>(rr) < n_rows) {
                if (OUT == TPQ_OUT_FP32)
                    *reinterpret_cast<float *>(out_row[rr] + 4u * j) = acc[rr];
                else
                    *reinterpret_cast<uint16_t *>(out_row[rr] + 2u * j) =
                        static_cast<uint16_t>(pack_bf16x2(acc[rr], acc[rr]));
            }
        }
        return;
    }

    // ---- one pass of quantised features ---------------------------------------------
    const uint32_t chunk = task * 64u + lane;
    // the pass's store entries: where they start, blocks, blocks + narrow entries
    const uint4 sp = reinterpret_cast<const uint4 *>(a.plan + a.off_spass)[task];
    const uint32_t first = min(sp.x, static_cast<uint32_t>(a.sblk_cap));
    const uint32_t *entries = reinterpret_cast<const uint32_t *>(a.plan + a.off_sblk) + first;
    const uint32_t nall = min(sp.y + sp.z, static_cast<uint32_t>(a.sblk_cap) - first), nb = min(sp.y, nall);
    const uint32_t e0 = lane < nall ? entries[lane] : 0u;
    const uint32_t e1 = 64u + lane < nall ? entries[64u + lane] : 0u;
    // One 32-bit byte offset per section and row serves every rank (the host keeps
    // T * pitch below 2^31 per launch): the rank only changes the scalar base.
    uint32_t off_codes[R];
#pragma unroll
    for (int rr = 0; rr < R; ++rr)
        off_codes[rr] = tr[rr] * static_cast<uint32_t>(a.pitch_codes) +
                        (GEN ? static_cast<uint32_t>(a.bits) : 4u) * min(chunk, chunks - 1u);
    float acc[R][8];

    // static mode, 4 ranks at a time: a code word per row and 8 steps each
    auto batch_static = [&](uint32_t i0, auto full_tag, auto bits_tag) {
        constexpr bool FULL = decltype(full_tag)::value;
        constexpr int BITS = decltype(bits_tag)::value;  // (one copy of the loop per width)
        uint32_t w[R][4];
        uint64_t wq[R][4];  // GEN
        float4 sa[4], sb[4];
        const void *const *pc = codesp.p + i0;
        const float *tab = a.step_c + 8u * chunk;  // chunk < chunks_padded: inside the row
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const uint32_t i = FULL ? static_cast<uint32_t>(j) : min(static_cast<uint32_t>(j), N - 1u - i0);
#pragma unroll
            for (int rr = 0; rr < R; ++rr)
                if constexpr (GEN)
                    wq[rr][j] = __builtin_nontemporal_load(reinterpret_cast<const u64_a1 *>(
                        static_cast<const uint8_t *>(pc[i]) + off_codes[rr]));
                else
                    w[rr][j] = __builtin_nontemporal_load(reinterpret_cast<const uint32_t *>(
                        static_cast<const uint8_t *>(pc[i]) + off_codes[rr]));
            const float *row = tab + static_cast<int64_t>(i0 + i) * a.static_stride;
            sa[j] = *reinterpret_cast<const float4 *>(row);
            sb[j] = *reinterpret_cast<const float4 *>(row + 4);
        }
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            if (FULL || i0 + j < N) {  // uniform
                const float st[8] = {sa[j].x, sa[j].y, sa[j].z, sa[j].w, sb[j].x, sb[j].y, sb[j].z, sb[j].w};
                // (field - 8) * step as one fused multiply-add per value: -8 * step is exact, so
                // field * step - 8 * step is rounded once, from the same exact product; shared
                // by the wave's rows
                float m8[8];
#pragma unroll
                for (int e = 0; e < 8; ++e) m8[e] = -8.0f * st[e];
#pragma unroll
                for (int rr = 0; rr < R; ++rr) {
                    float x[8];
                    if constexpr (GEN) {
                        float c[8];
                        unpack_codes<BITS>(wq[rr][j], c);
                        constexpr float half = static_cast<float>(1u << (BITS - 1));
#pragma unroll
                        for (int e = 0; e < 8; ++e) x[e] = (c[e] - half) * st[e];
                    } else {
                        // fields to floats two at a time (FP8 pair conversion, as in k_decode_pass)
                        const uint32_t lo = w[rr][j] & 0x0F0F0F0Fu, hi = (w[rr][j] >> 4) & 0x0F0F0F0Fu;
                        const f32x2 c02 = __builtin_amdgcn_cvt_scalef32_pk_f32_fp8(lo, 512.0f, false);
                        const f32x2 c46 = __builtin_amdgcn_cvt_scalef32_pk_f32_fp8(lo, 512.0f, true);
                        const f32x2 c13 = __builtin_amdgcn_cvt_scalef32_pk_f32_fp8(hi, 512.0f, false);
                        const f32x2 c57 = __builtin_amdgcn_cvt_scalef32_pk_f32_fp8(hi, 512.0f, true);
                        x[0] = __builtin_fmaf(c02.x, st[0], m8[0]); x[1] = __builtin_fmaf(c13.x, st[1], m8[1]);
                        x[2] = __builtin_fmaf(c02.y, st[2], m8[2]); x[3] = __builtin_fmaf(c13.y, st[3], m8[3]);
                        x[4] = __builtin_fmaf(c46.x, st[4], m8[4]); x[5] = __builtin_fmaf(c57.x, st[5], m8[5]);
                        x[6] = __builtin_fmaf(c46.y, st[6], m8[6]); x[7] = __builtin_fmaf(c57.y, st[7], m8[7]);
                    }
                    accumulate8<ACC, !GEN>(acc[rr], x, i0 + j == 0);  // (GEN: a step of 0 makes -0 of a negative code)
                }
            }
        }
    };
    auto run = [&](auto bits_tag) {
        uint32_t i0 = 0;
        for (; i0 + 4 <= N; i0 += 4) batch_static(i0, std::true_type{}, bits_tag);
        if (i0 < N) batch_static(i0, std::false_type{}, bits_tag);
    };
    if constexpr (GEN) {
        switch (a.bits) {
        case 2: run(std::integral_constant<int, 2>{}); break;
        case 3: run(std::integral_constant<int, 3>{}); break;
        case 5: run(std::integral_constant<int, 5>{}); break;
        case 6: run(std::integral_constant<int, 6>{}); break;
        default: run(std::integral_constant<int, 8>{}); break;
        }
    } else {
        run(std::integral_constant<int, 4>{});
    }
    if (bad) return;
    __shared__ u32x4 stage[4 * 64 * (OUT == TPQ_OUT_FP32 ? 2 : 1)];
#pragma unroll
    for (int rr = 0; rr < R; ++rr) {
        if (static_cast<uint32_t>(rr) >= n_rows) break;  // uniform
        round8<ACC>(acc[rr]);
        store_pass<OUT>(stage + wave * (64u * (OUT == TPQ_OUT_FP32 ? 2u : 1u)), acc[rr], out_row[rr], lane,
                        entries, nb, nall, e0, e1);
    }
}

// ---------------------------------------------------------------------------
// The static mode with many rows and up to kStaticLdsRanks ranks: a workgroup takes one pass of 512 compacted features of 16 rows
// (8 PAIRS), 2 rows of a wave at a time, and holds the pass's steps of all ranks in LDS, so that the table is read from L2 once for 16 rows
// instead of once for 4 and a wave's registers hold codes and sums only (6 waves per SIMD; k_decode_static with 4
// rows has 4, and twice as many waves as fit at once at the size below).  Kernel times, k_decode_static / this, fp32 and bf16 chain: 2048 x 5120, N = 8
// 20.2 / 17.8 us and 21.4 / 21.4; N = 3 13.6 / 12.3; N = 5 18.2 / 14.3 and 18.2 / 16.8; 1300 x 5120, N = 8 21.5 / 13.2 and 21.0 / 16.1;
// 5332 x 4216, N = 2 27.2 / 23.3; 8192 x 8192, N = 8 107 / 95 and 110 / 98.  Where the line lies: 700 x 5120, N = 8 10.5 / 10.0 and 11.1 / 13.0, 600 x 8192 14.6 / 11.0 and
// 15.0 / 13.6, 512 x 5120 8.2 / 8.5; N = 16, bf16 chain 34.5 / 36.5.
// grid: (block of rows, pass or 64 selected features) pairs, rounded up to a multiple of 8.
// ---------------------------------------------------------------------------
constexpr int kStaticLdsRanks = 16;
template <int ACC, int OUT, int PAIRS, bool GEN>
__global__ __launch_bounds__(256, GEN ? 5 : 6) void k_decode_static_lds(DecodeArgs a, RankPtrs codesp, RankPtrs outlp)
{
    const bool bad = plan_header_bad(a.plan, a.E, a.k, a.G);  // checked before any store
    const uint32_t lane = threadIdx.x & 63u;
    const uint32_t wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const uint32_t passes = static_cast<uint32_t>(a.chunks_padded) >> 6;
    const uint32_t tasks = passes + ((static_cast<uint32_t>(a.k) + 63u) >> 6);
    const uint32_t logical = xcd_contiguous_index(blockIdx.x, gridDim.x);
    const uint32_t rb = logical / tasks, task = logical - rb * tasks;
    const uint32_t T = static_cast<uint32_t>(a.T), t0 = rb * (8u * PAIRS);
    if (t0 >= T) return;  // (grid rounded up to 8)

    constexpr uint32_t OB = OUT == TPQ_OUT_FP32 ? 4u : 2u;  // bytes per output value
    const uint32_t N = static_cast<uint32_t>(a.n_ranks);
    const uint32_t row0 = t0 + wave * (2u * PAIRS);  // the wave's first row; rows past the end are read as the last and not stored
    auto out_of = [&](uint32_t t) { return static_cast<uint8_t *>(a.out) + static_cast<int64_t>(t) * a.ldOut * OB; };

    if (task >= passes) {
        // ---- selected features ------------------------------------------------------
        const uint32_t p = (task - passes) * 64u + lane;
        if (bad || p >= static_cast<uint32_t>(a.k)) return;
        const uint32_t j = static_cast<uint32_t>(reinterpret_cast<const int32_t *>(a.plan + a.off_idx)[p]);
#pragma unroll
        for (uint32_t rr = 0; rr < 2u * PAIRS; ++rr) {
            const uint32_t t = row0 + rr;
            if (t >= T) break;  // uniform
            float acc = 0.f;
            for (uint32_t i0 = 0; i0 < N; i0 += 8) {
                uint32_t v[8];
#pragma unroll
                for (int jj = 0; jj < 8; ++jj)
                    v[jj] = reinterpret_cast<const uint16_t *>(static_cast<const uint8_t *>(outlp.p[min(i0 + jj, N - 1u)]) +
                                                               t * static_cast<uint32_t>(a.pitch_outl))[p];
#pragma unroll
                for (int jj = 0; jj < 8; ++jj)
                    if (i0 + jj < N) acc = i0 + jj == 0 ? bf16_bits_to_f32(v[jj]) : add_term<ACC>(acc, bf16_bits_to_f32(v[jj]));
            }
            if (OUT == TPQ_OUT_FP32)
                *reinterpret_cast<float *>(out_of(t) + 4u * j) = acc;
            else
                *reinterpret_cast<uint16_t *>(out_of(t) + 2u * j) = static_cast<uint16_t>(pack_bf16x2(acc, acc));
        }
        return;
    }

    // ---- one pass of quantised features ---------------------------------------------
    const uint32_t chunk = task * 64u + lane;
    extern __shared__ u32x4 smem_static[];
    u32x4 *const table = smem_static;                                                // [rank][first / second four of a chunk][64]
    u32x4 *const stage = smem_static + N * 128u + wave * (64u * (OUT == TPQ_OUT_FP32 ? 2u : 1u));
    for (uint32_t u = threadIdx.x; u < N * 128u; u += 256u) {
        const uint32_t i = u >> 7, q = u & 127u;  // (q < 128: inside the pass, and the table's row has whole passes)
        table[i * 128u + (q & 1u) * 64u + (q >> 1)] =
            *reinterpret_cast<const u32x4 *>(a.step_c + static_cast<int64_t>(i) * a.static_stride + 512u * task + 4u * q);
    }
    // the pass's store entries: where they start, blocks, blocks + narrow entries
    const uint4 sp = reinterpret_cast<const uint4 *>(a.plan + a.off_spass)[task];
    const uint32_t first = min(sp.x, static_cast<uint32_t>(a.sblk_cap));
    const uint32_t *entries = reinterpret_cast<const uint32_t *>(a.plan + a.off_sblk) + first;
    const uint32_t nall = min(sp.y + sp.z, static_cast<uint32_t>(a.sblk_cap) - first), nb = min(sp.y, nall);
    const uint32_t e0 = lane < nall ? entries[lane] : 0u;
    const uint32_t e1 = 64u + lane < nall ? entries[64u + lane] : 0u;
    __syncthreads();

    const uint32_t at = (GEN ? static_cast<uint32_t>(a.bits) : 4u) * min(chunk, static_cast<uint32_t>(a.chunks) - 1u);
#pragma nounroll
    for (uint32_t pr = 0; pr < static_cast<uint32_t>(PAIRS); ++pr) {
        const uint32_t ta = row0 + 2u * pr;
        if (ta >= T) break;  // uniform
        const uint32_t off_a = ta * static_cast<uint32_t>(a.pitch_codes) + at;
        const uint32_t off_b = min(ta + 1u, T - 1u) * static_cast<uint32_t>(a.pitch_codes) + at;
        float acc[2][8];
        // NB ranks at a time, as in k_decode_pass
        auto batch = [&](uint32_t i0, uint32_t left, auto size_tag, auto bits_tag, auto first_tag) __attribute__((always_inline)) {
            constexpr int NB = decltype(size_tag)::value;
            constexpr int BITS = decltype(bits_tag)::value;
            constexpr bool FIRST = decltype(first_tag)::value;
            uint32_t w[2][NB];
            uint64_t wq[2][NB];  // GEN
            const void *const *pc = codesp.p + i0;
            uint32_t oa = off_a, ob = off_b;
            TPQ_LOADS_STAY(NB);
            asm volatile("" : "+v"(oa), "+v"(ob));
#pragma unroll
            for (int j = 0; j < NB; ++j) {
#pragma unroll
                for (int rr = 0; rr < 2; ++rr) {
                    const uint8_t *src = static_cast<const uint8_t *>(pc[j]) + (rr ? ob : oa);
                    if constexpr (GEN)
                        wq[rr][j] = __builtin_nontemporal_load(reinterpret_cast<const u64_a1 *>(src));
                    else
                        w[rr][j] = __builtin_nontemporal_load(reinterpret_cast<const uint32_t *>(src));
                }
                TPQ_LOADS_STAY(NB);
            }
#pragma unroll
            for (int j = 0; j < NB; ++j) {
                if (j < NB - 1 || left == NB) {  // uniform

                    const u32x4 sa = table[(i0 + j) * 128u + lane], sb = table[(i0 + j) * 128u + 64u + lane];
                    const float st[8] = {__uint_as_float(sa.x), __uint_as_float(sa.y), __uint_as_float(sa.z), __uint_as_float(sa.w),
                                         __uint_as_float(sb.x), __uint_as_float(sb.y), __uint_as_float(sb.z), __uint_as_float(sb.w)};
                    // 4 bits: (field - 8) * step as one fused multiply-add per value: 8 * step is exact, so the sum is rounded
                    // once, from the same exact product; shared by the rows.  Other widths: the product itself (a step of
                    // 0 makes -0 of a negative code)
                    float m8[8];
#pragma unroll
                    for (int e = 0; e < 8; ++e) m8[e] = -8.0f * st[e];
#pragma unroll
                    for (int rr = 0; rr < 2; ++rr) {
                        float c[8], x[8];
                        if constexpr (GEN) {
                            unpack_signed<BITS>(wq[rr][j], c);
#pragma unroll
                            for (int e = 0; e < 8; ++e) x[e] = c[e] * st[e];
                        } else {
                            codes8(c, w[rr][j]);
#pragma unroll
                            for (int e = 0; e < 8; ++e) x[e] = __builtin_fmaf(c[e], st[e], m8[e]);
                        }
                        accumulate8<ACC, !GEN>(acc[rr], x, FIRST && j == 0);
                        // (rank by rank: all ranks' steps and terms at once do not fit the registers)
                        asm volatile("" : "+v"(acc[rr][0]), "+v"(acc[rr][1]), "+v"(acc[rr][2]), "+v"(acc[rr][3]), "+v"(acc[rr][4]),
                                     "+v"(acc[rr][5]), "+v"(acc[rr][6]), "+v"(acc[rr][7]) :: "memory");
                    }
                }
            }
        };
        auto some = [&](uint32_t i0, auto bits_tag, auto first_tag) __attribute__((always_inline)) {
            const uint32_t left = N - i0;
            if (left > 6u) batch(i0, left, std::integral_constant<int, 8>{}, bits_tag, first_tag);
            else if (left > 4u) batch(i0, left, std::integral_constant<int, 6>{}, bits_tag, first_tag);
            else if (left > 2u) batch(i0, left, std::integral_constant<int, 4>{}, bits_tag, first_tag);
            else batch(i0, left, std::integral_constant<int, 2>{}, bits_tag, first_tag);
        };
        auto run = [&](auto bits_tag) __attribute__((always_inline)) {
            if (N <= 8u) {
                some(0, bits_tag, std::true_type{});
            } else {
                batch(0, 8u, std::integral_constant<int, 8>{}, bits_tag, std::true_type{});
                some(8, bits_tag, std::false_type{});
            }
        };
        if constexpr (GEN) {
            switch (a.bits) {
            case 2: run(std::integral_constant<int, 2>{}); break;
            case 3: run(std::integral_constant<int, 3>{}); break;
            case 5: run(std::integral_constant<int, 5>{}); break;
            case 6: run(std::integral_constant<int, 6>{}); break;
            default: run(std::integral_constant<int, 8>{}); break;
            }
        } else {
            run(std::integral_constant<int, 4>{});
        }
        if (bad) return;
#pragma unroll
        for (uint32_t rr = 0; rr < 2; ++rr) {
            if (ta + rr >= T) break;  // uniform
            round8<ACC>(acc[rr]);
            uint32_t f0 = e0, f1 = e1;
            asm volatile("" : "+v"(f0), "+v"(f1));  // (what follows from the entries is worked out anew, not kept across the rows)
            store_pass<OUT>(stage, acc[rr], out_of(ta + rr), lane, entries, nb, nall, f0, f1);
        }
    }
}

#ifndef TPQ_STATIC_RPW
#define TPQ_STATIC_RPW 4
#endif
// Rows per wave.  Static mode: 4 once the launch fills the machine (the rows share the
// step table's loads); dynamic mode: 1 (measured: more rows per wave gain nothing there).
static int rows_per_wave(bool is_static, int64_t T, int tasks)
{
    return (is_static && T * tasks >= 2 * 8192) ? TPQ_STATIC_RPW : 1;
}

// How the sums are taken (see the kernels for what each is good at).  Rows need workgroups that are all there at once, or an
// odd number of them per row: consecutive workgroups of an XCD go to its shader engines in turn, so that with 2 or 4 a row the
// last, partly idle one always falls to the same engines (N = 16, 2048 x 2048, k = 32, 2 a row: 16.7 us, as columns 12.2; 2048 x
// 5120, 3 a row: k = 128 25.9 / 26.8; 4 a row: k = 182 33.8 / 28.3; 64 rows of either 4.1 / 4.8).  Codes of 5 bits and more
// bring 8 ranks to the same side (6 bits, 2048 x 5120 26.0 / 27.1, 512 rows 7.6 / 8.7; 5 ranks 24.8 / 23.7).
enum class Decode { kStatic, kStaticLds, kRows, kColumns, kColumnsLanes };
static Decode decode_form(const DecodeArgs &a, int accum, int out_dtype)
{
    if (a.step_c) {
        // (k_decode_static_lds, which says what was measured on either side)
        const int64_t waves = a.T * (a.chunks_padded / 64 + (a.k + 63) / 64);
        const bool bf16 = accum == TPQ_ACC_BF16;
        return a.n_ranks <= (bf16 ? 12 : kStaticLdsRanks) && waves >= (bf16 ? 10000 : 8000) ? Decode::kStaticLds : Decode::kStatic;
    }
    const bool few = 32 * a.k <= a.E;  // (16 selected columns a pass)
    if (a.n_ranks >= (a.bits > 4 ? 8 : 9) && out_dtype == TPQ_OUT_BF16 && !a.addend && !a.bias) {
        const int groups = (a.chunks_padded / 64 + (a.k + 63) / 64 + 3) / 4;
        if (a.T * groups <= 512 || (few && groups % 2 == 1)) return Decode::kRows;
    }
    return a.n_ranks > 8 || !few ? Decode::kColumnsLanes : Decode::kColumns;
}

template <int LPG, int ACC, int OUT, bool LANES>
static void launch_columns(dim3 grid, hipStream_t s, const DecodeArgs &a, const RankPtrs &codes, const RankPtrs &scale,
                           const RankPtrs &zero, const RankPtrs &outl)
{
    if (a.addend || a.bias)  // (4 bits only: the host refuses the epilogue at other widths)
        launch_kernel(k_decode_pass<LPG, ACC, OUT, false, true, LANES>, grid, dim3(256), 0, s, a, codes, scale, zero, outl);
    else if (a.bits != 4)
        launch_kernel(k_decode_pass<LPG, ACC, OUT, true, false, LANES>, grid, dim3(256), 0, s, a, codes, scale, zero, outl);
    else
        launch_kernel(k_decode_pass<LPG, ACC, OUT, false, false, LANES>, grid, dim3(256), 0, s, a, codes, scale, zero, outl);
}

template <int LPG, int ACC, int OUT>
static void launch_rows(Decode form, int rpw, dim3 grid, hipStream_t s, const DecodeArgs &a, const RankPtrs &codes,
                        const RankPtrs &scale, const RankPtrs &zero, const RankPtrs &outl)
{
    if constexpr (LPG == 0) {
        const size_t lds = a.n_ranks * 2048 + 4 * 64 * 16 * (OUT == TPQ_OUT_FP32 ? 2 : 1);
        if (form == Decode::kStaticLds) {
            if (a.bits != 4)
                launch_kernel(k_decode_static_lds<ACC, OUT, 2, true>, grid, dim3(256), lds, s, a, codes, outl);
            else
                launch_kernel(k_decode_static_lds<ACC, OUT, 2, false>, grid, dim3(256), lds, s, a, codes, outl);
        } else if (a.bits != 4) {
            if (rpw == 4)
                launch_kernel(k_decode_static<ACC, OUT, 4, true>, grid, dim3(256), 0, s, a, codes, outl);
            else
                launch_kernel(k_decode_static<ACC, OUT, 1, true>, grid, dim3(256), 0, s, a, codes, outl);
        } else if (rpw == 4) {
            launch_kernel(k_decode_static<ACC, OUT, 4, false>, grid, dim3(256), 0, s, a, codes, outl);
        } else {
            launch_kernel(k_decode_static<ACC, OUT, 1, false>, grid, dim3(256), 0, s, a, codes, outl);
        }
    } else if (form == Decode::kColumns) {
        launch_columns<LPG, ACC, OUT, false>(grid, s, a, codes, scale, zero, outl);
    } else if (form == Decode::kColumnsLanes) {
        launch_columns<LPG, ACC, OUT, true>(grid, s, a, codes, scale, zero, outl);
    } else if constexpr (OUT == TPQ_OUT_BF16) {
        if (a.bits != 4)
            launch_kernel(k_decode_rows<LPG, ACC, true>, grid, dim3(256), 0, s, a, codes, scale, zero, outl);
        else
            launch_kernel(k_decode_rows<LPG, ACC, false>, grid, dim3(256), 0, s, a, codes, scale, zero, outl);
    }
}

int launch_decode(const DecodeArgs &a_in, const RankPtrs &codes_in, const RankPtrs &scale_in,
                  const RankPtrs &zero_in, const RankPtrs &outl_in, int accum, int out_dtype,
                  hipStream_t s)
{
    // TPQ_ACC_FAST is evaluated as the fp32 chain (one final rounding), which is within its tolerance
    if (accum == TPQ_ACC_FAST) accum = TPQ_ACC_FP32;
    const int lpg = a_in.G / 8;
    // waves per row
    const Decode form = decode_form(a_in, accum, out_dtype);
    const bool columns = form == Decode::kColumns || form == Decode::kColumnsLanes;
    const int tasks = !columns ? a_in.chunks_padded / 64 + (a_in.k + 63) / 64 : cpass_cap_of(a_in.E);
    if (tasks == 0) return TPQ_OK;
    // The kernel addresses a rank's sections with 32-bit byte offsets: rows are handed
    // over in blocks whose sections stay below 2 GiB (one block unless T is huge).
    int64_t max_pitch = a_in.pitch_codes;
    if (a_in.pitch_meta > max_pitch) max_pitch = a_in.pitch_meta;
    if (a_in.pitch_outl > max_pitch) max_pitch = a_in.pitch_outl;
    int64_t rows_per_launch = max_pitch > 0 ? (0x7FFFFFFFLL / max_pitch) : a_in.T;
    if (rows_per_launch > 0x7FFFFFFFLL) rows_per_launch = 0x7FFFFFFFLL;
    if (rows_per_launch < 1) return TPQ_ERR_SHAPE;
    const int64_t ny = (tasks + 3) / 4;  // groups of 4 waves per row
    // one-dimensional grid of 256-thread workgroups: grid * block stays below 2^32
    const int64_t max_blocks = (1LL << 24) - 8;
    if (rows_per_launch > max_blocks / ny) rows_per_launch = max_blocks / ny;
    if (columns) {  // the numbers of a launch's waves, those that fill up its grid with them, stay below 2^32 / stride
        const int64_t stride = cpass_stride_of(a_in.E), most = ((1LL << 32) / stride - 64) / stride;
        if (rows_per_launch > most) rows_per_launch = most;
    }
    if (rows_per_launch < 1) return TPQ_ERR_SHAPE;
    const size_t ob = out_dtype == TPQ_OUT_FP32 ? 4 : 2;
    hipError_t e = hipSuccess;
    for (int64_t row0 = 0; row0 < a_in.T && e == hipSuccess; row0 += rows_per_launch) {
        DecodeArgs a = a_in;
        {
            const PlanOffsets o = plan_offsets(a.k, a.r, a.G);
            a.off_idx = o.idx;
            a.off_spass = o.spass;
            a.off_sblk = o.sblk;
            a.sblk_cap = sblk_cap_of(a.k, a.r);
            a.off_src = o.src;
            a.off_cpass = o.cpass;
            a.cpasses = cpass_cap_of(a.E);
            a.cpass_stride = cpass_stride_of(a.E);
            a.cpass_magic = a.cpass_stride > 1 ? static_cast<uint32_t>((1ull << 32) / a.cpass_stride + 1) : 0u;  // unused for 1
        }
        RankPtrs codes = codes_in, scale = scale_in, zero = zero_in, outl = outl_in;
        a.T = a_in.T - row0 < rows_per_launch ? a_in.T - row0 : rows_per_launch;
        a.out = static_cast<uint8_t *>(a_in.out) + row0 * a_in.ldOut * ob;
        if (a_in.addend) a.addend = a_in.addend + row0 * a_in.ldAdd * 2;
        for (int i = 0; i < a_in.n_ranks; ++i) {
            if (codes.p[i]) codes.p[i] = static_cast<const uint8_t *>(codes.p[i]) + row0 * a_in.pitch_codes;
            if (scale.p[i]) scale.p[i] = static_cast<const uint8_t *>(scale.p[i]) + row0 * a_in.pitch_meta;
            if (zero.p[i]) zero.p[i] = static_cast<const uint8_t *>(zero.p[i]) + row0 * a_in.pitch_meta;
            if (outl.p[i]) outl.p[i] = static_cast<const uint8_t *>(outl.p[i]) + row0 * a_in.pitch_outl;
        }
        if (columns && a.k == 0) {  // no section to read from: the codes' first bytes, whatever pitch_outl the caller chose
            outl = codes;
            a.pitch_outl = 0;
        }
        // The kernels read two ranks' pointers at a time, and the selected features' of 8, whether or not they look at what is
        // there: the last rank again, and the first.
        if (a.n_ranks & 1) {  // (the static mode has no scale and zero: null pointers)
            codes.p[a.n_ranks] = codes.p[a.n_ranks - 1];
            scale.p[a.n_ranks] = scale.p[a.n_ranks - 1];
            zero.p[a.n_ranks] = zero.p[a.n_ranks - 1];
        }
        if (columns)
            for (int i = a.n_ranks; i & 7; ++i) outl.p[i] = outl.p[0];
        const int rpw = rows_per_wave(a.step_c != nullptr, a.T, tasks);
        // one dimension, dealt out over the XCDs by the kernel: 4 (row, column pass) pairs a workgroup, else (row block,
        // wave group) pairs
        const int64_t blocks = columns ? (a.T * a.cpass_stride + 3) / 4 : form == Decode::kStaticLds ? (a.T + 15) / 16 * tasks : (a.T + rpw - 1) / rpw * ny;
        const dim3 grid(static_cast<unsigned>((blocks + 7) / 8 * 8));
#define TPQ_LAUNCH3(LPG, ACC, OUT) launch_rows<LPG, ACC, OUT>(form, rpw, grid, s, a, codes, scale, zero, outl)
#define TPQ_LAUNCH2(LPG)                                                                     \
    do {                                                                                     \
        if (accum == TPQ_ACC_FP32 && out_dtype == TPQ_OUT_BF16)                              \
            TPQ_LAUNCH3(LPG, TPQ_ACC_FP32, TPQ_OUT_BF16);                                    \
        else if (accum == TPQ_ACC_FP32)                                                      \
            TPQ_LAUNCH3(LPG, TPQ_ACC_FP32, TPQ_OUT_FP32);                                    \
        else if (out_dtype == TPQ_OUT_BF16)                                                  \
            TPQ_LAUNCH3(LPG, TPQ_ACC_BF16, TPQ_OUT_BF16);                                    \
        else                                                                                 \
            TPQ_LAUNCH3(LPG, TPQ_ACC_BF16, TPQ_OUT_FP32);                                    \
    } while (0)
        switch (a.step_c ? 0 : lpg) {
        case 0: TPQ_LAUNCH2(0); break;  // static symmetric mode
        case 4: TPQ_LAUNCH2(4); break;
        case 8: TPQ_LAUNCH2(8); break;
        case 16: TPQ_LAUNCH2(16); break;
        case 32: TPQ_LAUNCH2(32); break;
        default: return TPQ_ERR_UNSUPPORTED;
        }
#undef TPQ_LAUNCH2
#undef TPQ_LAUNCH3
        e = hipGetLastError();
    }
    return hip_result(e);
}

}  // namespace tpq
