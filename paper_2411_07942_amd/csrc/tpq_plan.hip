// Builds the compaction tables for a static outlier index set (paper Sec. 3: the
// selected features are fixed across sequences and devices, so this runs once
// per block, not per call).
#include "tpq_device.h"
#include "tpq_internal.h"

namespace tpq {

// First column of chunk c's own window: the even column at or below its first feature,
// pulled back so that 8 columns from there stay inside the row.  Chunk 0 starts its
// window at column 0 when selected features precede it and all fits in 16 columns, so
// that its slot can hold them.
__device__ inline int dir_window_a(const uint16_t *src, int c, int E, int r)
{
    const int nv = r - 8 * c < 8 ? r - 8 * c : 8;
    const int c0 = src[8 * c];
    if (c == 0 && c0 > 0 && src[nv - 1] < 16 && E >= 16) return 0;
    const int wa = c0 & ~1;
    return wa < E - 8 ? wa : E - 8;
}

// byte offset of column `col` in the 32 bytes (window a, then window b) of a slot, or -1
__device__ inline int dir_slot_offset(int col, int wa, int E)
{
    int wb = wa + 8;
    if (wb > E - 8) wb = E - 8;
    if (col >= wa && col < wa + 8) return 2 * (col - wa);
    if (col >= wb && col < wb + 8) return 16 + 2 * (col - wb);
    return -1;
}

// does chunk c need a slot?  f: its features (16 bits each), last: the last real one, next0: the next chunk's first, or -1
__device__ inline bool dir_needs_slot(const u32x4 &f, int last, int next0, int c, int E, int r)
{
    const int nv = r - 8 * c < 8 ? r - 8 * c : 8, c0 = f.x & 0xFFFFu;
    const bool contiguous = nv == 8 && last == c0 + 7;
    // selected features inside the chunk, between it and the next one (or the row's
    // end), or before the first chunk: this chunk's slot holds them
    const bool hosts = last - c0 != nv - 1 || (next0 >= 0 ? next0 : E) - last - 1 > 0 || (c == 0 && c0 > 0);
    // where the first feature is odd the 8th is the first half-word of the next lane's window
    const bool next_ok = (c & 63) != 63 && next0 == c0 + 8 && min(next0 & ~1, E - 8) == (c0 & ~1) + 8;
    return !contiguous || hosts || ((c0 & 1) && !next_ok);
}

// The store entries of 64 positions, word w of a pass of n (tables of the decoder's stores), by one wave: `starts` = the
// pass's 512-bit mask of positions that start a run.  lead: a block of 8 starts at the lane's position; single: it is a
// feature of a run shorter than 8; re: where its run ends.
__device__ inline void word_entries(const uint64_t *starts, int w, int n, int lane, bool &lead, bool &single, int &re)
{
    // the last start before the word and the first one behind it: a lane per word of the pass (the second half of each row of 16
    // lanes repeats the first), met by row
    const int i = lane & 7;
    const uint64_t m = starts[i], own = starts[w];
    const int last = static_cast<int>(row16_max(i < w && m ? 64u * i + 63u - __builtin_clzll(m) : 0u));
    const int next = n - static_cast<int>(row16_max(i > w && m ? static_cast<uint32_t>(n - 64 * i - __builtin_ctzll(m)) : 0u));
    const uint64_t upto = lane == 63 ? ~0ull : (2ull << lane) - 1ull;
    const int a0 = 64 * w + lane;
    const int rs = own & upto ? 64 * w + 63 - __builtin_clzll(own & upto) : last;
    re = own & ~upto ? 64 * w + __builtin_ctzll(own & ~upto) : next;
    lead = a0 < n && re - rs >= 8 && ((a0 - rs) & 7) == 0;
    single = a0 < n && re - rs < 8;
}

// The decoder's column passes, by one thread: as many blocks as fit.  (Serial over at most 66 passes, in a
// workgroup of its own beside the others.)
__device__ inline void column_passes(const uint32_t *sel, const uint16_t *sel_before, int E, int k, int cap, uint4 *out)
{
    const int blocks = E / 8;
    // selected columns below column 8 b
    auto before = [&](int b) {
        return b >= blocks ? k : sel_before[b >> 2] + __builtin_popcount(sel[b >> 2] & ((1u << (8 * (b & 3))) - 1u));
    };
    int b0 = 0, s0 = 0;
    for (int p = 0; p < cap; ++p) {
        int n = min(blocks - b0, 64);
        const int w0 = (8 * b0 - s0) / 8;
        int s1 = before(b0 + n);
        if ((8 * (b0 + n) - s1 + 7) / 8 - w0 > 64) s1 = before(b0 + --n);
        const int f0 = 8 * b0 - s0, f1 = 8 * (b0 + n) - s1;  // the pass's features
        const int nw = f1 > f0 ? (f1 + 7) / 8 - w0 : 0;
        out[p] = n > 0 ? make_uint4(static_cast<uint32_t>(b0) | (static_cast<uint32_t>(n) << 16),
                                    static_cast<uint32_t>(w0) | (static_cast<uint32_t>(nw) << 16),
                                    static_cast<uint32_t>(s0) | (static_cast<uint32_t>(s1 - s0) << 16), 0u)
                       : make_uint4(0u, 0u, 0u, 0u);
        b0 += n;
        s0 = s1;
    }
}

// All tables in one launch.  A workgroup builds the encoder's tables of one segment (up to 5 passes), another one its store
// entries, the last one the decoder's column passes; what they need of the rest of the row -- which feature sits where, how
// many slots and store entries come before their own -- they work out themselves in LDS (a few thousand integers; the runs of consecutive
// columns straight from the index list), so that no workgroup waits for another and no table makes a round trip through memory.
// Bound by instruction issue and LDS latency on the compute unit that holds the workgroup, not by bytes.  E = 5120, k = 80: as twelve dependent
// launches, three of them serial walks over the row, it took 165 us; in one launch with the store entries in the same
// workgroups, counted word by word for the whole row, 13.6; now 6.0.
constexpr int kPlanThreads = 1024;
constexpr int kPlanMaxPasses = TPQ_MAX_E / 512, kPlanWords = 8 * 5;  // (a segment has 5 passes at most)
static size_t plan_lds_bytes(int chunks_padded)
{
    // features of the compacted positions
    return static_cast<size_t>(chunks_padded) * 16;
}

__global__ __launch_bounds__(kPlanThreads) void k_plan(uint8_t *plan, const int32_t *__restrict__ idx, int E, int k,
                                                       int G, int r, int chunks, int chunks_padded, int dslots,
                                                       int sblk_cap, PlanOffsets o)
{
    extern __shared__ u32x4 smem_plan[];
    uint16_t *src = reinterpret_cast<uint16_t *>(smem_plan);                       // [8 * chunks_padded]
    __shared__ uint64_t starts[kPlanWords];             // bit of position in the segment: starts a run
    __shared__ uint32_t sel[TPQ_MAX_E / 32];            // bit j: feature j is selected
    __shared__ uint16_t sel_before[TPQ_MAX_E / 32];     // selected features below 32 w
    __shared__ int wave_part[kPlanThreads / 64];
    __shared__ uint64_t flags[kPlanMaxPasses];          // bit of chunk: has a slot
    __shared__ int slots_before[kPlanMaxPasses + 1];
    __shared__ int n_blocks[kPlanMaxPasses], n_narrow[kPlanMaxPasses], entry0[kPlanMaxPasses + 1];
    __shared__ uint32_t word_count[kPlanWords];         // store entries of the segment's words: blocks | narrow ones << 16
    __shared__ int invalid;                             // the index set is not ascending
    __shared__ uint16_t pos16[64][8];                   // the segment's window entries
    __shared__ uint32_t seg_slot[128][2], seg_sel[128]; // its first 128 slots and selected features

    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int passes = chunks_padded / 64, P = dir_passes_of(passes);
    // this workgroup's segment, and whether it builds the decoder's store entries or the encoder's tables
    const int segs = static_cast<int>(gridDim.x) / 2;
    const bool stores = static_cast<int>(blockIdx.x) >= segs;
    const int sg = stores ? blockIdx.x - segs : blockIdx.x, p0 = sg * P, p1 = min(p0 + P, passes);
    const int n_words = 8 * max(p1 - p0, 0);

    // ---- the index set: valid? as a bit mask -------------------------------------------
    // (a thread's first entry and its neighbours are fetched before anything else)
    int v0 = 0, prev0 = -1, next0 = E;
    if (tid < k) {
        v0 = idx[tid];
        if (tid > 0) prev0 = idx[tid - 1];
        if (tid + 1 < k) next0 = idx[tid + 1];
    }
    const int words = (E + 31) / 32;
    for (int w = tid; w < words; w += kPlanThreads) sel[w] = 0u;
    if (tid < 512) pos16[tid >> 3][tid & 7] = 0;
    if (tid < kPlanMaxPasses) n_blocks[tid] = n_narrow[tid] = 0;
    if (tid < n_words) starts[tid] = (tid & 7) == 0 ? 1u : 0u;  // (every pass starts one)
    if (tid == 0) invalid = 0;
    __syncthreads();
    // a run of consecutive columns in the compacted row, [start, end) within one pass, in blocks of 8 or one by one
    auto count_run = [&](int start, int end) {
        const int q = start >> 9, n = min(min(end, r), 512 * (q + 1)) - start;
        if (n >= 8)
            atomicAdd(&n_blocks[q], (n + 7) / 8);
        else
            atomicAdd(&n_narrow[q], n);
    };
    int32_t *pidx = reinterpret_cast<int32_t *>(plan + o.idx);
    auto take = [&](int p, int v, int prev, int next) {
        if (p < k) {
            if (v >= 0 && v < E && v > prev) {
                atomicOr(&sel[v >> 5], 1u << (v & 31));
                // the run behind it, if there is one and it does not start with its pass (those are counted below).
                // (Of an invalid set the counts are not used, but they have to stay in their arrays: 0 < start < r.)
                const int start = v - p, w = (start >> 6) - 8 * p0;
                if (next > v + 1 && start > 0 && start < r && (start & 511)) {
                    count_run(start, max(next - p - 1, start + 1));
                    if (w >= 0 && w < n_words) atomicOr(reinterpret_cast<uint32_t *>(starts + w) + ((start >> 5) & 1), 1u << (start & 31));
                }
            } else {
                v = 0;
                invalid = 1;
            }
        }
        if (blockIdx.x == 0) pidx[p] = p < k ? v : 0;
    };
    const int k4 = (k + 3) / 4 * 4;
    if (tid < k4) take(tid, v0, prev0, next0);
    for (int p = tid + kPlanThreads; p < k4; p += kPlanThreads)
        take(p, idx[min(p, k - 1)], idx[min(p, k) - 1], p + 1 < k ? idx[p + 1] : E);
    __syncthreads();
    const bool bad = invalid != 0;

    // the words of the segment's store entries that this wave takes
    constexpr int kPlanShare = (kPlanWords + kPlanThreads / 64 - 1) / (kPlanThreads / 64);
    bool lead[kPlanShare] = {}, single[kPlanShare] = {};
    int re[kPlanShare] = {};
    if (!bad) {
        // ---- compacted positions -> features -----------------------------------------------
        const int mine = tid < words ? __builtin_popcount(sel[tid]) : 0;  // (TPQ_MAX_E / 32 = one word a thread)
        int before = wave_inclusive_sum(mine) - mine;
        if (lane == 63) wave_part[wave] = before + mine;
        __syncthreads();
        before += row16_sum((lane & 15) < wave ? wave_part[lane & 15] : 0);
        if (tid < words) sel_before[tid] = static_cast<uint16_t>(before);
        __syncthreads();
        if (blockIdx.x == gridDim.x - 1) {
            if (tid == 0) column_passes(sel, sel_before, E, k, cpass_cap_of(E), reinterpret_cast<uint4 *>(plan + o.cpass));
            return;
        }
        for (int j = 8 * tid; j < E; j += 8 * kPlanThreads) {  // 8 features a thread (E is a multiple of 8)
            const uint32_t word = sel[j >> 5], m = word >> (j & 24);
            int c = j - sel_before[j >> 5] - __builtin_popcount(word & ((1u << (j & 24)) - 1u));
#pragma unroll
            for (int e = 0; e < 8; ++e)
                if (!((m >> e) & 1u)) src[c++] = static_cast<uint16_t>(j + e);
        }
        __syncthreads();
        // positions past r repeat the last real one
        for (int c = r + tid; c < 8 * chunks_padded; c += kPlanThreads) src[c] = src[r - 1];
        // the chunks that need a slot
        for (int c = tid; c < chunks_padded && !stores; c += kPlanThreads) {
            const u32x4 f = reinterpret_cast<const u32x4 *>(src)[c];
            const int last = 8 * c + 8 < r ? static_cast<int>(f.w >> 16) : src[r - 1];
            const uint64_t m = __builtin_amdgcn_ballot_w64(
                c < chunks && dir_needs_slot(f, last, 8 * c + 8 < r ? src[8 * c + 8] : -1, c, E, r));
            if (lane == 0) flags[c >> 6] = m;
        }
        // the runs that start with their pass
        if (tid < passes) {
            const int start = 512 * tid, p = src[start] - start;  // (selected columns before it)
            count_run(start, p < k ? idx[p] - p : r);
        }
        __syncthreads();

        // ---- slots and store entries of every pass, and how many come before ---------------
        if (stores) {
#pragma unroll
            for (int u = 0; u < kPlanShare; ++u) {
                const int w = wave + u * (kPlanThreads / 64);
                if (w >= n_words) break;
                word_entries(starts + (w & ~7), w & 7, min(512, r - 512 * (p0 + w / 8)), lane, lead[u], single[u], re[u]);
                const uint64_t bl = __builtin_amdgcn_ballot_w64(lead[u]), bn = __builtin_amdgcn_ballot_w64(single[u]);
                if (lane == 0) word_count[w] = __builtin_popcountll(bl) | (static_cast<uint32_t>(__builtin_popcountll(bn)) << 16);
            }
        }
        if (wave == kPlanThreads / 64 - 1) {
            const int nq = lane < passes && !stores ? __builtin_popcountll(flags[lane]) : 0;
            const int ne = lane < passes ? n_blocks[lane] + n_narrow[lane] : 0;
            const int q = wave_inclusive_sum(nq) - nq, e = wave_inclusive_sum(ne) - ne;
            slots_before[lane] = q;
            entry0[lane] = e;
            if (lane == 63) {
                slots_before[64] = q + nq;
                entry0[64] = e + ne;
            }
        }
        __syncthreads();
    }

    // ---- header ------------------------------------------------------------------------
    if (blockIdx.x == 0 && tid == 0) {
        PlanHeader h = {};
        h.magic = kPlanMagic;
        h.status = bad ? kPlanBadIndex : kPlanOk;
        h.E = E;
        h.k = k;
        h.G = G;
        h.r = r;
        h.chunks = chunks;
        h.chunks_padded = chunks_padded;
        h.idx_offset = o.idx;
        h.src_offset = o.src;
        h.dirr_offset = o.dirr;
        h.dsel_offset = o.dsel;
        h.dslots = dslots;
        h.dslot8_offset = o.dslot8;
        h.dir_P = P;
        h.dseg_offset = o.dseg;
        h.drec_offset = o.drec;
        h.drec2_offset = o.drec2;
        h.spass_offset = o.spass;
        h.sblk_offset = o.sblk;
        h.sblk_cap = sblk_cap;
        h.cpass_offset = o.cpass;
        if (!bad) {
            h.n_dirr = slots_before[64];
            // the bounds of dir_slots_of() and sblk_cap_of() hold for every index set; a plan
            // for which they did not would be refused
            if (slots_before[64] > dslots || entry0[64] > sblk_cap) h.status = kPlanInternal;
        }
        *reinterpret_cast<PlanHeader *>(plan) = h;
    }
    if (bad || p0 >= passes || slots_before[64] > dslots || entry0[64] > sblk_cap) return;

    // ---- this segment's tables -----------------------------------------------------------
    if (stores) {
        {
            uint32_t *dst = reinterpret_cast<uint32_t *>(plan + o.src);
            const uint32_t *s32 = reinterpret_cast<const uint32_t *>(src);
            for (int i = 256 * p0 + tid; i < 256 * p1; i += kPlanThreads) dst[i] = s32[i];
        }
        // store entries
        if (tid < p1 - p0) {
            const int p = p0 + tid;
            reinterpret_cast<uint4 *>(plan + o.spass)[p] = make_uint4(
                static_cast<uint32_t>(entry0[p]), static_cast<uint32_t>(n_blocks[p]), static_cast<uint32_t>(n_narrow[p]), 0u);
        }
#pragma unroll
        for (int u = 0; u < kPlanShare; ++u) {
            const int w = wave + u * (kPlanThreads / 64), p = p0 + w / 8, c0 = 512 * p;
            if (w >= n_words) break;
            const int earlier = row16_sum((lane & 15) < (w & 7) ? static_cast<int>(word_count[(w & ~7) + (lane & 7)]) : 0);
            const uint64_t bl = __builtin_amdgcn_ballot_w64(lead[u]), bn = __builtin_amdgcn_ballot_w64(single[u]), below = (1ull << lane) - 1ull;
            uint32_t *out = reinterpret_cast<uint32_t *>(plan + o.sblk) + entry0[p];
            const int a0 = 64 * (w & 7) + lane;
            if (lead[u]) {
                const int a = a0 + 8 <= re[u] ? a0 : re[u] - 8;
                out[(earlier & 0xFFFF) + __builtin_popcountll(bl & below)] = src[c0 + a] | (static_cast<uint32_t>(a) << 16);
            } else if (single[u]) {
                out[n_blocks[p] + (earlier >> 16) + __builtin_popcountll(bn & below)] = src[c0 + a0] | (static_cast<uint32_t>(a0) << 16);
            }
        }
        return;
    }
    const int q_lo = slots_before[p0], n_q = slots_before[p1] - q_lo;
    const int s_lo = sg == 0 ? 0 : src[512 * p0] - 512 * p0;                      // selected columns below the
    const int s_hi = p1 == passes ? k : src[512 * p1] - 512 * p1;                 // segment's first feature
    // slot number and window of a chunk that has one
    auto slot_of = [&](int c) {
        return slots_before[c >> 6] + __builtin_popcountll(flags[c >> 6] & ((1ull << (c & 63)) - 1ull));
    };
    for (int c = 64 * p0 + tid; c < min(64 * p1, chunks); c += kPlanThreads) {
        const u32x4 f4 = reinterpret_cast<const u32x4 *>(src)[c];
        const uint32_t fw[4] = {f4.x, f4.y, f4.z, f4.w};
        const int p = (c >> 6) - p0, c0 = fw[0] & 0xFFFFu;
        if (!((flags[c >> 6] >> (c & 63)) & 1u)) {
            pos16[c & 63][p] = static_cast<uint16_t>((c0 >> 1) | ((c0 & 1) ? kDir16Odd : 0u));
            continue;
        }
        const int q = slot_of(c);
        const int wa = dir_window_a(src, c, E, r), wb = min(wa + 8, E - 8);
        pos16[c & 63][p] = static_cast<uint16_t>((wa >> 1) | kDir16Slot);
        int at[8];
        bool wide = false;
#pragma unroll
        for (int e = 0; e < 8; ++e) {  // (absent features repeat the last one)
            at[e] = dir_slot_offset((fw[e >> 1] >> (16 * (e & 1))) & 0xFFFFu, wa, E);
            wide |= at[e] < 0;
        }
        uint32_t nib = 0, dw[4];
#pragma unroll
        for (int e = 0; e < 8; ++e)
            if (!wide) nib |= static_cast<uint32_t>(at[e] >> 1) << (4 * e);
#pragma unroll
        for (int w = 0; w < 4; ++w)
            dw[w] = wide ? fw[w] | (kDirWide | (kDirWide << 16)) : static_cast<uint32_t>(at[2 * w]) | (static_cast<uint32_t>(at[2 * w + 1]) << 16);
        reinterpret_cast<u32x4 *>(plan + o.dirr)[q] = u32x4{dw[0], dw[1], dw[2], dw[3]};
        // does the next lane of the pass load exactly the second window?
        bool next_has_b = false;
        if ((c & 63) != 63 && c + 1 < chunks) {
            const bool next_slot = (flags[c >> 6] >> ((c & 63) + 1)) & 1u;
            next_has_b = (next_slot ? dir_window_a(src, c + 1, E, r) : (src[8 * (c + 1)] & ~1)) == wb;
        }
        const uint32_t second = static_cast<uint32_t>(2 * wb) | (wide ? kDirWide8 : 0u) | (next_has_b ? 0u : kDirLoadB8);
        *reinterpret_cast<uint2 *>(plan + o.dslot8 + 8 * q) = make_uint2(nib, second);
        if (q - q_lo < 128) {
            seg_slot[q - q_lo][0] = nib;
            seg_slot[q - q_lo][1] = second;
        }
    }
    // the slot that holds each selected column of the segment: that of the chunk with the feature
    // before it
    for (int p = s_lo + (kPlanThreads - 1 - tid); p < s_hi; p += kPlanThreads) {  // (from the last waves down: the first ones have the chunks)
        const int j = idx[p], f = j - p;  // compacted features before column j
        const int c = f >= 1 ? (f - 1) / 8 : 0;
        uint32_t v = kDirFar;
        if ((flags[c >> 6] >> (c & 63)) & 1u) {
            const int off = dir_slot_offset(j, dir_window_a(src, c, E, r), E);
            if (off >= 0) v = (static_cast<uint32_t>(slot_of(c)) << 5) | static_cast<uint32_t>(off);
        }
        reinterpret_cast<uint32_t *>(plan + o.dsel)[p] = v;
        if (p - s_lo < 128) seg_sel[p - s_lo] = v;
    }
    __syncthreads();
    // the records the encoder's lanes start from
    if (tid == 0)
        *reinterpret_cast<uint2 *>(plan + o.dseg + 8 * sg) =
            make_uint2(static_cast<uint32_t>(q_lo) | (static_cast<uint32_t>(n_q) << 16),
                       static_cast<uint32_t>(s_lo) | (static_cast<uint32_t>(s_hi - s_lo) << 16));
    if (tid < 128) {
        const int n_sel = s_hi - s_lo;
        const uint32_t a0 = tid < n_q ? seg_slot[tid][0] : 0u, a1 = tid < n_q ? seg_slot[tid][1] : 0u;
        const uint32_t sv = tid < n_sel ? seg_sel[tid] : static_cast<uint32_t>(q_lo) << 5;  // idle: the first slot
        if (tid < 64) {
            u32x4 *rec = reinterpret_cast<u32x4 *>(plan + o.drec) + 2 * (64 * sg + tid);
            const uint32_t *pw = reinterpret_cast<const uint32_t *>(pos16[tid]);
            rec[0] = u32x4{pw[0], pw[1], pw[2], pw[3]};
            rec[1] = u32x4{a0, a1, sv, 0u};
        } else {
            reinterpret_cast<u32x4 *>(plan + o.drec2)[64 * sg + lane] = u32x4{a0, a1, sv, 0u};
        }
    }
}

// Static symmetric mode (Sec. 3): per device i and compacted position c (feature j =
// src_of[c]): R = 2*max(-m, M), step = R/(2^bits - 1), inv = 1/step; a vanishing range gives 0, 0.
__global__ void k_static_params(const uint8_t *plan, const float *__restrict__ m,
                                const float *__restrict__ M, int E, int r, int stride, float qmax,
                                float *__restrict__ step, float *__restrict__ inv)
{
    const PlanHeader *h = reinterpret_cast<const PlanHeader *>(plan);
    const uint16_t *src = reinterpret_cast<const uint16_t *>(plan + h->src_offset);
    const int c = blockIdx.x * blockDim.x + threadIdx.x;
    const int i = blockIdx.y;
    if (c >= stride) return;
    float d = 0.0f, v = 0.0f;
    if (h->magic == kPlanMagic && h->status == kPlanOk && c < r) {
        const int j = src[c];
        const float lo = -m[static_cast<int64_t>(i) * E + j], hi = M[static_cast<int64_t>(i) * E + j];
        float R = 2.0f * (lo > hi ? lo : hi);
        R += 0.0f;
        const float q = R / qmax;
        if (q >= 1e-30f) {
            d = q;
            v = 1.0f / q;
        }
    }
    step[static_cast<int64_t>(i) * stride + c] = d;
    inv[static_cast<int64_t>(i) * stride + c] = v;
}

int launch_static_params(const tpq_layout *L, const void *plan, const float *m, const float *M,
                         int n_ranks, float *step, float *inv, hipStream_t s)
{
    const int stride = 8 * chunks_padded_of(L->r);
    if (stride == 0) return TPQ_OK;
    const dim3 grid((stride + 255) / 256, n_ranks);
    k_static_params<<<grid, 256, 0, s>>>(static_cast<const uint8_t *>(plan), m, M, L->E, L->r, stride,
                                        static_cast<float>((1 << L->bits) - 1), step, inv);
    return hip_result(hipGetLastError());
}

int launch_plan_build(const tpq_layout *L, const int32_t *idx, void *plan, hipStream_t s)
{
    const int cp = chunks_padded_of(L->r);
    const size_t lds = plan_lds_bytes(cp);
    if (lds > 49152) {  // (with the static tables past the default limit of 64 KiB)
        const hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void *>(&k_plan),
                                                 hipFuncAttributeMaxDynamicSharedMemorySize, static_cast<int>(lds));
        if (e != hipSuccess) return hip_result(e);
    }
    const int segs = dir_segs_of(cp / 64);
    k_plan<<<2 * (segs > 0 ? segs : 1) + 1, kPlanThreads, lds, s>>>(
        static_cast<uint8_t *>(plan), idx, L->E, L->k, L->G, L->r, chunks_of(L->r), cp, dir_slots_of(L->k, L->r),
        sblk_cap_of(L->k, L->r), plan_offsets(L->k, L->r, L->G));
    return hip_result(hipGetLastError());
}

}  // namespace tpq
