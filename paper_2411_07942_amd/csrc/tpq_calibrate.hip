// tpq_calibrate kernels: per-feature min / max of a calibration sequence, the
// moving-average update of Eq. (1), (2), and the final range aggregation and top-k
// selection (paper Sec. 3).
#include <atomic>
#include <mutex>

#include "tpq_device.h"
#include "tpq_internal.h"

namespace tpq {

constexpr int kStripLanes = 64;        // lanes across columns; 8 columns per lane
constexpr int kStripCols = 8 * kStripLanes;
constexpr int kWavesPerBlock = 8;      // waves of a block share columns, split rows
constexpr int kUnroll = 8;             // rows in flight per lane
// Workspace: the partial minima / maxima as [part][0 = min, 1 = max][E] floats.
size_t calibrate_workspace_bytes(int E)
{
    return static_cast<size_t>(kCalMaxParts) * 2u * static_cast<size_t>(E) * sizeof(float);
}

// How many row slices ("parts") a sequence of S rows is cut into.  Each (column strip,
// part) is one workgroup of 8 waves with 8 rows of loads in flight per wave; one such
// workgroup per compute unit reads fastest on this part (measured: two per unit 8 % slower,
// three and four slower still), and nothing is left over for a second round, which a partly
// filled round would make as long as a full one.
int calibrate_parts(int64_t S, int E, int compute_units, int max_parts)
{
    const int strips = (E + kStripCols - 1) / kStripCols;
    int64_t parts = static_cast<int64_t>(compute_units) / strips;
    // at least one row per wave and unrolled step where S allows
    if (parts > S / (kWavesPerBlock * kUnroll)) parts = S / (kWavesPerBlock * kUnroll);
    if (parts > max_parts) parts = max_parts;
    if (parts < 1) parts = 1;
    return static_cast<int>(parts);
}

typedef unsigned int u32x4_cal __attribute__((ext_vector_type(4)));

// Column min / max over one slice of rows.  Lane l of every wave owns columns
// 8*(64*blockIdx.x + l) .. +7 and keeps 8 running minima and maxima in registers;
// the block's waves take interleaved rows, kUnroll 128-bit loads in flight each (one after the other, the
// rows past the last whole step of a slice cost 1.5 to 2.5 us: 450 rows of 16384 features 10.1 -> 7.8 us),
// and are combined through LDS.  The upper bf16 of a word is compared as the whole
// word (it orders like the value itself; the low half is masked off at the end).
// Partials go to `partial` as [part][0 = min, 1 = max][E].
__global__ __launch_bounds__(kStripLanes *kWavesPerBlock) void k_colminmax(
    const uint16_t *__restrict__ Y, int64_t S, int64_t ldY, int E, int rows_per_part,
    float *__restrict__ partial)
{
    const int lane = threadIdx.x & 63;
    const int wave = threadIdx.x >> 6;
    const int col8 = blockIdx.x * kStripLanes + lane;  // which group of 8 columns
    const bool live = col8 * 8 < E;
    const int64_t row0 = static_cast<int64_t>(blockIdx.y) * rows_per_part;
    int64_t row1 = row0 + rows_per_part;
    if (row1 > S) row1 = S;

    float mn[8], mx[8];
#pragma unroll
    for (int e = 0; e < 8; ++e) {
        mn[e] = 3.4028235e38f;   // every finite bf16 value lies inside (-FLT_MAX, FLT_MAX)
        mx[e] = -3.4028235e38f;
    }
    if (live) {
        const u32x4_cal *p = reinterpret_cast<const u32x4_cal *>(Y + col8 * 8);
        const int64_t stride = ldY / 8;  // in 16-byte units
        auto fold = [&](const u32x4_cal &v) {
            const uint32_t w[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const float lo = bf16_lo_to_f32(w[e]);
                const float hi = __uint_as_float(w[e]);
                mn[2 * e] = fminf(mn[2 * e], lo);
                mx[2 * e] = fmaxf(mx[2 * e], lo);
                mn[2 * e + 1] = fminf(mn[2 * e + 1], hi);
                mx[2 * e + 1] = fmaxf(mx[2 * e + 1], hi);
            }
        };
        int64_t t = row0 + wave;
        for (; t + (kUnroll - 1) * kWavesPerBlock < row1; t += kUnroll * kWavesPerBlock) {
            u32x4_cal v[kUnroll];
#pragma unroll
            for (int u = 0; u < kUnroll; ++u)
                v[u] = __builtin_nontemporal_load(p + (t + u * kWavesPerBlock) * stride);
#pragma unroll
            for (int u = 0; u < kUnroll; ++u) fold(v[u]);
        }
        if (t < row1) {  // the rest in one step too (a row past the slice's last is the last one again)
            u32x4_cal v[kUnroll];
#pragma unroll
            for (int u = 0; u < kUnroll; ++u)
                v[u] = __builtin_nontemporal_load(p + min(t + u * kWavesPerBlock, row1 - 1) * stride);
#pragma unroll
            for (int u = 0; u < kUnroll; ++u) fold(v[u]);
        }
#pragma unroll
        for (int e = 1; e < 8; e += 2) {
            mn[e] = __uint_as_float(__float_as_uint(mn[e]) & 0xFFFF0000u);
            mx[e] = __uint_as_float(__float_as_uint(mx[e]) & 0xFFFF0000u);
        }
    }

    __shared__ float red[kWavesPerBlock][2][8][kStripLanes];
#pragma unroll
    for (int e = 0; e < 8; ++e) {
        red[wave][0][e][lane] = mn[e];
        red[wave][1][e][lane] = mx[e];
    }
    __syncthreads();
    // thread (wave, lane): each of the 8 waves finishes one of the 8 features of every
    // lane's column group
    const int j = col8 * 8 + wave;  // this thread's feature
    if (live) {
        float a = red[0][0][wave][lane], b = red[0][1][wave][lane];
#pragma unroll
        for (int w2 = 1; w2 < kWavesPerBlock; ++w2) {
            a = fminf(a, red[w2][0][wave][lane]);
            b = fmaxf(b, red[w2][1][wave][lane]);
        }
        partial[(static_cast<int64_t>(blockIdx.y) * 2 + 0) * E + j] = a;
        partial[(static_cast<int64_t>(blockIdx.y) * 2 + 1) * E + j] = b;
    }
}

// One feature's extreme c of the sequence -> its moving average (Eq. (1), (2)).  old: the state before, which callers load ahead of
// everything, so that it is no second wait for memory at the end
__device__ __forceinline__ float ema_update(float old, float c, int first, float gamma)
{
    c += 0.0f;  // a zero is taken as +0
    if (first) return c;
    const float keep = 1.0f - gamma;
    const float x = keep * old;
    const float y = gamma * c;
    return x + y;
}

// Combine the parts and apply Eq. (1), (2) to one device's state.  A block owns 64 features; its
// kEmaWaves waves take interleaved parts, two at a time with their loads in flight together (so that with 16 waves up to
// 32 parts are one wait for memory, kCalMaxParts four), and are combined through LDS.  Bound by latency: with 4 waves
// that walked over their parts one after the other a 16384 x 4608 chunk took 1.5 us longer (28 parts; four chunks and what
// follows 148 -> 142 us).  Wide rows have few parts and many blocks, and 16 waves a block are then idle ones that are
// launched all the same: up to 8 parts take 4 waves (both launches at E = 32768, 512 rows:
// 10.75 -> 10.5 us).
template <int kEmaWaves>
__global__ __launch_bounds__(64 * kEmaWaves) void k_ema(const float *__restrict__ partial, int parts, int E,
                                                        int first, float gamma, float *__restrict__ m,
                                                        float *__restrict__ M)
{
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int j = blockIdx.x * 64 + lane;
    float *const state = (wave ? M : m) + j;
    float old = 0.0f;
    if (!first && wave <= 1 && j < E) old = *state;
    float cmin = 3.4028235e38f, cmax = -3.4028235e38f;
    if (j < E) {
        for (int p0 = wave; p0 < parts; p0 += 2 * kEmaWaves) {
            // (a part past the last is the last one again)
            const int64_t a = p0, b = min(p0 + kEmaWaves, parts - 1);
            const float lo0 = partial[2 * a * E + j], hi0 = partial[(2 * a + 1) * E + j];
            const float lo1 = partial[2 * b * E + j], hi1 = partial[(2 * b + 1) * E + j];
            cmin = fminf(cmin, fminf(lo0, lo1));
            cmax = fmaxf(cmax, fmaxf(hi0, hi1));
        }
    }
    __shared__ float red[2][kEmaWaves][64];
    red[0][wave][lane] = cmin;
    red[1][wave][lane] = cmax;
    __syncthreads();
    if (wave > 1 || j >= E) return;
    float c = red[wave][0][lane];
#pragma unroll
    for (int w2 = 1; w2 < kEmaWaves; ++w2) c = wave ? fmaxf(c, red[wave][w2][lane]) : fminf(c, red[wave][w2][lane]);
    *state = ema_update(old, c, first, gamma);
}

// Short sequences: both steps in one launch.  A workgroup owns 32 features for all rows, so that
// nothing has to meet in memory: 4 lanes span the features (64 bytes of a row), a wave's load covers 16
// rows, 8 of them in flight per lane.  Minima are kept negated, so that all 64 results of a workgroup are
// maxima: 16 lanes meet by DPP, the rows of lanes through LDS, 8 threads per result.
// Bound by launch and latency, then by what E / 32 compute units can have outstanding; the lines below
// say up to which size that is less than the two launches above.  U: rows in flight per lane, the smallest of 1, 2, 4 and 8 that take the
// sequence in one step (with 8 for 256 rows three loads of four were the last row again); the moving average's state is loaded with the rows, not
// behind them.  256 x 5120: 4.5 -> 4.0 us a launch.
constexpr int kColLanes = 4, kColFeatures = 8 * kColLanes, kColWaves = 8;
template <int U>
__global__ __launch_bounds__(64 * kColWaves) void k_columns(const uint16_t *__restrict__ Y, int S, int64_t ldY,
                                                            int E, int first, float gamma, float *__restrict__ m,
                                                            float *__restrict__ M)
{
    constexpr int kRows = 64 / kColLanes, kStep = kRows * kColWaves;  // rows of a load; of a step of the workgroup
    constexpr int kParts = 4 * kColWaves;                             // rows of 16 lanes
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int col8 = blockIdx.x * kColLanes + (lane & (kColLanes - 1));
    const int v = threadIdx.x / 8, s = threadIdx.x & 7;  // this thread's share of the end: result; slice of the parts
    const bool low = v < kColFeatures;
    const int j = blockIdx.x * kColFeatures + (low ? v : v - kColFeatures);
    float *const state = (low ? m : M) + j;
    float old = 0.0f;
    if (!first && s == 0 && j < E) old = *state;
    float lo[8], hi[8];  // the minima negated
#pragma unroll
    for (int e = 0; e < 8; ++e) lo[e] = hi[e] = -3.4028235e38f;
    if (col8 * 8 < E) {
        const u32x4_cal *p = reinterpret_cast<const u32x4_cal *>(Y + col8 * 8);
        const int64_t stride = ldY / 8;  // in 16-byte units
        for (int t = wave * kRows + lane / kColLanes; t < S; t += U * kStep) {
            u32x4_cal v[U];
#pragma unroll
            for (int u = 0; u < U; ++u)  // (a row past the last is the last one again)
                v[u] = __builtin_nontemporal_load(p + min(t + u * kStep, S - 1) * stride);
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const uint32_t w[4] = {v[u].x, v[u].y, v[u].z, v[u].w};
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    const float x0 = bf16_lo_to_f32(w[e]), x1 = __uint_as_float(w[e]);
                    lo[2 * e] = fmaxf(lo[2 * e], -x0);
                    hi[2 * e] = fmaxf(hi[2 * e], x0);
                    lo[2 * e + 1] = fmaxf(lo[2 * e + 1], -x1);
                    hi[2 * e + 1] = fmaxf(hi[2 * e + 1], x1);
                }
            }
        }
#pragma unroll
        for (int e = 1; e < 8; e += 2) {
            lo[e] = __uint_as_float(__float_as_uint(lo[e]) & 0xFFFF0000u);
            hi[e] = __uint_as_float(__float_as_uint(hi[e]) & 0xFFFF0000u);
        }
    }
#pragma unroll
    for (int e = 0; e < 8; ++e) {  // lanes 4 and 8 on in the row of 16
        lo[e] = fmaxf(lo[e], dpp_f32<0x124>(lo[e]));
        hi[e] = fmaxf(hi[e], dpp_f32<0x124>(hi[e]));
        lo[e] = fmaxf(lo[e], dpp_f32<0x128>(lo[e]));
        hi[e] = fmaxf(hi[e], dpp_f32<0x128>(hi[e]));
    }
    __shared__ float red[kParts][2 * kColFeatures + 1];
    if ((lane & 15) < kColLanes) {
        float *r = red[wave * 4 + lane / 16] + 8 * (lane & (kColLanes - 1));
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            r[e] = lo[e];
            r[kColFeatures + e] = hi[e];
        }
    }
    __syncthreads();
    float c = red[s][v];
#pragma unroll
    for (int i = 8; i < kParts; i += 8) c = fmaxf(c, red[s + i][v]);
    c = fmaxf(c, dpp_f32<0xB1>(c));
    c = fmaxf(c, dpp_f32<0x4E>(c));
    c = fmaxf(c, dpp_f32<0x141>(c));
    if (s == 0 && j < E) *state = ema_update(old, low ? -c : c, first, gamma);
}
static_assert(64 * kColWaves == 8 * 2 * kColFeatures, "eight threads per result");

// Up to how many rows a sequence is short: one launch takes as long as a compute unit needs for its share of the
// columns, so what counts is how many workgroups of 32 features share one.  Measured against the two launches, inputs from
// memory, in us, one / two: E = 5120 (a unit each) 400 rows 4.8 / 6.5, 800 rows 6.7 / 7.1, 900 7.1 / 7.1, 1024 7.7 / 7.2; E = 512
// 900 rows 5.6 / 6.0 to 6.4, 1024 6.0 / 5.8 to 6.3; E = 12288 (two) 300 rows 6.1 / 7.3, 400 7.0 / 7.0, 450 7.4 / 6.9; E = 24576 (three) 150 rows
// 6.2 / 7.4, 192 6.7 / 6.7, 256 7.6 / 7.1; E = 32768 (four) 100 rows 6.3 / 7.2, 150 7.4 / 7.5, 192 8.1 / 7.3, 1024 25.6 / 14.8.
int64_t calibrate_columns_rows(int E, int compute_units)
{
    const int share = ((E + kColFeatures - 1) / kColFeatures + compute_units - 1) / compute_units;
    return share <= 1 ? 1024 : share == 2 ? 400 : 600 / share;
}

// The number of compute units of the current device (looked up once per device: the query is
// slow compared with a launch).
hipError_t compute_units_of_current_device(int *out)
{
    constexpr int kMaxDevices = 64;
    static std::atomic<int> known[kMaxDevices];
    int dev = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return e;
    if (dev >= 0 && dev < kMaxDevices) {
        const int c = known[dev].load(std::memory_order_relaxed);
        if (c > 0) {
            *out = c;
            return hipSuccess;
        }
    }
    int cus = 0;
    e = hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev);
    if (e != hipSuccess) return e;
    if (cus < 1) cus = 1;
    if (dev >= 0 && dev < kMaxDevices) known[dev].store(cus, std::memory_order_relaxed);
    *out = cus;
    return hipSuccess;
}

int launch_colminmax_ema(const uint16_t *Y, int64_t S, int64_t ldY, int E, int first,
                         float gamma, float *m, float *M, void *ws, int max_parts, hipStream_t s)
{
    int cus = 0;
    const hipError_t e0 = compute_units_of_current_device(&cus);
    if (e0 != hipSuccess) return hip_result(e0);
    if (S <= calibrate_columns_rows(E, cus)) {
        constexpr int kStep = 64 / kColLanes * kColWaves;
        const auto kernel = S <= kStep ? k_columns<1> : S <= 2 * kStep ? k_columns<2> : S <= 4 * kStep ? k_columns<4> : k_columns<8>;
        kernel<<<(E + kColFeatures - 1) / kColFeatures, 64 * kColWaves, 0, s>>>(Y, static_cast<int>(S), ldY, E, first, gamma,
                                                                                 m, M);
        return hip_result(hipGetLastError());
    }
    const int parts = calibrate_parts(S, E, cus, max_parts);
    const int rows_per_part = static_cast<int>((S + parts - 1) / parts);
    // the last parts may be empty when S is not a multiple; recompute the live count
    const int live_parts = static_cast<int>((S + rows_per_part - 1) / rows_per_part);
    const dim3 grid((E + kStripCols - 1) / kStripCols, live_parts);
    float *partial = static_cast<float *>(ws);
    k_colminmax<<<grid, kStripLanes * kWavesPerBlock, 0, s>>>(Y, S, ldY, E, rows_per_part, partial);
    if (live_parts <= 8)
        k_ema<4><<<(E + 63) / 64, 64 * 4, 0, s>>>(partial, live_parts, E, first, gamma, m, M);
    else
        k_ema<16><<<(E + 63) / 64, 64 * 16, 0, s>>>(partial, live_parts, E, first, gamma, m, M);
    return hip_result(hipGetLastError());
}

// ---- scratch of tpq_calibrate_fixed ------------------------------------------------
// The partials for callers that cannot bring a workspace: part of the device image, so every
// GPU the library runs on holds its own copy.  Nothing in it has to start at zero: a call
// writes every partial that it reads.  In host code the array's name is only a handle: the
// device address comes from hipGetSymbolAddress, once per device.
static __device__ __align__(256) unsigned char scratch[TPQ_CALIBRATE_FIXED_SCRATCH_BYTES];
static_assert(TPQ_CALIBRATE_FIXED_SCRATCH_BYTES ==
                  static_cast<size_t>(kCalFixedMaxParts) * 2u * TPQ_CALIBRATE_FIXED_MAX_E * sizeof(float),
              "scratch holds kCalFixedMaxParts slices of partials at the largest E");

int calibrate_fixed_scratch(void **ptr)
{
    constexpr int kMaxDevices = 64;
    static std::mutex mu;
    static void *addr[kMaxDevices] = {};
    int dev = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return hip_result(e);
    if (dev < 0 || dev >= kMaxDevices) return TPQ_ERR_UNSUPPORTED;
    std::lock_guard<std::mutex> lock(mu);
    if (!addr[dev]) {
        void *p = nullptr;
        e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
        if (e != hipSuccess) return hip_result(e);
        addr[dev] = p;
    }
    *ptr = addr[dev];
    return TPQ_OK;
}

// ---- finalize -------------------------------------------------------------------

// R = 2*max(-m, M) per device, Rbar = sum over devices in ascending order.  The devices' rows are
// read 8 at a time, so that a thread waits for memory N / 8 times instead of N times.
__global__ __launch_bounds__(256) void k_ranges(const float *__restrict__ m, const float *__restrict__ M, int N,
                                                int E, float *__restrict__ R, float *__restrict__ Rbar)
{
    const int j = blockIdx.x * 256 + threadIdx.x;
    if (j >= E) return;
    float acc = 0.f;
    for (int i0 = 0; i0 < N; i0 += 8) {
        float lo[8], hi[8];
#pragma unroll
        for (int q = 0; q < 8; ++q) {
            const int64_t at = static_cast<int64_t>(min(i0 + q, N - 1)) * E + j;
            lo[q] = -m[at];
            hi[q] = M[at];
        }
#pragma unroll
        for (int q = 0; q < 8; ++q) {
            if (i0 + q < N) {
                float r = 2.0f * (lo[q] > hi[q] ? lo[q] : hi[q]);
                r += 0.0f;
                if (R) R[static_cast<int64_t>(i0 + q) * E + j] = r;
                acc = i0 + q == 0 ? r : acc + r;
            }
        }
    }
    Rbar[j] = acc;
}

// Rank of feature j in the order (Rbar descending, index ascending), by counting the features
// that come before it: a quadratic count without a sort (E <= 32768, once per block of the model).
// A workgroup of 1024 threads owns 16 features and holds all ranges in LDS (in tiles of 8192);
// lane = (feature of the 16, one of 64 interleaved slices of the others), so that E / 16
// workgroups of E / 64 steps cover the chip (320 workgroups at E = 5120) and the counts meet in
// the workgroup.  Bound by instruction issue: two instructions per comparison.  Measured at
// E = 5120: 341 us with one workgroup per 256 features walking over all others (20 workgroups,
// a serial chain of E steps each), 20 us with 256 x 256 tiles that add up through atomics,
// 7 us this way.
constexpr int kRankOwn = 16, kRankTile = 8192;
__global__ __launch_bounds__(1024) void k_rank(const float *__restrict__ Rbar, int E, int k,
                                               int32_t *__restrict__ rank_of, int32_t *__restrict__ idx_ranked)
{
    __shared__ float4 tile[kRankTile / 4];
    __shared__ int32_t part[16][kRankOwn];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int u = wave * 4 + (lane >> 4);  // slice: groups of 4 features u, u + 64, ...
    const int j0 = blockIdx.x * kRankOwn, j = j0 + (lane & 15);
    const float mine = j < E ? Rbar[j] : 0.f;
    int before = 0;
    for (int base = 0; base < E; base += kRankTile) {
        const int n = min(E - base, kRankTile);
        if (base) __syncthreads();
        for (int q = threadIdx.x; q < n; q += 1024) reinterpret_cast<float *>(tile)[q] = Rbar[base + q];
        __syncthreads();
        // the groups below the workgroup's own features (a tie comes before), its own, and the
        // groups above (a tie does not); E is a multiple of 8, so groups are whole
        const int g_n = n / 4, own0 = (j0 - base) / 4;
        const int below = min(max(own0, 0), g_n), above = max(own0 + kRankOwn / 4, 0);
        int g = u;
        for (; g < below; g += 64) {
            const float4 t = tile[g];
            before += (t.x >= mine) + (t.y >= mine) + (t.z >= mine) + (t.w >= mine);
        }
        for (; g < above && g < g_n; g += 64) {
            const float4 t = tile[g];
            const int o = base + 4 * g;
            before += ((t.x > mine) | ((t.x == mine) & (o < j))) + ((t.y > mine) | ((t.y == mine) & (o + 1 < j))) +
                      ((t.z > mine) | ((t.z == mine) & (o + 2 < j))) + ((t.w > mine) | ((t.w == mine) & (o + 3 < j)));
        }
        for (; g < g_n; g += 64) {
            const float4 t = tile[g];
            before += (t.x > mine) + (t.y > mine) + (t.z > mine) + (t.w > mine);
        }
    }
    before += __shfl_xor(before, 16, 64);
    before += __shfl_xor(before, 32, 64);
    if (lane < kRankOwn) part[wave][lane] = before;
    __syncthreads();
    if (threadIdx.x < kRankOwn && j < E) {
        int rank = 0;
#pragma unroll
        for (int w = 0; w < 16; ++w) rank += part[w][lane];
        rank_of[j] = rank;
        if (rank < k) idx_ranked[rank] = j;
    }
}

// Ascending list of the selected features, from their ranks: position = selected features below j.  A workgroup of 1024 features counts
// the selected ones before its own in one sweep over their ranks, all loads in flight at once (it was a serial walk, 256 at a time through
// LDS: 130 us at E = 5120, now 4).
constexpr int kSelectTile = 1024;
__global__ __launch_bounds__(kSelectTile) void k_select(const int32_t *__restrict__ rank_of, int E, int k,
                                                        int32_t *__restrict__ idx_sorted)
{
    __shared__ int32_t wave_sum[2][kSelectTile / 64];  // selected before the tile / in the tile, per wave
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int base = blockIdx.x * kSelectTile;
    const int j = base + threadIdx.x;
    const int rank = j < E ? rank_of[j] : k;
    int earlier = 0;
#pragma unroll 8
    for (int o = threadIdx.x; o < base; o += kSelectTile) earlier += rank_of[o] < k;
#pragma unroll
    for (int d = 32; d > 0; d >>= 1) earlier += __shfl_xor(earlier, d, 64);
    const uint64_t sel = __builtin_amdgcn_ballot_w64(rank < k);
    if (lane == 0) {
        wave_sum[0][wave] = earlier;
        wave_sum[1][wave] = __builtin_popcountll(sel);
    }
    __syncthreads();
    int pos = __builtin_popcountll(sel & ((1ull << lane) - 1ull));
#pragma unroll
    for (int w = 0; w < kSelectTile / 64; ++w) pos += wave_sum[0][w] + (w < wave ? wave_sum[1][w] : 0);
    if (rank < k && pos < k) idx_sorted[pos] = j;  // (ranges that are NaN share ranks: more than k features may have one below k)
}

// Ascending list of the k features with the largest ranges, the lower index first where ranges are equal: the k-th largest
// range by radix selection, then the features above it, and the first ones equal to it, in order.  One workgroup of 1024 threads with
// all ranges in registers (wave w owns the w-th piece of the row, 64 R features, R a thread): a few dozen kilobytes that
// would cost a second launch wherever they meet, and counting every feature's rank over the chip takes E / 64 steps for what is
// three rounds of digits here.  Digits are 11 bits, from the first bit in which the ranges differ; a round counts
// them in LDS, and is the last if all of a digit's features are wanted.  Bound by latency: launch, one load, some ten barriers.
// E = 5120: 6.4 us, against 7.6 for all ranks and 3.9 for the list that follows from them.  R is the smallest of 4, 8, 16 and 32 that holds the row: every round of
// it is paid for (E = 8200 with 32 of them 23 us a call, the ranks' list 18.7).
// Ranges that are NaN come before all others and do not count towards the k; the list ends at k all the same.
constexpr int kTopWaves = 16, kTopDigit = 11, kTopBins = 1 << kTopDigit;
constexpr uint32_t kTopLow = 0x007FFFFFu, kTopHigh = 0xFF800000u;  // keys of -inf and +inf
template <int R>
__global__ __launch_bounds__(64 * kTopWaves) void k_top(const float *__restrict__ Rbar, int E, int k, int32_t *__restrict__ idx_sorted)
{
    __shared__ uint32_t hist[kTopBins];
    __shared__ uint32_t part[2][3][kTopWaves], found[2][3];  // (written anew in every other step only)
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int rounds = (E + 64 * kTopWaves - 1) / (64 * kTopWaves), first = wave * rounds * 64 + lane;  // (rounds <= R)
    hist[2 * threadIdx.x] = hist[2 * threadIdx.x + 1] = 0u;
    // keys in the order of the ranges; 0: no feature, all ones: NaN
    uint32_t key[R], lo = ~0u, hi = 0u, real = 0u;
#pragma unroll
    for (int i = 0; i < R; ++i) key[i] = __float_as_uint(Rbar[min(first + 64 * i, E - 1)]);
#pragma unroll
    for (int i = 0; i < R; ++i) {
        const uint32_t x = key[i] ^ (static_cast<uint32_t>(static_cast<int32_t>(key[i]) >> 31) | 0x80000000u);
        const bool there = i < rounds && first + 64 * i < E, number = there && x >= kTopLow && x <= kTopHigh;
        key[i] = there ? (number ? x : ~0u) : 0u;
        if (number) {
            lo = min(lo, x);
            hi = max(hi, x);
        }
        real += __builtin_popcountll(__builtin_amdgcn_ballot_w64(number));
    }
    lo = ~wave_max(~lo);
    hi = wave_max(hi);
    if (lane == 63) {
        part[0][0][wave] = ~lo;
        part[0][1][wave] = hi;
        part[0][2][wave] = real;
    }
    __syncthreads();
    lo = ~row16_max(part[0][0][lane & 15]);
    hi = row16_max(part[0][1][lane & 15]);
    real = row16_sum(static_cast<int>(part[0][2][lane & 15]));
    // the k-th largest number: `left` bits of it are open, of those that share its other bits `need` are wanted
    uint32_t need = min(static_cast<uint32_t>(k), real), top = hi;
    uint32_t left = real && lo != hi ? 32u - __builtin_clz(lo ^ hi) : 0u;
    bool any = true;  // (the numbers all share the bits above `left`)
    int turn = 1;
    while (left > 0u && need > 0u) {
        const uint32_t digit = min(left, static_cast<uint32_t>(kTopDigit)), shift = left - digit, mask = (1u << digit) - 1u;
#pragma unroll
        for (int i = 0; i < R; ++i) {
            const bool number = key[i] >= kTopLow && key[i] <= kTopHigh;
            if (number && (any || key[i] >> left == top >> left)) atomicAdd(&hist[(key[i] >> shift) & mask], 1u);
        }
        __syncthreads();
        // digits from the largest down, two a thread
        const uint32_t at = kTopBins - 2u - 2u * threadIdx.x, c1 = hist[at + 1u], c0 = hist[at];
        hist[at + 1u] = hist[at] = 0u;
        const uint32_t incl = wave_inclusive_sum(static_cast<int>(c0 + c1));
        if (lane == 63) part[turn][0][wave] = incl;
        __syncthreads();
        const uint32_t others = row16_sum((lane & 15) < wave ? static_cast<int>(part[turn][0][lane & 15]) : 0);
        const uint32_t before = others + incl - c0 - c1;
        if (before < need && before + c0 + c1 >= need) {  // (one thread)
            const bool upper = before + c1 >= need;
            found[turn][0] = at + (upper ? 1u : 0u);
            found[turn][1] = need - before - (upper ? 0u : c1);
            found[turn][2] = upper ? c1 : c0;
        }
        __syncthreads();
        top = (any ? (left < 32u ? hi >> left << left : 0u) : top) | (found[turn][0] << shift);
        any = false;
        need = found[turn][1];
        left = shift;
        turn ^= 1;
        if (found[turn ^ 1][2] == need) break;
    }
    // what lies above, and the first `need` of those that are equal
    const uint32_t bound = real ? top >> left : ~0u - 1u;  // (left < 32: at least one round, or none open)
    uint32_t above = 0u, equal = 0u;
#pragma unroll
    for (int i = 0; i < R; ++i) {
        above += __builtin_popcountll(__builtin_amdgcn_ballot_w64(key[i] >> left > bound));
        equal += __builtin_popcountll(__builtin_amdgcn_ballot_w64(key[i] >> left == bound));
    }
    if (lane == 0) {
        part[turn][1][wave] = above;
        part[turn][2][wave] = equal;
    }
    __syncthreads();
    above = row16_sum((lane & 15) < wave ? static_cast<int>(part[turn][1][lane & 15]) : 0);
    equal = row16_sum((lane & 15) < wave ? static_cast<int>(part[turn][2][lane & 15]) : 0);
    const uint64_t below = (1ull << lane) - 1ull;
#pragma unroll
    for (int i = 0; i < R; ++i) {
        const bool g = key[i] >> left > bound, e = key[i] >> left == bound;
        const uint64_t bg = __builtin_amdgcn_ballot_w64(g), be = __builtin_amdgcn_ballot_w64(e);
        const uint32_t eq = equal + __builtin_popcountll(be & below);
        const uint32_t pos = above + __builtin_popcountll(bg & below) + min(eq, need);
        if ((g || (e && eq < need)) && pos < static_cast<uint32_t>(k)) idx_sorted[pos] = first + 64 * i;
        above += __builtin_popcountll(bg);
        equal += __builtin_popcountll(be);
    }
}
static_assert(kTopBins == 2 * 64 * kTopWaves, "two digits a thread");

int launch_finalize(const float *m, const float *M, int N, int E, int k, float *R, float *Rbar,
                    int32_t *idx_sorted, int32_t *idx_ranked, int32_t *ws, hipStream_t s)
{
    k_ranges<<<(E + 255) / 256, 256, 0, s>>>(m, M, N, E, R, Rbar);
    // Where the ranked list is asked for, every rank is there and the ascending list follows from them in 3.9 us (k_top 6.4): the whole call,
    // E = 5120, 12.1 us against 15.2 with k_top behind the ranks, E = 8200 18.7 against 35.  Without it k_top alone: E = 5120 8.4 us
    // against 12.3, E = 32768 23 against 99.
    if (k > 0 && idx_ranked) {
        k_rank<<<(E + kRankOwn - 1) / kRankOwn, 1024, 0, s>>>(Rbar, E, k, ws, idx_ranked);
        k_select<<<(E + kSelectTile - 1) / kSelectTile, kSelectTile, 0, s>>>(ws, E, k, idx_sorted);
    } else if (k > 0) {
        const auto top = E <= 4096 ? k_top<4> : E <= 8192 ? k_top<8> : E <= 16384 ? k_top<16> : k_top<32>;  // (1024 features a round)
        top<<<1, 64 * kTopWaves, 0, s>>>(Rbar, E, k, idx_sorted);
    }
    return hip_result(hipGetLastError());
}

}  // namespace tpq
