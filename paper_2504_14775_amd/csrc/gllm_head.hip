// First / last pipeline-stage extras (arxiv 2504.14775, section 2.1): embedding layer, projection of the final
// hidden states to logits, sampling strategy.  Contract of every entry point: include/gllm_head.h.
#include "../../include/gllm_head.h"
#include "common.h"

#include <climits>
#include <cmath>
#include <mutex>
#include <string>

namespace {

// ---- embedding: one workgroup per token row, 16-byte pieces -----------------------------------------------
__global__ __launch_bounds__(256) void embedding_kernel(const int32_t* __restrict__ ids, const bf16_t* __restrict__ table,
                                                        bf16_t* __restrict__ out, int hidden, int vocab, int64_t ld_out) {
    const int t = blockIdx.x;
    const int id = ids[t];
    const bool known = id >= 0 && id < vocab;
    const u32x4* src = reinterpret_cast<const u32x4*>(table + (int64_t)(known ? id : 0) * hidden);
    u32x4* dst = reinterpret_cast<u32x4*>(out + (int64_t)t * ld_out);
    if (known) {
        for (int i = threadIdx.x; i < hidden / 8; i += 256) dst[i] = src[i];
    } else {
        for (int i = threadIdx.x; i < hidden / 8; i += 256) dst[i] = u32x4{0u, 0u, 0u, 0u};
    }
}

// ---- final norm of selected rows: h[i] = bf16(x[rows[i]] * rsqrt(mean x^2 + eps) * gain) --------------------
__global__ __launch_bounds__(256) void gather_rmsnorm_kernel(const float* __restrict__ x, int num_x_rows,
                                                             const int32_t* __restrict__ rows,
                                                             const bf16_t* __restrict__ gain, bf16_t* __restrict__ h,
                                                             int hidden, float eps) {
    __shared__ float part[4];
    const int r = min(max(rows[blockIdx.x], 0), num_x_rows - 1);
    const f32x4* src = reinterpret_cast<const f32x4*>(x + (int64_t)r * hidden);
    float ss = 0.f;
    for (int i = threadIdx.x; i < hidden / 4; i += 256) {
        const f32x4 v = src[i];
        ss += v[0] * v[0] + v[1] * v[1] + v[2] * v[2] + v[3] * v[3];
    }
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) ss += __shfl_xor(ss, o);
    if ((threadIdx.x & 63) == 0) part[threadIdx.x >> 6] = ss;
    __syncthreads();
    const float rstd = rsqrtf((part[0] + part[1] + part[2] + part[3]) / (float)hidden + eps);
    bf16_t* dst = h + (int64_t)blockIdx.x * hidden;
    for (int i = threadIdx.x; i < hidden / 4; i += 256) {
        const f32x4 v = src[i];
        const f32x4 g = __builtin_convertvector(*reinterpret_cast<const bf16x4*>(gain + i * 4), f32x4);
        f32x4 y;
#pragma unroll
        for (int e = 0; e < 4; ++e) y[e] = v[e] * rstd * g[e];
        *reinterpret_cast<bf16x4*>(dst + i * 4) = __builtin_convertvector(y, bf16x4);
    }
}

// rows of w [vocab][hidden] -> the GEMM's tiled weight layout with vocab_pad rows, zero rows past vocab
__global__ __launch_bounds__(256) void pad_rows_kernel(const bf16_t* __restrict__ w, bf16_t* __restrict__ out, int vocab,
                                                       int hidden) {
    const int v = blockIdx.x;
    const u32x4* src = reinterpret_cast<const u32x4*>(w + (int64_t)v * hidden);
    for (int i = threadIdx.x; i < hidden / 8; i += 256)
        *reinterpret_cast<u32x4*>(out + w_tiled_index(v, i * 8, hidden)) = v < vocab ? src[i] : u32x4{0u, 0u, 0u, 0u};
}

// ---- sampling: one workgroup per row ----------------------------------------------------------------------
// What bounds it: a row of logits (0.5 MB at a 128k vocabulary) does not fit on chip, so the cost is the number of
// passes over it (6 to 8 us each for a compute unit of its own, 24 us for 256 rows: 5.5 TB/s) and the chains of barriers
// behind them.  One workgroup per row, because a call has one row per sequence and the rows are independent; 64 registers
// per thread and 43 KiB of LDS let two rows share a compute unit, so 257 rows are not two rounds.
//
// The row is read once.  Its first 16384 logits to be read (four blocks from all over it) stay in registers while a
// bound is taken from them, and from there on every logit at or above the bound goes into a list in LDS:
//   top-k     the bound has at least k logits at or above it, so the list holds the k largest;
//   nucleus   the bound is a guess (the list comes to two or three thousand logits) that is checked at the end: the mass of the
//             list must reach top_p of the mass of the row.
// Everything else happens on the list: the k-th largest, the nucleus threshold and the draw are each a weighted radix
// selection ("the largest key above which the weight reaches a value") with 12-bit digits and 64-bit integer weights --
// masses in fixed point -- so the result does not depend on the order the atomics took.
// Where the list overflows or the guess fails, a second pass takes a tighter bound from the maxima of the 1024 threads
// over the whole row; where that fails too (nearly flat distributions, very large k, masses of ties), the selection
// runs over the row, one pass per digit, and the draw takes a pass that sums masses per 4096 consecutive tokens.
// Measured at a vocabulary of 128256 (first: four to ten passes per row, one row per compute unit; then: one pass, a list of 4096 with
// whole keys; now: keys relative to the bound, a list of 5120 of which only the entries in use are walked, a top-k of up to 64
// finished by one wave; us):
//   top-k 50 + nucleus 0.95   1 row 160 -> 27.5 -> 22.0, 64 rows 31.2 -> 25.2, 256 rows 171 -> 42.6 -> 36.7, 257 rows 320 -> 56.0 -> 47.8
//   top-k 300 + nucleus 0.95   1 row 32.1 -> 29.9, 256 rows 60.5 -> 58.1, 257 rows 71.1 -> 68.5 (75.3 with ten more registers spilled)
//   nucleus 0.95 (logits of standard deviation 4.3)   1 row 780 -> 30.5 -> 29.1, 64 rows 880 -> 35.0 -> 33.1, 257 rows 1740 -> 57.0 -> 54.4
//   nucleus 0.95 of nearly flat rows (the selection runs over the row)   64 rows 183
//   greedy   1 row 8.6, 257 rows 33
constexpr int kSampleThreads = 1024;
constexpr int kSampleWaves = kSampleThreads / 64;
constexpr int kDigitBits = 12, kBins = 1 << kDigitBits;
// Candidates held in LDS, then in registers.  A nucleus lists 2450 logits on average and up to 4400 in 256 rows; with room for 4096
// one such row took a second pass and the launch 59 us instead of 37.
constexpr int kList = 5120, kPerThread = kList / kSampleThreads;
static_assert(kBins == 4 * kSampleThreads, "find_bin gives every thread four bins; a block of for_row is one bin of the draw");

// order-preserving map from float to unsigned: a < b  <=>  key(a) < key(b) (for non-NaN values), and back
__device__ __forceinline__ uint32_t float_key(float f) {
    const uint32_t b = __float_as_uint(f);
    return b ^ ((b >> 31) ? 0xFFFFFFFFu : 0x80000000u);
}
__device__ __forceinline__ float key_float(uint32_t k) { return __uint_as_float((k & 0x80000000u) ? k ^ 0x80000000u : ~k); }

// The thread's pieces of blocks first .. first + U - 1, as far as the row reaches.
template <int U>
__device__ __forceinline__ void load_tail(f32x4 (&v)[U], const float* __restrict__ lg, int first, int vocab) {
#pragma unroll
    for (int q = 0; q < U; ++q) {
        const int i = ((first + q) << 12) + 4 * (int)threadIdx.x;
        if (i + 4 <= vocab) v[q] = *reinterpret_cast<const f32x4*>(lg + i);
        else if (i < vocab)
            for (int e = 0; e < 4; ++e) v[q][e] = lg[min(i + e, vocab - 1)];
    }
}

// Calls f(block, index, logit, valid) for the elements of a row that this thread owns, in increasing index order, the
// whole workgroup walking blocks of 4096 consecutive logits (block = index / 4096): 16-byte loads, `U` blocks in flight,
// when the row starts on a 16-byte boundary, single ones otherwise.  block_end(block) follows the four calls of a block.  The
// last blocks are loaded together like the others: one by one they cost a memory latency each.
template <int U, class F, class E>
__device__ __forceinline__ void for_row(const float* __restrict__ lg, int vocab, F&& f, E&& block_end) {
    const int tid = threadIdx.x;
    const int blocks = (vocab + 4095) >> 12, whole = vocab >> 12;
    if ((reinterpret_cast<uintptr_t>(lg) & 15) == 0) {
        int b = 0;
        for (; b + U <= whole; b += U) {
            f32x4 v[U];
#pragma unroll
            for (int q = 0; q < U; ++q) v[q] = *reinterpret_cast<const f32x4*>(lg + ((b + q) << 12) + 4 * tid);
#pragma unroll
            for (int q = 0; q < U; ++q) {
#pragma unroll
                for (int e = 0; e < 4; ++e) f(((b + q) << 12) + 4 * tid + e, v[q][e]);
                block_end(b + q);
            }
        }
        if (b < blocks) {  // at most U: fewer than U whole ones and the one that ends the row
            f32x4 v[U];
            load_tail(v, lg, b, vocab);
#pragma unroll
            for (int q = 0; q < U; ++q) {
                if (b + q >= blocks) continue;
                const int i = ((b + q) << 12) + 4 * tid;
                if (i < vocab) {
#pragma unroll
                    for (int e = 0; e < 4; ++e)
                        if (i + e < vocab) f(i + e, v[q][e]);
                }
                block_end(b + q);
            }
        }
    } else {
        for (int b = 0; b < blocks; ++b) {
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const int i = (b << 12) + 4 * tid + e;
                if (i < vocab) f(i, lg[i]);
            }
            block_end(b);
        }
    }
}

struct SampleShared {
    union {
        uint64_t bins[kBins];       // weights per digit value
        struct {
            float v[kList];         // candidates: logit and token id
            int id[kList];
        } list;
        uint32_t keys[kSampleThreads];
    };
    struct __attribute__((aligned(16))) Few {
        uint32_t key;
        int id;
        uint64_t weight;
    } few[64];                      // what top-k leaves, where that is little; the others weigh nothing
    uint64_t wave_sum[kSampleWaves];
    uint64_t above;
    float wave_f[kSampleWaves];
    int wave_i[kSampleWaves];
    uint32_t digit;
    int count, few_count;
};

// Lane l receives v of lane l - N of its row of 16 (row_shr), or of the last lane of the row(s) before it (row_bcast),
// 0 where there is none: the steps of a scan without a trip through LDS.
template <int CTRL, int ROWS>
__device__ __forceinline__ uint64_t dpp_add(uint64_t v) {
    const uint32_t lo = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)(uint32_t)v, CTRL, ROWS, 0xF, true);
    const uint32_t hi = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)(uint32_t)(v >> 32), CTRL, ROWS, 0xF, true);
    return v + ((uint64_t)hi << 32 | lo);
}
__device__ __forceinline__ uint64_t row_scan(uint64_t v) {  // inclusive, within rows of 16 lanes
    v = dpp_add<0x111, 0xF>(v);
    v = dpp_add<0x112, 0xF>(v);
    v = dpp_add<0x114, 0xF>(v);
    return dpp_add<0x118, 0xF>(v);
}
__device__ __forceinline__ uint64_t wave_scan(uint64_t v) {  // inclusive
    v = row_scan(v);
    v = dpp_add<0x142, 0xA>(v);
    return dpp_add<0x143, 0xC>(v);
}
__device__ __forceinline__ uint64_t lane_value(uint64_t v, int lane) {
    return (uint64_t)(uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)(v >> 32), lane) << 32 |
           (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)v, lane);
}

// Place of a digit value in sh.bins: the four bins a thread sums (see find_bin) lie 1024 apart, so that its and its
// neighbours' reads hit different banks.
__device__ __forceinline__ uint32_t bin_place(uint32_t digit) { return (digit & 3u) * kSampleThreads + (digit >> 2); }

__device__ __forceinline__ void clear_bins(SampleShared& sh) {
    __syncthreads();
#pragma unroll
    for (int j = 0; j < kBins / kSampleThreads; ++j) sh.bins[j * kSampleThreads + threadIdx.x] = 0;
    __syncthreads();
}
__device__ __forceinline__ void add_to_bin(SampleShared& sh, uint32_t digit, uint64_t w) {
    atomicAdd((unsigned long long*)&sh.bins[bin_place(digit)], (unsigned long long)w);
}

// The largest digit d with weight(digits >= d) >= need, and the weight above it; digit 0 when the whole does not reach
// `need`, and a need of 0 counts as 1: whatever the weights, exactly one thread writes the result.  Called when every thread has added its weights; leaves the bins cleared for the next selection.
__device__ __forceinline__ uint32_t find_bin(SampleShared& sh, uint64_t need, uint64_t& above) {
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    need = need > 0 ? need : 1;
    __syncthreads();
    // thread t owns the t-th quadruple of digits counted from the top
    const int quad = kSampleThreads - 1 - tid;
    uint64_t w[4], mine = 0;
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        w[j] = sh.bins[j * kSampleThreads + quad];
        sh.bins[j * kSampleThreads + quad] = 0;
        mine += w[j];
    }
    const uint64_t incl = wave_scan(mine);
    if (lane == 63) sh.wave_sum[wave] = incl;
    __syncthreads();
    const uint64_t waves = row_scan(sh.wave_sum[lane & (kSampleWaves - 1)]);
    const uint64_t all = lane_value(waves, kSampleWaves - 1);
    const bool reached = all >= need;
    uint64_t before = incl - mine + (wave > 0 ? lane_value(waves, wave - 1) : 0);
    // the thread in whose bins the sum passes `need`; the last one (it owns digit 0) if none
    if (reached ? before < need && before + mine >= need : tid == kSampleThreads - 1) {
        int d = 4 * quad + 3;
#pragma unroll
        for (int j = 3; j > 0; --j) {
            const bool on = d == 4 * quad + j && (!reached || before + w[j] < need);
            before += on ? w[j] : 0;
            d -= on ? 1 : 0;
        }
        sh.digit = (uint32_t)d;
        sh.above = before;
    }
    __syncthreads();
    above = sh.above;
    return sh.digit;
}

// The largest key t with weight(entries with key >= t) >= need, over the workgroup's list (entry j of a thread weighs weight(j), 0
// where there is none; the list ends within entries `per` - 1); `bits` (at most 32) is the width of the keys.  The bins must be clear.
template <class W>
__device__ __forceinline__ uint32_t select_key(SampleShared& sh, const uint32_t (&key)[kPerThread], int per, W&& weight, int bits, uint64_t need) {
    uint32_t prefix = 0;
    int low = bits;  // bits below `low` are still open
    while (low > 0) {
        const int step = low < kDigitBits ? low : kDigitBits, shift = low - step;
        const uint32_t digit_mask = (1u << step) - 1u;
#pragma unroll
        for (int j = 0; j < kPerThread; ++j) {
            if (j >= per) break;
            const bool same = low == 32 || (key[j] >> low) == (prefix >> low);
            const uint64_t w = weight(j);
            if (same && w) add_to_bin(sh, (key[j] >> shift) & digit_mask, w);
        }
        uint64_t above;
        const uint32_t d = find_bin(sh, need, above);
        prefix |= d << shift;
        need = need > above ? need - above : 1;
        low = shift;
    }
    return prefix;
}

// A butterfly over the wave without addresses: by __shfl_xor its six lane addresses were kept in registers, or in scratch memory,
// from one to the next.  (The swap of halves gives every lane both its own value and that of lane ^ 32.)
template <int O>
__device__ __forceinline__ float lane_xor(float v) {
    return __int_as_float(__builtin_amdgcn_ds_swizzle(__float_as_int(v), O << 10 | 0x1F));
}
template <class F>
__device__ __forceinline__ float wave_reduce(float v, F&& f) {
    const auto halves = __builtin_amdgcn_permlane32_swap(__float_as_uint(v), __float_as_uint(v), false, false);
    v = f(__uint_as_float(halves[0]), __uint_as_float(halves[1]));
    v = f(v, lane_xor<16>(v));
    v = f(v, lane_xor<8>(v));
    v = f(v, lane_xor<4>(v));
    v = f(v, lane_xor<2>(v));
    return f(v, lane_xor<1>(v));
}
__device__ __forceinline__ int wave_id() { return __builtin_amdgcn_readfirstlane(threadIdx.x >> 6); }
__device__ __forceinline__ float first_lane(float v) { return __uint_as_float(__builtin_amdgcn_readfirstlane(__float_as_uint(v))); }
// Sum over the workgroup with a fixed association (lanes by butterfly, then the wave sums in order).
__device__ __forceinline__ float block_sum(SampleShared& sh, float v) {
    v = wave_reduce(v, [](float a, float b) { return a + b; });
    __syncthreads();
    if ((threadIdx.x & 63) == 0) sh.wave_f[wave_id()] = v;
    __syncthreads();
    float s = 0.f;
#pragma unroll
    for (int w = 0; w < kSampleWaves; ++w) s += sh.wave_f[w];
    return first_lane(s);
}
__device__ __forceinline__ uint64_t block_sum(SampleShared& sh, uint64_t v) {
    v = wave_scan(v);
    __syncthreads();
    if ((threadIdx.x & 63) == 63) sh.wave_sum[wave_id()] = v;
    __syncthreads();
    return lane_value(row_scan(sh.wave_sum[threadIdx.x & (kSampleWaves - 1)]), kSampleWaves - 1);
}

// A lower bound (its low 12 bits are 0) of the k-th largest of N x 64 keys, N per lane, found bit by bit with ballots;
// 0 when there are not k of them.
template <int N>
__device__ __forceinline__ uint32_t wave_kth(const uint32_t (&keys)[N], int k) {
    uint32_t t = 0;
    for (int bit = 31; bit >= 12; --bit) {
        const uint32_t probe = t | (1u << bit);
        int n = 0;
#pragma unroll
        for (int j = 0; j < N; ++j) n += __popcll(__ballot(keys[j] >= probe));
        if (n >= k) t = probe;
        if (n == k) break;  // exactly the k largest: a finer bound gains nothing
    }
    return t;
}
// A value with at least k of the 1024 threads' keys at or above it, 1 <= k <= 1024.  Exact: the k-th largest of all
// (wave 0 searches, 2 us).  Otherwise the lowest of the waves' own (k/16)-th largest: a little lower, a tenth of the time.
template <bool EXACT>
__device__ __forceinline__ uint32_t kth_of_threads(SampleShared& sh, uint32_t key, int k) {
    uint32_t t = 0xFFFFFFFFu;
    __syncthreads();
    if constexpr (EXACT) {
        sh.keys[threadIdx.x] = key;
        __syncthreads();
        if (threadIdx.x < 64) {
            uint32_t mine[kSampleWaves];
#pragma unroll
            for (int j = 0; j < kSampleWaves; ++j) mine[j] = sh.keys[j * 64 + threadIdx.x];
            t = wave_kth(mine, k);
            if (threadIdx.x == 0) sh.wave_i[0] = (int)t;
        }
        __syncthreads();
        t = (uint32_t)sh.wave_i[0];
    } else {
        const uint32_t mine[1] = {key};
        const uint32_t own = wave_kth(mine, (k + kSampleWaves - 1) / kSampleWaves);
        if ((threadIdx.x & 63) == 0) sh.wave_i[wave_id()] = (int)own;
        __syncthreads();
#pragma unroll
        for (int q = 0; q < kSampleWaves; ++q) t = min(t, (uint32_t)sh.wave_i[q]);
    }
    return __builtin_amdgcn_readfirstlane(t);
}
// Largest value of the workgroup.
__device__ __forceinline__ float block_max(SampleShared& sh, float v) {
    v = wave_reduce(v, [](float a, float b) { return fmaxf(a, b); });
    __syncthreads();
    if ((threadIdx.x & 63) == 0) sh.wave_f[wave_id()] = v;
    __syncthreads();
#pragma unroll
    for (int w = 0; w < kSampleWaves; ++w) v = fmaxf(v, sh.wave_f[w]);
    return first_lane(v);
}

// (double)v, made where it stands: hoisted out of the passes over a row the widened constants took scratch memory instead
__device__ __forceinline__ double widened(float v) {
    asm volatile("" : "+s"(v));
    return (double)v;
}
// nucleus: the weight that has to be reached, of `total`
__device__ __forceinline__ uint64_t nucleus_need(float p, uint64_t total) {
    const double need = ceil(widened(p) * (double)total);
    return need >= 1.0 ? (uint64_t)need : 1;
}
// draw: the first token whose running sum exceeds u * total
__device__ __forceinline__ uint64_t draw_need(float u, uint64_t total) {
    const double target = floor((double)u * (double)total);
    const uint64_t need = (target > 0.0 ? (uint64_t)target : 0) + 1;
    return need < total ? need : total;
}

// Greedy: the lowest index among the largest logits.
__device__ __forceinline__ int row_argmax(SampleShared& sh, const float* __restrict__ lg, int vocab) {
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    float best = -INFINITY;
    int best_i = INT_MAX;
    for_row<4>(lg, vocab, [&](int i, float v) {
        if (v > best) {
            best = v;
            best_i = i;
        }
    }, [](int) {});
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) {
        const float ov = __shfl_xor(best, o);
        const int oi = __shfl_xor(best_i, o);
        if (ov > best || (ov == best && oi < best_i)) {
            best = ov;
            best_i = oi;
        }
    }
    if (lane == 0) {
        sh.wave_f[wave] = best;
        sh.wave_i[wave] = best_i;
    }
    __syncthreads();
#pragma unroll
    for (int w = 0; w < kSampleWaves; ++w) {
        const float ov = sh.wave_f[w];
        const int oi = sh.wave_i[w];
        if (ov > best || (ov == best && oi < best_i)) {
            best = ov;
            best_i = oi;
        }
    }
    return best_i == INT_MAX ? 0 : best_i;
}

constexpr int kRoomyMaxRows = 256;   // up to here every row has a compute unit
constexpr int kFirstList = 1400;     // first bound of a nucleus: taken so that the list comes to 1.5 - 2 times this many
constexpr int kMaxFirstK = 256;      // largest k for which the list taken with the first bound is expected to fit
constexpr int kSecondKeys = 960;     // second bound of a nucleus: 960 of the thread maxima of the whole row, about 2800 logits

// ROOMY: a row has a compute unit to itself, so twice the registers, and twice the loads in flight in the pass over the row.
template <bool ROOMY>
__global__ __launch_bounds__(kSampleThreads, ROOMY ? 4 : 8) void sample_kernel(const float* __restrict__ logits, int64_t ld, int vocab,
                                                                   float mass_one, const float* __restrict__ temperature,
                                                                   const int32_t* __restrict__ top_k,
                                                                   const float* __restrict__ top_p,
                                                                   const float* __restrict__ uniform,
                                                                   int32_t* __restrict__ out) {
    __shared__ SampleShared sh;
    constexpr int U = ROOMY ? 8 : 4;
    constexpr int kFewStep = ROOMY ? 8 : 1;  // entries that finish_on_few reads from LDS at one time (with 64 registers four at a time spill 29 more)
    const int tid = threadIdx.x, lane = tid & 63, row = blockIdx.x;
    const float* lg = logits + (int64_t)row * ld;
    const float temp = temperature[row];
    if (!(temp > 0.f)) {
        const int best_i = row_argmax(sh, lg, vocab);
        if (tid == 0) out[row] = best_i;
        return;
    }
    const int k = top_k[row];
    const float p = top_p[row], u = uniform[row];
    const bool by_k = k > 0 && k < vocab, by_p = p < 1.f;
    const float c = 1.4426950408889634f / temp;
    const auto no_end = [](int) {};

    // ---- the pass over the row: maxima of the threads, and, where it is likely to work, the list ----
    const int quarter = vocab >> 14;
    const bool first_list = quarter > 0 && (reinterpret_cast<uintptr_t>(lg) & 15) == 0 && (by_k ? k <= kMaxFirstK : by_p);
    if (tid == 0) sh.count = 0;
    float bound = -INFINITY, ref = 0.f;
    float rest = 0.f;            // mass of the tokens that are not on the list, relative to a token with logit `ref`
    float own_max = -INFINITY;
    auto push = [&](int i, float v) {
        const int slot = atomicAdd(&sh.count, 1);
        if (slot < kList) {
            sh.list.v[slot] = v;
            sh.list.id[slot] = i;
        }
    };
    auto take = [&](int i, float v) {
        own_max = fmaxf(own_max, v);
        const bool in = v >= bound;
        if (in) push(i, v);
        if (!by_k) rest += in ? 0.f : fmaxf(__builtin_amdgcn_exp2f((v - ref) * c), 0.f);
    };
    // a bound on logits from a key: division by the temperature may round smaller logits to the same z (they tie)
    auto bound_of = [&](uint32_t key) {
        const float edge = key_float(key);
        return edge == edge ? edge - fabsf(edge) * 0x1p-20f - temp * 0x1p-148f : -INFINITY;
    };
    if (first_list) {
        f32x4 v[4];
#pragma unroll
        for (int q = 0; q < 4; ++q) v[q] = *reinterpret_cast<const f32x4*>(lg + ((q * quarter) << 12) + 4 * tid);
#pragma unroll
        for (int q = 0; q < 4; ++q)
#pragma unroll
            for (int e = 0; e < 4; ++e) own_max = fmaxf(own_max, v[q][e]);
        bound = bound_of(kth_of_threads<false>(sh, float_key(own_max), by_k ? k : kSampleWaves * min(40, max(4, kFirstList * 1024 / vocab))));
        if (!by_k) ref = block_max(sh, own_max);
        auto load = [&](f32x4 (&to)[4], int i) {
#pragma unroll
            for (int q = 0; q < 4; ++q) to[q] = *reinterpret_cast<const f32x4*>(lg + ((q * quarter + i) << 12) + 4 * tid);
        };
        auto take_all = [&](const f32x4 (&from)[4], int i) {
#pragma unroll
            for (int q = 0; q < 4; ++q)
#pragma unroll
                for (int e = 0; e < 4; ++e) take(((q * quarter + i) << 12) + 4 * tid + e, from[q][e]);
        };
        if constexpr (ROOMY) {
            f32x4 w[4];
            for (int i = 0; i < quarter; i += 2) {
                if (i + 1 < quarter) load(w, i + 1);
                take_all(v, i);
                if (i + 2 < quarter) load(v, i + 2);
                if (i + 1 < quarter) take_all(w, i + 1);
            }
        } else {
            for (int i = 0;;) {
                take_all(v, i);
                if (++i >= quarter) break;
                load(v, i);
            }
        }
        load_tail(v, lg, 4 * quarter, vocab);  // (at most four blocks are left)
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const int i = ((4 * quarter + q) << 12) + 4 * tid;
            if (i >= vocab) continue;
#pragma unroll
            for (int e = 0; e < 4; ++e)
                if (i + e < vocab) take(i + e, v[q][e]);
        }
    } else {
        for_row<U>(lg, vocab, [&](int, float v) { own_max = fmaxf(own_max, v); }, no_end);
    }
    const float best = block_max(sh, own_max);
    // probability of a token relative to the most probable one (0 for a logit that is no number); a mass is that in units
    // of 1 / mass_one
    auto prob = [&](float v) { return fmaxf(__builtin_amdgcn_exp2f((v - best) * c), 0.f); };
    auto mass = [&](float v) { return (uint64_t)(prob(v) * mass_one); };
    // Nothing has mass where the largest logit is infinite (a forced token, a row that is masked as a whole) or the
    // temperature so small that its reciprocal overflows: the row goes to its largest logit.  Past this point the token
    // with logit `best` has mass_one, on the list and on the row.
    if (!(prob(best) > 0.f)) {
        __syncthreads();
        const int best_i = row_argmax(sh, lg, vocab);
        if (tid == 0) out[row] = best_i;
        return;
    }

    // Nucleus and draw among the n <= 64 entries of sh.few, by one wave: an entry compares itself with all others.  (A key is in
    // the nucleus when the keys above it do not reach the mass by themselves; the token drawn is the one in whose interval of the
    // running sum `need` falls.)
    auto finish_on_few = [&](int n) {
        const uint32_t key = lane < n ? sh.few[lane].key : 0;
        const int id = lane < n ? sh.few[lane].id : 0;
        uint64_t weight = lane < n ? sh.few[lane].weight : 0;
        uint64_t total = lane_value(wave_scan(weight), 63);
        if (by_p) {
            uint64_t above = 0;
            for (int i = 0; i < n; i += kFewStep) {
                SampleShared::Few f[kFewStep];
#pragma unroll
                for (int j = 0; j < kFewStep; ++j) f[j] = sh.few[i + j];
#pragma unroll
                for (int j = 0; j < kFewStep; ++j) above += f[j].key > key ? f[j].weight : 0;
            }
            if (above >= nucleus_need(p, total)) weight = 0;
            total = lane_value(wave_scan(weight), 63);
        }
        sh.few[lane].weight = weight;  // read back by other lanes of this wave, which LDS serves in order; the fence keeps
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");  // the compiler from using what it read above (no instruction)
        __builtin_amdgcn_wave_barrier();
        const uint64_t need = draw_need(u, total);
        uint64_t before = 0;
        for (int i = 0; i < n; i += kFewStep) {
            SampleShared::Few f[kFewStep];
#pragma unroll
            for (int j = 0; j < kFewStep; ++j) f[j] = sh.few[i + j];
#pragma unroll
            for (int j = 0; j < kFewStep; ++j) before += f[j].id < id ? f[j].weight : 0;
        }
        if (total == 0 ? lane == 0 : before < need && before + weight >= need) out[row] = total ? id : 0;
    };

    // Finishes the row on the list of n candidates; false when the guess of a nucleus does not hold.
    auto finish_on_list = [&](int n, float others) -> bool {
        // Keys relative to that of the bound, below which nothing is listed: 24 bits, and so two digits instead of three, where
        // the largest logit is less than about four times the bound (wider ranges take the three of whole keys).  Zeros compare
        // equal, so both are listed with a bound that is one, and either may be the largest logit: the range holds the keys of
        // both.  (A bound of -infinity over an infinite temperature is no number.)
        const float z_lo = bound / temp, z_hi = best / temp;
        const uint32_t key_lo = z_lo == 0.f ? float_key(-0.f) : z_lo == z_lo ? float_key(z_lo) : 0u;
        const uint32_t key_span = float_key(z_hi == 0.f ? 0.f : z_hi) - key_lo;
        const int key_bits = 32 - __clz((int)key_span);  // (0 bits: all keys are equal)
        const int per = __builtin_amdgcn_readfirstlane((n + kSampleThreads - 1) / kSampleThreads);  // entries that threads hold
        uint32_t key[kPerThread], ikey[kPerThread];
        uint64_t weight[kPerThread];
        const auto weight_of = [&](int j) { return weight[j]; };
        uint64_t own = 0;
#pragma unroll
        for (int j = 0; j < kPerThread; ++j) {
            const int s = j * kSampleThreads + tid;
            key[j] = ikey[j] = 0;
            weight[j] = 0;
            if (s < n) {
                const float v = sh.list.v[s];
                key[j] = float_key(v / temp) - key_lo;
                ikey[j] = 0xFFFFFFu - (uint32_t)sh.list.id[s];  // larger for tokens that come first
                weight[j] = mass(v);
                own += weight[j];
            }
        }
        clear_bins(sh);
        uint64_t total;
        if (by_k) {
            const uint32_t floor_key =
                select_key(sh, key, per, [&](int j) -> uint64_t { return j * kSampleThreads + tid < n ? 1 : 0; }, key_bits, (uint64_t)k);
            own = 0;
#pragma unroll
            for (int j = 0; j < kPerThread; ++j) {
                if (key[j] < floor_key) weight[j] = 0;
                own += weight[j];
            }
            if (k <= 64) {  // (more than 64 are left where many are equal to the k-th largest)
                if (tid == 0) sh.few_count = 0;
                if (tid < 64) sh.few[tid].weight = 0;
                __syncthreads();
#pragma unroll
                for (int j = 0; j < kPerThread; ++j)
                    if (weight[j]) {
                        const int at = atomicAdd(&sh.few_count, 1);
                        if (at < 64) {
                            sh.few[at].key = key[j];
                            sh.few[at].id = (int)(0xFFFFFFu - ikey[j]);
                            sh.few[at].weight = weight[j];
                        }
                    }
                __syncthreads();
                const int few = sh.few_count;
                if (few <= 64) {
                    if (tid < 64) finish_on_few(few);
                    return true;
                }
            }
            total = block_sum(sh, own);
        } else {
            const uint64_t listed = block_sum(sh, own);
            total = listed + (uint64_t)((double)block_sum(sh, others) * widened(mass_one));
            if (listed < nucleus_need(p, total)) return false;
        }
        if (by_p) {
            const uint32_t t = select_key(sh, key, per, weight_of, key_bits, nucleus_need(p, total));
            own = 0;
#pragma unroll
            for (int j = 0; j < kPerThread; ++j) {
                if (key[j] < t) weight[j] = 0;
                own += weight[j];
            }
            total = block_sum(sh, own);
        }
        const uint32_t first = select_key(sh, ikey, per, weight_of, 24, draw_need(u, total));
        if (tid == 0) out[row] = total ? (int)(0xFFFFFFu - first) : 0;
        return true;
    };

    for (int attempt = first_list ? 0 : 1; attempt < 2; ++attempt) {
        if (attempt == 1) {
            // a second pass, with a bound from the whole row
            if (!(by_k ? k <= kSampleThreads : by_p)) break;
            bound = bound_of(kth_of_threads<true>(sh, float_key(own_max), by_k ? k : kSecondKeys));
            __syncthreads();
            if (tid == 0) sh.count = 0;
            __syncthreads();
            ref = best;
            rest = 0.f;
            for_row<U>(lg, vocab, take, no_end);
            __syncthreads();
        }
        const int n = sh.count;
        if (n <= kList && finish_on_list(n, rest * __builtin_amdgcn_exp2f((ref - best) * c))) return;
    }

    // ---- on the row ----
    // The largest key t >= lo with weight(key(z) >= t) >= need: the interval up to the
    // largest key is cut into up to 4096 bins per pass.  `skip` is a logit below which no key of the interval lies.
    auto select_row = [&](uint32_t lo, float skip, uint64_t need, auto&& weight_of) -> uint32_t {
        uint32_t hi = float_key(best / temp);
        while (lo < hi) {
            const uint32_t span = hi - lo;
            const int bits = 32 - __clz((int)span);
            const int shift = bits > kDigitBits ? bits - kDigitBits : 0;
            for_row<2>(lg, vocab, [&](int, float v) {
                if (v >= skip) {
                    const uint32_t zk = float_key(v / temp);
                    if (zk >= lo && zk <= hi) {
                        const uint64_t w = weight_of(v);
                        if (w) add_to_bin(sh, (zk - lo) >> shift, w);
                    }
                }
            }, no_end);
            uint64_t above;
            const uint32_t d = find_bin(sh, need, above);
            need = need > above ? need - above : 1;
            lo += d << shift;
            hi = min(hi, lo + ((1u << shift) - 1u));
            const float z = key_float(lo) * temp;  // back to a logit, minus what the division may have rounded
            const float s = z - fabsf(z) * 0x1p-20f - temp * 0x1p-148f;
            if (s > skip) skip = s;
        }
        return lo;
    };
    uint32_t floor_key = 0;
    clear_bins(sh);
    if (by_k) floor_key = select_row(0u, -INFINITY, (uint64_t)k, [](float) -> uint64_t { return 1; });
    if (by_p) {
        float own = 0.f;
        if (by_k) for_row<4>(lg, vocab, [&](int, float v) { own += float_key(v / temp) >= floor_key ? prob(v) : 0.f; }, no_end);
        else for_row<4>(lg, vocab, [&](int, float v) { own += prob(v); }, no_end);
        const float row_mass = block_sum(sh, own);
        float skip = -INFINITY;
        if (!by_k) {
            // tokens below `skip` hold less than half of what the nucleus may leave out, even if all of the vocabulary
            // lay there
            const float edge = best + log2f((1.f - p) * row_mass / (2.f * (float)vocab)) / c;
            if (edge == edge) skip = edge - fabsf(edge) * 0x1p-20f;
            if (skip > -INFINITY) floor_key = float_key(skip / temp);
        }
        floor_key = select_row(floor_key, skip, nucleus_need(p, (uint64_t)((double)row_mass * widened(mass_one))), mass);
    }
    // the draw: masses of 4096 consecutive tokens each, then the tokens of the block it falls into
    const bool all = !by_k && !by_p;
    auto kept_mass = [&](float v) -> uint64_t { return all || float_key(v / temp) >= floor_key ? mass(v) : 0; };
    uint64_t in_block = 0, own_total = 0;
    for_row<2>(lg, vocab, [&](int, float v) { in_block += kept_mass(v); }, [&](int b) {
        own_total += in_block;
        in_block = wave_scan(in_block);
        if (lane == 63) add_to_bin(sh, (uint32_t)(kBins - 1 - b), in_block);
        in_block = 0;
    });
    const uint64_t total = block_sum(sh, own_total);
    const uint64_t need = draw_need(u, total);
    uint64_t above;
    const int b = kBins - 1 - (int)find_bin(sh, need, above);
#pragma unroll
    for (int e = 0; e < 4; ++e) {
        const int o = 4 * tid + e, i = (b << 12) + o;
        if (i < vocab) sh.bins[bin_place((uint32_t)(kBins - 1 - o))] = kept_mass(lg[i]);
    }
    uint64_t unused;
    const int o = kBins - 1 - (int)find_bin(sh, need > above ? need - above : 1, unused);
    if (tid == 0) {
        const int i = (b << 12) + o;
        out[row] = total && i < vocab ? i : 0;
    }
}

}  // namespace

struct gllm_head {
    gllm_head_config cfg;
    int32_t vocab_pad = 0;
    bf16_t* w = nullptr;      // [vocab_pad][hidden]
    bf16_t* gain = nullptr;   // [hidden]
    bf16_t* h = nullptr;      // workspace: [round_up(max_rows, 256)][hidden]
    bool loaded = false;
    std::string err;
};

// Scratch of gllm_head_logits_static: the normalised bf16 rows between the two kernels of the projection, for callers
// that can neither allocate nor bind a workspace.  One array per GPU, held until the process ends; its device address
// is looked up once per device (host code must never use the array's name as an address).
constexpr size_t kStaticScratchBytes = (size_t)8 << 20;
static __device__ __align__(256) unsigned char scratch[kStaticScratchBytes];

namespace {
constexpr int kMaxDevices = 64;
std::mutex g_scratch_mutex;
void* g_scratch_ptr[kMaxDevices] = {};

// Device address of `scratch` on the current device (looked up on first use there).
hipError_t static_scratch(void** out) {
    int dev = -1;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return e;
    if (dev < 0 || dev >= kMaxDevices) return hipErrorInvalidDevice;
    std::lock_guard<std::mutex> lock(g_scratch_mutex);
    if (!g_scratch_ptr[dev]) {
        void* p = nullptr;
        e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
        if (e != hipSuccess) return e;
        if (!p) return hipErrorInvalidSymbol;
        g_scratch_ptr[dev] = p;
    }
    *out = g_scratch_ptr[dev];
    return hipSuccess;
}

gllm_status fail(gllm_head* s, gllm_status st, const std::string& msg) {
    if (s) s->err = msg;
    return st;
}
}  // namespace

extern "C" {

gllm_status gllm_op_embedding(const int32_t* ids, const void* table, void* out, int32_t num_tokens, int32_t hidden,
                              int32_t vocab, int64_t ld_out, void* stream) {
    if (!ids || !table || !out || num_tokens < 0 || hidden < 8 || hidden % 8 != 0 || vocab < 1 || ld_out < hidden ||
        ld_out % 8 != 0)
        return GLLM_E_INVALID;
    if (num_tokens == 0) return GLLM_OK;
    embedding_kernel<<<num_tokens, 256, 0, (hipStream_t)stream>>>(ids, (const bf16_t*)table, (bf16_t*)out, hidden, vocab, ld_out);
    return hipGetLastError() == hipSuccess ? GLLM_OK : GLLM_E_HIP;
}

gllm_status gllm_head_create(const gllm_head_config* cfg, gllm_head** out) {
    if (!out) return GLLM_E_INVALID;
    *out = nullptr;
    if (!cfg || cfg->hidden < 64 || cfg->hidden % 64 != 0 || cfg->vocab < 1 || cfg->vocab > (1 << 24) || cfg->max_rows < 1 ||
        !(cfg->rms_eps >= 0.0))
        return GLLM_E_INVALID;
    int n = 0;
    if (hipGetDeviceCount(&n) != hipSuccess || n < 1) return GLLM_E_HIP;
    gllm_head* s = new gllm_head();
    s->cfg = *cfg;
    s->vocab_pad = (int32_t)round_up(cfg->vocab, 256);
    if (hipMalloc((void**)&s->w, (size_t)s->vocab_pad * cfg->hidden * 2) != hipSuccess ||
        hipMalloc((void**)&s->gain, (size_t)cfg->hidden * 2) != hipSuccess) {
        if (s->w) (void)hipFree(s->w);
        delete s;
        return GLLM_E_HIP;
    }
    void* unused = nullptr;
    (void)static_scratch(&unused);  // set-up time: gllm_head_logits_static finds the address ready (it retries if this failed)
    *out = s;
    return GLLM_OK;
}

void gllm_head_destroy(gllm_head* s) {
    if (!s) return;
    (void)hipFree(s->w);
    (void)hipFree(s->gain);
    delete s;
}

const char* gllm_head_last_error(const gllm_head* s) { return s ? s->err.c_str() : "null head"; }

size_t gllm_head_workspace_bytes(const gllm_head* s) {
    return s ? (size_t)round_up(s->cfg.max_rows, 256) * s->cfg.hidden * 2 : 0;
}

gllm_status gllm_head_bind_workspace(gllm_head* s, void* workspace, size_t bytes) {
    if (!s || !workspace) return GLLM_E_INVALID;
    if (bytes < gllm_head_workspace_bytes(s)) return fail(s, GLLM_E_CAPACITY, "workspace too small");
    if ((uintptr_t)workspace % 256 != 0) return fail(s, GLLM_E_INVALID, "workspace must be 256-byte aligned");
    s->h = (bf16_t*)workspace;
    return GLLM_OK;
}

gllm_status gllm_head_load(gllm_head* s, const void* norm_gain, const void* w_vocab, void* stream) {
    if (!s || !norm_gain || !w_vocab) return GLLM_E_INVALID;
    hipStream_t st = (hipStream_t)stream;
    if (hipMemcpyAsync(s->gain, norm_gain, (size_t)s->cfg.hidden * 2, hipMemcpyDeviceToDevice, st) != hipSuccess)
        return fail(s, GLLM_E_HIP, "copy of the norm gain failed");
    pad_rows_kernel<<<s->vocab_pad, 256, 0, st>>>((const bf16_t*)w_vocab, s->w, s->cfg.vocab, s->cfg.hidden);
    if (hipGetLastError() != hipSuccess) return fail(s, GLLM_E_HIP, "weight repack launch failed");
    s->loaded = true;
    return GLLM_OK;
}

int32_t gllm_head_padded_vocab(const gllm_head* s) { return s ? s->vocab_pad : 0; }

// Both projection entry points: rows of x -> normalised bf16 rows in h_buf (num_rows of them) -> logits.
static gllm_status head_logits_into(gllm_head* s, bf16_t* h_buf, const float* x, int32_t num_x_rows, const int32_t* rows,
                                    int32_t num_rows, float* logits, int64_t ld_logits, hipStream_t st) {
    const int H = s->cfg.hidden;
    gather_rmsnorm_kernel<<<num_rows, 256, 0, st>>>(x, num_x_rows, rows, s->gain, h_buf, H, (float)s->cfg.rms_eps);
    if (hipGetLastError() != hipSuccess) return fail(s, GLLM_E_HIP, "norm launch failed");
    const GemmPlan plan = gemm_plan(num_rows, s->vocab_pad, H, GEMM_STORE_F32, 1);
    const hipError_t e = launch_gemm_bf16(h_buf, H, s->w, H, logits, ld_logits, num_rows, s->vocab_pad, H, GEMM_STORE_F32,
                                          plan.tile, 1, 0, st);
    if (e != hipSuccess) return fail(s, GLLM_E_HIP, std::string("projection launch failed: ") + hipGetErrorString(e));
    return GLLM_OK;
}

gllm_status gllm_head_logits(gllm_head* s, const float* x, int32_t num_x_rows, const int32_t* rows, int32_t num_rows,
                             float* logits, int64_t ld_logits, void* stream) {
    if (!s || !x || !rows || !logits || num_x_rows < 1 || num_rows < 0) return GLLM_E_INVALID;
    if (!s->loaded || !s->h) return fail(s, GLLM_E_STATE, "load the weights and bind the workspace first");
    if (num_rows > s->cfg.max_rows) return fail(s, GLLM_E_CAPACITY, "more rows than max_rows");
    if (ld_logits < s->vocab_pad || ld_logits % 4 != 0) return fail(s, GLLM_E_INVALID, "ld_logits must cover the padded vocabulary");
    if (num_rows == 0) return GLLM_OK;
    return head_logits_into(s, s->h, x, num_x_rows, rows, num_rows, logits, ld_logits, (hipStream_t)stream);
}

size_t gllm_head_static_scratch_bytes(void) { return kStaticScratchBytes; }

gllm_status gllm_head_logits_static(gllm_head* s, const float* x, int32_t num_x_rows, const int32_t* rows, int32_t num_rows,
                                    float* logits, int64_t ld_logits, void* stream) {
    if (!s || !x || !rows || !logits || num_x_rows < 1 || num_rows < 0) return GLLM_E_INVALID;
    if (!s->loaded) return fail(s, GLLM_E_STATE, "load the weights first");
    if (ld_logits < s->vocab_pad || ld_logits % 4 != 0) return fail(s, GLLM_E_INVALID, "ld_logits must cover the padded vocabulary");
    // the documented limit counts whole bands of 256 rows (the projection itself reads num_rows rows only)
    const int64_t rows_counted = round_up(num_rows, 256);
    if ((size_t)rows_counted * s->cfg.hidden * 2 > kStaticScratchBytes)
        return fail(s, GLLM_E_CAPACITY, "num_rows (rounded up to bands of 256) x hidden x 2 bytes exceeds the " +
                                            std::to_string(kStaticScratchBytes >> 20) + " MiB static scratch: use gllm_head_logits with a bound workspace");
    if (num_rows == 0) return GLLM_OK;
    void* buf = nullptr;
    const hipError_t e = static_scratch(&buf);
    if (e != hipSuccess) return fail(s, GLLM_E_HIP, std::string("static scratch address: ") + hipGetErrorString(e));
    return head_logits_into(s, (bf16_t*)buf, x, num_x_rows, rows, num_rows, logits, ld_logits, (hipStream_t)stream);
}

gllm_status gllm_op_sample(const float* logits, int64_t ld_logits, int32_t num_rows, int32_t vocab,
                           const float* temperature, const int32_t* top_k, const float* top_p, const float* u,
                           int32_t* out_ids, void* stream) {
    if (!logits || !temperature || !top_k || !top_p || !u || !out_ids || num_rows < 0 || vocab < 1 || vocab > (1 << 24) ||
        ld_logits < vocab)
        return GLLM_E_INVALID;
    if (num_rows == 0) return GLLM_OK;
    // unit of the fixed-point masses: the sum of a whole row stays below 2^63
    int log_vocab = 0;
    while ((1 << log_vocab) < vocab) ++log_vocab;
    auto kernel = num_rows <= kRoomyMaxRows ? sample_kernel<true> : sample_kernel<false>;
    kernel<<<num_rows, kSampleThreads, 0, (hipStream_t)stream>>>(logits, ld_logits, vocab, ldexpf(1.f, 62 - log_vocab), temperature,
                                                                 top_k, top_p, u, out_ids);
    return hipGetLastError() == hipSuccess ? GLLM_OK : GLLM_E_HIP;
}

}  // extern "C"
