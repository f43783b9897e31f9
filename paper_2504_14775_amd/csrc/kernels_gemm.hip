// bf16 x bf16 -> fp32 GEMM on the CDNA4 matrix cores:  out[m][n] (op)= sum_k a[m][k] * w[n][k].
//
// Both operands are contiguous along k, which is the order the MFMA operand registers want
// (each lane feeds 8 consecutive k of one row), so tiles go global -> LDS -> registers without
// any transposition.  A workgroup of WGM x WGN wavefronts owns a BM x BN output tile and walks k
// in steps of 64 through two to four LDS stages, filled by buffer loads that write 16 bytes per lane straight
// into LDS (no staging registers, no address arithmetic: the k position is the scalar offset).
//
// What bounds it: many rows, the 1400 W power limit (a bare MFMA loop on random operands reaches 1.6-1.8 PFLOP/s); few
// rows, the stream of the weights (5.5-6.8 TB/s) and the ~5 us a launch costs before and after it; in between what a compute unit
// loads: a k-step's weights from HBM and activations from the L2 take nearly as long as one after the other, 66 KB/us of both together
// where activations alone come at 120 (profiles/gemm_loads_of_a_k_step.txt), so that a result of a narrow tile costs more.  Under
// the power limit the clock follows the busy share of the matrix cores, so cycles in the k-loop count in full, and so does
// the energy of a product.  16x16x32 MFMAs touch an accumulator half as often per product as 32x32x16 ones: the same tile at
// the same order of loads took 99.3 -> 90.6 us for gate/up at 512 rows (28672 x 4096), 859 -> 833 at 2048 rows of 55296 x
// 5120, 387 -> 378 at 4096x8192x8192 (1455 TFLOP/s); where the weights' stream bounds a product there is no difference (64
// rows).  Four waves with a wave tile of 128x128 read LDS two thirds as often per MFMA as eight of 128x64, and the order of
// MFMAs, LDS reads and global loads is written out (see step): over whole launches of 256x256 tiles the matrix cores are busy
// for 0.67 to 0.74 of the time at 1.8 to 2.0 GHz (profiles/stage_*_mfma_counters.txt; a bare MFMA loop 1.0 at 1.68).  Where
// tiles fill a part of the chip, power is no limit and the smaller MFMAs cost up to 5 % (5184 x 4096, 257 rows 56.4 -> 59.2).
//
// LDS stage layout: rows of 64 k-values (128 bytes = eight 16-byte groups), A rows first, then W
// rows.  Two consecutive rows form a 256-byte line of 16 group positions (the width of the 64 LDS
// banks); group c of row r sits at position ((r & 1) * 8 + c) ^ ((r >> 1) & 7) of line r >> 1.  The
// 16-byte operand reads of the MFMA loop take, per 16 lanes, one group index of 16 consecutive rows:
// with this placement those 16 reads fall into 16 different bank groups (measured: the plain
// c ^ (r & 7) placement costs a 2-way bank conflict on every read).  A load instruction
// fills 1 KiB = 4 lines: lane l owns position l % 16 of line l / 16 and fetches the global group that
// belongs there; the 16 lanes of a line still cover the full 128 bytes of both of its rows.
//
// Workgroup -> tile mapping: hardware hands consecutive workgroup ids to the 8 XCDs in turn, each
// with its own L2.  Ids are first regrouped so that an XCD receives a contiguous range of tile
// numbers; tiles are numbered band by band (a band is 8 tile-columns wide, walked row by row), so
// the tiles an XCD works on at one time share a few A row-panels and W row-panels in its L2.
#include "common.h"

#include <algorithm>
#include <cmath>

namespace {

constexpr int BK = 64;
[[maybe_unused]] constexpr int MB = 16, MK = 32;  // v_mfma_f32_16x16x32_bf16: a block of 16x16 results over 32 k values
constexpr int kMaxTileM = 384;            // tallest tile

// silu(z) = z / (1 + e^-z) with the hardware exp2 and reciprocal (1 ulp each; the result is rounded to bf16)
__device__ __forceinline__ float silu(float z) {
    return z * __builtin_amdgcn_rcpf(1.0f + __builtin_amdgcn_exp2f(-1.4426950408889634f * z));
}

typedef __attribute__((address_space(3))) void* lptr_t;

// Hardware hands consecutive workgroup ids to the 8 XCDs in turn; this turns id `wg` of `count` into a work number such
// that every XCD receives one contiguous range of work numbers (XCD x gets workgroups x, x+8, ...: count / 8 of them,
// one more for x < count % 8).
__device__ __forceinline__ int xcd_contiguous(int wg, int count) {
    const int q = count >> 3, rem = count & 7;
    const int xcd = wg & 7, idx = wg >> 3;
    return xcd * q + min(xcd, rem) + idx;
}

// The work of one workgroup: output tile number `tile_idx` (in XCD-contiguous numbering, see above) of a tiles_m x
// tiles_n grid of BM x BN tiles whose first column is n_base and whose first row is m_base, k-share `split` of
// `num_splits` (each share has its own output plane).
// NS LDS stages of 64 k-values for the A tile and NSW (NS or NS + 1, at least 3) for the W tile.  The weights stream from
// HBM, the activations are re-read from the caches by every tile column, so where LDS cannot hold one more stage of both
// (256x256: two of each fill 128 of the 160 KiB) the W tile alone gets the third: its loads then have two k-steps
// to land instead of one.
// THROUGH: the results are written through the L2 (see kAuxWriteThrough).
// W_FAR: 32-bit offsets do not reach over the row blocks of W in a tile or along its k range, so each block of each k-step
// gets a buffer of its own (two scalar additions per load).
template <int BM, int BN, int WGM, int WGN, int MODE, int NS = 2, int NSW = NS, bool W_ONCE = false, bool W_FAR = false, bool THROUGH = false>
__device__ __forceinline__ void gemm_tile(const bf16_t* __restrict__ A, int64_t lda, const bf16_t* __restrict__ W,
                                          int64_t ldw, void* __restrict__ out, int64_t ldc, int M, int K,
                                          int tiles_m, int tiles_n, int n_base, int tile_idx, int split, int num_splits,
                                          int64_t split_stride, int m_base = 0) {
#if defined(__HIP_DEVICE_COMPILE__)  // (the buffer resource type exists in device code only)
    constexpr int kAuxNonTemporal = 2;        // cache-policy operand of a buffer load: the nt bit
    // ... and of a buffer store: the sc1 bit.  Results that stay in the L2 are written back when the stream of the weights
    // displaces them, in pieces, and the reads wait for those writes all along; written through they are on their way at once.
    // 152064 x 5120 at 64 rows in a loop 296 -> 255 us (5.3 -> 6.1 TB/s of weights, 6.6 without any stores; with the nt hint 262); norm,
    // projection and sampling of 128256 x 4096, 64 rows 195 -> 176, 128 rows 213 -> 192.  In a single round all results are stored when the stream has ended, and the
    // next kernel reads them: there they are left to the L2 (197 rows, eight layers 1243 us, written through 1257).
    constexpr int kAuxWriteThrough = 16;
    constexpr int kBufferFlags = 0x00027000;  // raw buffer of 32-bit words, bounds checked in bytes
    constexpr int NW = WGM * WGN;
    constexpr int WTM = BM / WGM, WTN = BN / WGN;  // wave tile
    constexpr int TM = WTM / MB, TN = WTN / MB;    // MFMA blocks per wave
    constexpr int GA = BM / 8 / NW, GW = BN / 8 / NW;  // 1 KiB load groups per wave and stage: A, W
    constexpr int GPW = GA + GW;
    constexpr int A_STAGE = BM * BK * 2, W_STAGE = BN * BK * 2, W_BASE = NS * A_STAGE;
    constexpr int LDS_BYTES = NS * A_STAGE + NSW * W_STAGE;
    static_assert(NSW == NS || NSW == NS + 1, "the W tile has as many stages as the A tile, or one more");
    static_assert((BM / 8) % NW == 0 && (BN / 8) % NW == 0 && NW % 2 == 0, "load groups must divide among an even number of waves");
    static_assert(WTM % MB == 0 && WTN % MB == 0, "a wave tile is made of whole MFMA blocks");
    static_assert(MODE != GEMM_SWIGLU_BF16 || WTN % (2 * kSwigluGroup) == 0 || WTN == 2 * MB, "SwiGLU needs gate and up columns in one wave");
    // a wave tile of 32 columns takes 16 gate columns and the 16 up columns of the same outputs
    constexpr bool kPaired = MODE == GEMM_SWIGLU_BF16 && WTN == 2 * MB;
    extern __shared__ __attribute__((aligned(1024))) unsigned char smem[];

    // ---- tile assignment: tiles are numbered band by band ----
    const int wg = tile_idx;
    constexpr int BAND = 8;  // tile columns per band
    const int band = wg / (BAND * tiles_m);
    const int band_cols = min(BAND, tiles_n - band * BAND);
    const int in_band = wg - band * BAND * tiles_m;
    const int tile_m = in_band / band_cols;
    const int tile_n = band * BAND + in_band % band_cols;
    const int m0 = m_base + tile_m * BM, n0 = n_base + tile_n * BN;

    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int wm = wave / WGN, wn = wave % WGN;

    // split-K: a share is a contiguous part of the k range with its own output plane
    const int KT = (K / BK) / num_splits;
    const int kt_base = split * KT;
    const int64_t split_off = (int64_t)split * split_stride;

    // ---- loader: wave w fills groups w, w + NW, ...; lane offsets are the same for every group ----
    // group g covers rows 8g .. 8g+7 = lines 4g .. 4g+3; NW is even, so g has the parity of `wave`
    const int lline = lane >> 4;
    const int lq = (lane & 15) ^ ((4 * (wave & 1) + lline) & 7);
    const int lrow = 2 * lline + (lq >> 3), lgrp = lq & 7;
    // Buffer addressing: the k position is the scalar offset of a load, everything else one precomputed register per
    // group, so that a load costs no address arithmetic.  Rows past M lie outside the buffer: they read as zero.
    const int64_t w_blocks_k = ldw >> 6;
    const uint32_t a_rows = (uint32_t)min(BM, M - m0);
    const auto a_buf = __builtin_amdgcn_make_buffer_rsrc((void*)(A + (int64_t)m0 * lda), 0, (int)(uint32_t)(a_rows * lda * 2), kBufferFlags);
    const auto w_buf = __builtin_amdgcn_make_buffer_rsrc((void*)((const char*)W + (int64_t)(n0 >> 6) * w_blocks_k * kWBlockBytes), 0,
                                                         (int)(uint32_t)((BN >> 6) * w_blocks_k * kWBlockBytes), kBufferFlags);
    static_assert(!W_FAR || NW == 4, "the row block of a load must not depend on the wave");
    uint32_t off_a[GA], off_w[GW];
#pragma unroll
    for (int i = 0; i < GA; ++i) {
        const uint32_t r = (wave + i * NW) * 8 + lrow;
        off_a[i] = r < a_rows ? (uint32_t)(r * lda + lgrp * 8) * 2u : 0xFFFFFFF0u;
    }
    // W is tiled (see w_tiled_index): a group's 8 rows x 64 k values are 1 KiB in a row, a 64-row block 8 KiB, so a load
    // instruction reads one contiguous KiB and a k-step of the tile whole 8 KiB pieces; group g = KiB g % 8 of row block g / 8
#pragma unroll
    for (int i = 0; i < GW; ++i) {
        const int g = wave + i * NW;
        off_w[i] = (W_FAR ? 0u : (uint32_t)(g >> 3) * (uint32_t)(w_blocks_k * kWBlockBytes)) + (g & 7) * 1024u + (lrow * 64 + lgrp * 8) * 2u;
    }
    // Load i of a k-step (A: i < GA, W: the rest) into the stages at byte sa / sw of LDS.  Tiles past the last one re-read
    // the last into a stage nobody reads again.  With one band of rows (W_ONCE) every byte of W is read by one workgroup,
    // once: those loads carry the non-temporal hint, which keeps the one-pass stream from displacing the A panel in L2
    // (5-10 % on the weight-streaming products).
    auto issue = [&](int i, int kt_a, int sa, int kt_w, int sw) {
        if (i < GA)
            __builtin_amdgcn_raw_ptr_buffer_load_lds(a_buf, (lptr_t)(smem + sa + (wave + i * NW) * 1024), 16, off_a[i],
                                                     (min(kt_a, KT - 1) + kt_base) * (BK * 2), 0, 0);
        else if constexpr (W_FAR) {  // load i - GA fills rows 8 (wave + 4 (i - GA)) .. + 7: row block (i - GA) / 2
            const int64_t block = (int64_t)((n0 >> 6) + (i - GA) / 2) * w_blocks_k + min(kt_w, KT - 1) + kt_base;
            const auto buf = __builtin_amdgcn_make_buffer_rsrc((void*)((const char*)W + block * kWBlockBytes), 0, kWBlockBytes, kBufferFlags);
            __builtin_amdgcn_raw_ptr_buffer_load_lds(buf, (lptr_t)(smem + sw + (wave + (i - GA) * NW) * 1024), 16, off_w[i - GA], 0, 0, 0);
        } else
            __builtin_amdgcn_raw_ptr_buffer_load_lds(w_buf, (lptr_t)(smem + sw + (wave + (i - GA) * NW) * 1024), 16, off_w[i - GA],
                                                     (min(kt_w, KT - 1) + kt_base) * kWBlockBytes, 0, W_ONCE ? kAuxNonTemporal : 0);
    };

    f32x4 acc[TM][TN];
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};

    {
        // operand reads: lane supplies row (lane % 16), k-group (lane / 16) of each 32-wide k-step
        constexpr int KK = BK / MK;
        constexpr int kReads = TM + TN, kMfma = TM * TN;
        constexpr int kPart = (GPW + KK - 1) / KK;  // global loads issued per k-step
        const int frow = lane & (MB - 1), fgrp = lane / MB;
        const int fsw = (frow >> 1) & 7, fpar = (frow & 1) * 8;
        const int a_off = (wm * WTM + (frow & ~1)) * (BK * 2), w_off = ((kPaired ? wn / 2 * (2 * kSwigluGroup) + wn % 2 * MB : wn * WTN) + (frow & ~1)) * (BK * 2);
        int fg[KK];
#pragma unroll
        for (int kk = 0; kk < KK; ++kk) fg[kk] = ((fpar + kk * (MK / 8) + fgrp) ^ fsw) * 16;
        bf16x8 fa[2][TM], fw[2][TN];
        // operand read r of k-step kk of the tile in the stages at sa, sw, in the order the MFMAs want them
        auto read_frag = [&](int r, int kk, int sa, int sw, int buf) {
            if (r == 0) fa[buf][0] = *reinterpret_cast<const bf16x8*>(smem + sa + a_off + fg[kk]);
            else if (r <= TN) fw[buf][r - 1] = *reinterpret_cast<const bf16x8*>(smem + sw + w_off + fg[kk] + (r - 1) * (kPaired ? kSwigluGroup : MB) * (BK * 2));
            else fa[buf][r - TN] = *reinterpret_cast<const bf16x8*>(smem + sa + a_off + fg[kk] + (r - TN) * MB * (BK * 2));
        };
        // One k-step: multiply the fragments in `buf`, fetch those of k-step kk_next of the tile in the stages at ra, rw
        // into the other buffer, issue part q of the global loads.  The order is written out and held by scheduling
        // barriers: one operand read behind each of the first MFMAs, so that those left over cover the latency of the last
        // read, the global loads spread over all of them.  (Given groups to interleave instead, the compiler packs reads
        // into bursts with full waits between them.)
        auto step = [&](int buf, bool fetch, int kk_next, int ra, int rw, int q, int kt_a, int sa, int kt_w, int sw) {
            const int loads = q < 0 ? 0 : max(0, min(kPart, GPW - q * kPart));
#pragma unroll
            for (int r = 0; r < kMfma; ++r) {
                acc[r / TN][r % TN] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(fa[buf][r / TN], fw[buf][r % TN], acc[r / TN][r % TN], 0, 0, 0);
                __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                for (int f = 0; f < kReads; ++f)
                    if (fetch && f * kMfma / (kReads < kMfma ? kMfma : kReads) == r) read_frag(f, kk_next, ra, rw, buf ^ 1);
#pragma unroll
                for (int l = 0; l < kPart; ++l)
                    if (l < loads && l * kMfma / loads == r) issue(q * kPart + l, kt_a, sa, kt_w, sw);
                __builtin_amdgcn_sched_barrier(0);
            }
        };

        // Software pipeline.  Global: tiles kt+1 .. kt+NS-1 of A (.. kt+NSW-1 of W) are in flight while tile kt is
        // multiplied.  LDS -> registers: the fragments of k-step kk+1 are fetched while k-step kk is multiplied, also
        // across the tile boundary: the barrier sits before the last k-step of a tile, after which the next tile's
        // first fragments are fetched under the MFMAs of that last k-step.  The loads into the stages vacated at that
        // barrier are issued in KK parts, one per k-step from there on (part 0 behind the barrier, part q + 1 in
        // k-step q of the next tile), A before W: a load instruction keeps the address unit busy for 16 cycles, and all
        // of them at once stall every wave behind the barrier for longer than the MFMAs of one k-step last.
        // Every iteration issues the same number of loads (see issue), so the wait counts are compile-time constants.
        // Loads complete in issue order, so "all but the newest ..." leaves exactly the tiles that may be in flight.
        constexpr int kInFlight = (NS - 2) * GPW + (NSW - NS) * GW;  // loads that may be outstanding at a step's barrier
        constexpr int kFirstPart = kPart < GPW ? kPart : GPW;
        static_assert(NSW >= 3, "the loads of a tile are spread over a whole k-step of 64: its W tile needs one more to land");
        static_assert(kInFlight + GPW < 64, "outstanding loads must fit the vmcnt field");
#pragma unroll
        for (int t = 0; t < NSW - 1; ++t) {
#pragma unroll
            for (int i = t < NS - 1 ? 0 : GA; i < GPW; ++i) issue(i, t, t * A_STAGE, t, W_BASE + t * W_STAGE);
        }
        int fill_a = (NS - 1) * A_STAGE, fill_w = W_BASE + (NSW - 1) * W_STAGE;  // stages being filled
        int read_a = 0, read_w = W_BASE;                                         // stages being multiplied
#pragma unroll
        for (int l = 0; l < kFirstPart; ++l) issue(l, NS - 1, fill_a, NSW - 1, fill_w);
        asm volatile("s_waitcnt vmcnt(%0)" ::"n"((NS - 2) * GA + (NSW - 2) * GW + kFirstPart) : "memory");
        __builtin_amdgcn_s_barrier();
#pragma unroll
        for (int f = 0; f < kReads; ++f) read_frag(f, 0, read_a, read_w, 0);
        __builtin_amdgcn_sched_barrier(0);
        for (int kt = 0; kt < KT - 1; ++kt) {
#pragma unroll
            for (int kk = 0; kk < KK - 1; ++kk)
                step(kk & 1, true, kk + 1, read_a, read_w, kk + 1, kt - 1 + NS, fill_a, kt - 1 + NSW, fill_w);
            // tile kt+1 must have landed (later tiles may still be in flight) and this wave's last fragments of
            // tile kt must be in registers before anybody overwrites its stages
            asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)" ::"n"(kInFlight) : "memory");
            __builtin_amdgcn_s_barrier();
            __builtin_amdgcn_sched_barrier(0);
            // the stages just vacated are filled next; the first fragments of tile kt+1 are fetched
            fill_a = read_a;
            fill_w = read_w;
            read_a = read_a == (NS - 1) * A_STAGE ? 0 : read_a + A_STAGE;
            read_w = read_w == W_BASE + (NSW - 1) * W_STAGE ? W_BASE : read_w + W_STAGE;
            step((KK - 1) & 1, true, 0, read_a, read_w, 0, kt + NS, fill_a, kt + NSW, fill_w);
        }
#pragma unroll
        for (int kk = 0; kk < KK; ++kk) step(kk & 1, kk < KK - 1, kk + 1 < KK ? kk + 1 : 0, read_a, read_w, -1, 0, 0, 0, 0);
    }

    // ---- epilogue, staged through LDS so that every global access is a 16-byte piece of a long row
    // segment.  Accumulator element v of a 16x16 block sits at row 4*(lane/16) + v, column
    // lane%16; a wave writes one 16-row slab of its tile to its private LDS area, then reads it back row
    // by row, 4 consecutive columns per lane.  Only the first barrier is needed (the slabs overlay the tiles).
    constexpr int C = (MODE == GEMM_SWIGLU_BF16) ? WTN / 2 : WTN;  // result columns of a wave slab
    constexpr int CS = C + 8;                                       // padded row stride (floats)
    constexpr int LPR = C / 4;                                      // lanes per row on the way out
    constexpr int RPI = 64 / LPR;                                   // rows per read instruction (lanes >= RPI*LPR idle)
    static_assert(MB % RPI == 0, "a slab must be a whole number of read instructions");
    static_assert(NW * MB * CS * 4 <= LDS_BYTES, "epilogue slab must fit in the tile buffers");
    float* slab = reinterpret_cast<float*>(smem) + wave * (MB * CS);
    const int col_in = lane & (MB - 1), row_in = lane / MB * 4;
    const int orow = lane / LPR, ocol = (lane % LPR) * 4;
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");  // the redundant tail loads have landed too
    __syncthreads();  // all waves have finished reading the last tile
#pragma unroll
    for (int i = 0; i < TM; ++i) {
        if (MODE == GEMM_SWIGLU_BF16) {
            // the columns alternate between kSwigluGroup gate and as many up columns of the same outputs
            constexpr int GB = kPaired ? 1 : kSwigluGroup / MB;
#pragma unroll
            for (int j = 0; j < TN / 2; ++j) {
                const int gate = j / GB * (2 * GB) + j % GB;
#pragma unroll
                for (int v = 0; v < 4; ++v) slab[(row_in + v) * CS + j * MB + col_in] = silu(acc[i][gate][v]) * acc[i][gate + GB][v];
            }
        } else {
#pragma unroll
            for (int j = 0; j < TN; ++j)
#pragma unroll
                for (int v = 0; v < 4; ++v) slab[(row_in + v) * CS + j * MB + col_in] = acc[i][j][v];
        }
        // the slab is private to the wave and LDS executes a wave's instructions in order: no barrier needed
        const int mrow0 = m0 + wm * WTM + i * MB;
        const auto slab_out = __builtin_amdgcn_make_buffer_rsrc((void*)(reinterpret_cast<float*>(out) + split_off + (int64_t)mrow0 * ldc + n0 + wn * WTN),
                                                                0, -1, kBufferFlags);  // (THROUGH)
        const bool lane_on = RPI * LPR == 64 || lane < RPI * LPR;
        f32x4 val[MB / RPI];
#pragma unroll
        for (int r = 0; r < MB; r += RPI)  // all reads first, so that their latencies overlap
            val[r / RPI] = *reinterpret_cast<const f32x4*>(slab + (r + (lane_on ? orow : 0)) * CS + (lane_on ? ocol : 0));
#pragma unroll
        for (int r = 0; r < MB; r += RPI) {
            const int m = mrow0 + r + orow;
            if (!lane_on || m >= M) continue;
            if (MODE == GEMM_SWIGLU_BF16) {
                bf16_t* p = reinterpret_cast<bf16_t*>(out) + (int64_t)m * ldc + (n0 + wn * WTN) / 2 + ocol;
                *reinterpret_cast<bf16x4*>(p) = __builtin_convertvector(val[r / RPI], bf16x4);
            } else {
                float* p = reinterpret_cast<float*>(out) + split_off + (int64_t)m * ldc + n0 + wn * WTN + ocol;
                if (MODE == GEMM_ADD_F32) {
                    f32x4 old = *reinterpret_cast<const f32x4*>(p);
                    *reinterpret_cast<f32x4*>(p) = old + val[r / RPI];
                } else if (THROUGH) {  // (offsets count from the first row of the slab: 32 bits reach over its 16 rows, see kThroughMaxLd)
                    __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(u32x4, val[r / RPI]), slab_out,
                                                           (int)(((uint32_t)(r + orow) * (uint32_t)ldc + (uint32_t)ocol) * 4u), 0, kAuxWriteThrough);
                } else {
                    *reinterpret_cast<f32x4*>(p) = val[r / RPI];
                }
            }
        }
    }
#endif
}

// LDS stages of the A tile beside three of a 256-column W tile: what 160 KiB hold.
template <int H>
constexpr int kWideStages = H <= 160 ? 3 : 2;

template <int BM, int BN, int WGM, int WGN, int MODE, int NS = 2, int NSW = NS, bool W_ONCE = false, bool W_FAR = false, bool THROUGH = false>
__global__ __launch_bounds__(64 * WGM * WGN) void gemm_bf16_kernel(const bf16_t* __restrict__ A, int64_t lda,
                                                                    const bf16_t* __restrict__ W, int64_t ldw,
                                                                    void* __restrict__ out, int64_t ldc, int M,
                                                                    int K, int tiles_m, int tiles_n,
                                                                    int64_t split_stride) {
    // Split-K launches are a (tiles, splits) grid; workgroup ids run over the tiles first.  All of it is renumbered at
    // once, k-share by k-share, so that an XCD works on tiles of ONE k-share at a time where it can: the tiles that
    // share its L2 then read the same k range of their A and W panels (with both shares of a tile range on one XCD,
    // as the plain per-share numbering would place them, the L2 sees half as many tiles per panel).
    const int num_tiles = tiles_m * tiles_n;
    const int v = xcd_contiguous(blockIdx.x + blockIdx.y * num_tiles, num_tiles * (int)gridDim.y);
    gemm_tile<BM, BN, WGM, WGN, MODE, NS, NSW, W_ONCE, W_FAR, THROUGH>(A, lda, W, ldw, out, ldc, M, K, tiles_m, tiles_n, 0, v % num_tiles,
                                                       v / num_tiles, gridDim.y, split_stride);
}

// Two tile shapes in one launch: the first big_tiles workgroups cover columns [0, n_split) with H x 256 tiles (whole rounds
// of the 256 compute units), the rest cover [n_split, N) with H x 128 tiles, so that the last, partial round still gives
// every compute unit a (half-size) tile.
template <int MODE, int H, bool W_ONCE, bool THROUGH>
__global__ __launch_bounds__(256) void gemm_bf16_mixed_kernel(const bf16_t* __restrict__ A, int64_t lda,
                                                               const bf16_t* __restrict__ W, int64_t ldw,
                                                               void* __restrict__ out, int64_t ldc, int M, int K,
                                                               int tiles_m, int big_cols, int small_cols) {
    const int big_tiles = tiles_m * big_cols;
    if ((int)blockIdx.x < big_tiles)
        gemm_tile<H, 256, 2, 2, MODE, kWideStages<H>, 3, W_ONCE, false, THROUGH>(A, lda, W, ldw, out, ldc, M, K, tiles_m, big_cols, 0,
                                                                xcd_contiguous(blockIdx.x, big_tiles), 0, 1, 0);
    else
        gemm_tile<H, 128, 2, 2, MODE, 3, 3, W_ONCE, false, THROUGH>(A, lda, W, ldw, out, ldc, M, K, tiles_m, small_cols, big_cols * 256,
                                                    xcd_contiguous(blockIdx.x - big_tiles, tiles_m * small_cols), 0, 1, 0);
}

// One band of 257..288 rows, two widths in one launch: whole rounds of 288x192 tiles, then 288x128 ones for a last round.
template <bool THROUGH>
__global__ __launch_bounds__(256) void gemm_bf16_tall_mixed_kernel(const bf16_t* __restrict__ A, int64_t lda, const bf16_t* __restrict__ W,
                                                                   int64_t ldw, void* __restrict__ out, int64_t ldc, int M, int K,
                                                                   int big_cols, int small_cols) {
    if ((int)blockIdx.x < big_cols)
        gemm_tile<288, 192, 2, 2, GEMM_STORE_F32, 2, 3, true, false, THROUGH>(A, lda, W, ldw, out, ldc, M, K, 1, big_cols, 0,
                                                                              xcd_contiguous(blockIdx.x, big_cols), 0, 1, 0);
    else
        gemm_tile<288, 128, 2, 2, GEMM_STORE_F32, 3, 3, true, false, THROUGH>(A, lda, W, ldw, out, ldc, M, K, 1, small_cols, big_cols * 192,
                                                                              xcd_contiguous(blockIdx.x - big_cols, small_cols), 0, 1, 0);
}

// Two tile heights in one launch: the first big_tiles workgroups cover the whole bands of 256 rows with 256x256
// tiles, the rest cover the last band -- at most BMR rows are left -- with BMR x 256 tiles, so a row count just above a
// multiple of 256 does not pay for a whole band of padding.  blockIdx.y is the split-K share.
template <int MODE, int BMR>
__global__ __launch_bounds__(256) void gemm_bf16_rowmix_kernel(const bf16_t* __restrict__ A, int64_t lda,
                                                                const bf16_t* __restrict__ W, int64_t ldw,
                                                                void* __restrict__ out, int64_t ldc, int M, int K,
                                                                int bands, int tiles_n, int64_t split_stride) {
    const int big_tiles = bands * tiles_n;
    if ((int)blockIdx.x < big_tiles)
        gemm_tile<256, 256, 2, 2, MODE, 2, 3>(A, lda, W, ldw, out, ldc, M, K, bands, tiles_n, 0,
                                              xcd_contiguous(blockIdx.x, big_tiles), blockIdx.y, gridDim.y, split_stride);
    else
        gemm_tile<BMR, 256, 2, 2, MODE, 3>(A, lda, W, ldw, out, ldc, M, K, 1, tiles_n, 0,
                                           xcd_contiguous(blockIdx.x - big_tiles, tiles_n), blockIdx.y, gridDim.y,
                                           split_stride, bands * 256);
}

// Operands that the tiles cannot address: a row of A or the start of W off a 4-byte boundary (what a buffer load needs).  One thread per result, products summed in order of k; such operands come from
// callers' views, not from the stage or the head, so this is for completeness and not for speed.
template <int MODE>
__global__ __launch_bounds__(256) void gemm_any_address_kernel(const bf16_t* __restrict__ A, int64_t lda, const bf16_t* __restrict__ W,
                                                                int64_t ldw, void* __restrict__ out, int64_t ldc, int M, int cols, int K,
                                                                int64_t split_stride) {
    const int64_t at = (int64_t)blockIdx.x * 256 + threadIdx.x, m = at / cols;
    const int c = (int)(at % cols);
    if (m >= M) return;
    const int share = K / (int)gridDim.y, k0 = share * (int)blockIdx.y;
    const int64_t row = MODE == GEMM_SWIGLU_BF16 ? c / kSwigluGroup * (2 * kSwigluGroup) + c % kSwigluGroup : c;
    float sum = 0.f, up = 0.f;
    for (int k = k0; k < k0 + share; ++k) {
        const float x = (float)A[m * lda + k];
        sum += x * (float)W[w_tiled_index(row, k, ldw)];
        if (MODE == GEMM_SWIGLU_BF16) up += x * (float)W[w_tiled_index(row + kSwigluGroup, k, ldw)];
    }
    float* f = reinterpret_cast<float*>(out) + blockIdx.y * split_stride + m * ldc + c;
    if (MODE == GEMM_SWIGLU_BF16) reinterpret_cast<bf16_t*>(out)[m * ldc + c] = (bf16_t)(silu(sum) * up);
    else if (MODE == GEMM_ADD_F32) *f += sum;
    else *f = sum;
}

// Whether results are written through the L2 (see kAuxWriteThrough): where one band of rows takes more than a round, a tile per compute
// unit, and the results are more than the L2s keep until the launch ends.  us, left in the L2 / written through: 128256 x 4096, 8 rows (4
// MB) 160 / 158, 16 rows (8 MB) 164 / 161, 32 rows 172 / 160, 128 rows 197 / 175; 152064 x 5120, 16 rows (10 MB) 245 / 247, 32 rows 264 / 249;
// 49152 x 4096, 16 rows (3 MB) 64 / 65, 64 rows (13 MB) 80 / 75; 10240 x 8192, 17 rows in eight planes (6 MB) 29 / 31 (a workgroup ends
// when its stores have arrived).  With several bands there is no difference (4160 rows).  Rows must be near enough for 32-bit offsets over 16, and
// follow one another upwards.
constexpr int64_t kThroughMinTiles = 257, kThroughMinBytes = 12000000, kThroughMaxLd = ((int64_t)1 << 26) - 1;
bool write_through(int64_t tiles, int m, int n, int splits, int64_t ldc) {
    return tiles >= kThroughMinTiles && (int64_t)m * n * splits * 4 >= kThroughMinBytes && ldc >= 0 && ldc <= kThroughMaxLd;
}

// LDS that two workgroups do not have room for: launches whose results are written through ask for it where `alone` says that one
// tile at a time on a compute unit is better (see launch_skinny).
constexpr size_t kAloneLds = 84 * 1024;

template <int BM, int BN, int WGM, int WGN, int MODE, int NS, int NSW, bool W_ONCE, bool W_FAR = false, bool THROUGH = false>
hipError_t launch_tile_w(const bf16_t* a, int64_t lda, const bf16_t* w, int64_t ldw, void* out, int64_t ldc, int m,
                         int n, int k, int splits, int64_t split_stride, hipStream_t stream, bool alone = false) {
    if constexpr (MODE == GEMM_STORE_F32 && W_ONCE && !THROUGH) {
        if (m <= BM && write_through((int64_t)(n / BN) * splits, m, n, splits, ldc))
            return launch_tile_w<BM, BN, WGM, WGN, MODE, NS, NSW, W_ONCE, W_FAR, true>(a, lda, w, ldw, out, ldc, m, n, k, splits, split_stride, stream, alone);
    }
    const int tiles_m = (int)ceil_div(m, BM), tiles_n = n / BN;
    constexpr size_t kStages = (NS * BM + NSW * BN) * BK * sizeof(bf16_t), kMost = std::max(kStages, kAloneLds);
    const size_t smem = THROUGH && alone ? kMost : kStages;
    auto kern = gemm_bf16_kernel<BM, BN, WGM, WGN, MODE, NS, NSW, W_ONCE, W_FAR, THROUGH>;
    static bool configured = false;
    if (!configured) {
        hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(kern),
                                           hipFuncAttributeMaxDynamicSharedMemorySize, (int)kMost);
        if (e != hipSuccess) return e;
        configured = true;
    }
    kern<<<dim3(tiles_m * tiles_n, splits), 64 * WGM * WGN, smem, stream>>>(a, lda, w, ldw, out, ldc, m, k, tiles_m,
                                                                          tiles_n, split_stride);
    return hipGetLastError();
}

// All rows in one band: the weights are read once (W_ONCE, see gemm_tile).
template <int BM, int BN, int WGM, int WGN, int MODE, int NS = 2, int NSW = NS>
hipError_t launch_tile(const bf16_t* a, int64_t lda, const bf16_t* w, int64_t ldw, void* out, int64_t ldc, int m,
                       int n, int k, int splits, int64_t split_stride, hipStream_t stream) {
    return m <= BM ? launch_tile_w<BM, BN, WGM, WGN, MODE, NS, NSW, true>(a, lda, w, ldw, out, ldc, m, n, k, splits, split_stride, stream)
                   : launch_tile_w<BM, BN, WGM, WGN, MODE, NS, NSW, false>(a, lda, w, ldw, out, ldc, m, n, k, splits, split_stride, stream);
}

// Heights.  A band of 256 rows around 200 does a fifth of its MFMAs and LDS reads for nothing, two of 256 around 400 likewise,
// so rows are cut into bands of equal height, a multiple of 32 (16 rows a wave); from 257 to 384 rows one band of them all
// with 128 columns reads the weights once instead of twice.  us, before -> after (gate/up 28672 x 4096, best tile before): 200
// rows 55.4 -> 52.7, 257 rows 72.7 -> 58.4, 320 rows 76.8 -> 66.3, 352 rows 78.0 -> 69.6, 448 rows 97.4 -> 82.8; vocabulary
// 128256 x 4096: 200 rows 225.6 -> 208.3, 257 rows 303.1 -> 282.2, 320 rows 357.4 -> 301.1, 448 rows 417.0 -> 382.1.
// Height of `bands` bands of equal height that cover m rows: a multiple of 32 from 160 on (lower ones gain nothing: the
// weights' stream bounds them).
int band_height(int m, int bands) { return std::max(160, (int)round_up(ceil_div(m, bands), 32)); }

// Bands of at most 256 rows: as few as cover m rows, or one more where that pads less (960 rows: five of 192, not four of 256).
int gemm_band_height(int m, int mode) {
    if (mode == GEMM_ADD_F32) return 256;  // (no caller of this library's own: one height)
    const int few = (int)ceil_div(m, 256), h0 = band_height(m, few), h1 = band_height(m, few + 1);
    return round_up(m, h1) < round_up(m, h0) ? h1 : h0;
}

// Up to 64 rows: tiles of H rows (32 or 64) x COLS columns (128 or 64, see skinny_columns).  Up to 256 of them have a compute
// unit each and keep more loads in flight (four LDS stages, six of 32x64; 128-column tiles against three: 0.97 of the time at
// up to 32 rows, 0.97 at 33 to 64); from there two tiles or more share a compute unit, and three stages (four of 64 columns) let
// as many in (deeper 128-column tiles at 432 and 448 tiles 1.02, 64-column ones 1.01 to 1.04).  In several rounds of which
// the last is nearly full two stages of A and three of W: with more loads in flight some compute units run ahead of others and the
// last round is a long tail (128256 x 4096, 64 rows: the first tiles end between 62 and 91 us, so between 77 and 82).
// 128256 x 4096: one row 157 -> 153 us, 32 rows 178 -> 170, 64 rows 199 -> 179 (all with results left in
// the L2s); 128256 x 8192, 64 rows 355 -> 338.  Where the last round is short the tiles had better end at different times (152064 x
// 8192, 0.3 of a round left, 64 rows: 433 and 453).
// There, with results that are written through, one tile at a time on a compute unit keeps the rounds of 256 together (two tiles end
// apart, and the last ones run alone), from more than four of them on: norm, projection and sampling together 0.96 to 1.00 of the time at 24
// to 64 rows, 1.02 at most, k of 2048 to 8320 and 4.0 to 7.0 rounds alike (152064 x 5120, 64 rows 266 -> 258 us), up to 3.4 rounds 0.97 to
// 1.05; but 1.00 to 1.06 where the tiles lie 1 MiB apart (k of 4096; 3840 and 4224 gain; why is not known).  All of them:
// profiles/gemm_one_tile_at_a_time.txt.
// Two against three stages of A at 1.06 to 4 rounds, k of 4096, 5120 and 8192, one to 64 rows: a full last round takes 0.96 to
// 1.0 of the time, 0.75 and 0.88 of one 0.85 to 1.0, 0.62 of one 0.95 to 0.99, half of one 0.98 to 1.12, a quarter 0.95 to 1.15.
constexpr int kSkinnySlots = 512;  // 128-column tiles of three stages that run at one time, two per compute unit
constexpr int64_t kAloneMinTiles = 1025, kNotAloneApart = (int64_t)1 << 20;  // tiles, bytes from the weights of a tile to those of the next
template <int MODE, int H, int COLS>
hipError_t launch_skinny(const bf16_t* a, int64_t lda, const bf16_t* w, int64_t ldw, void* out, int64_t ldc, int m,
                         int n, int k, int splits, int64_t split_stride, hipStream_t stream) {
    constexpr int WM = H == 32 && COLS == 128 ? 1 : 2;  // waves along the rows
    const int64_t tiles = (int64_t)(n / COLS) * splits, last = tiles % kSkinnySlots;
    if constexpr (COLS == 64) {
        if constexpr (H == 32) {
            if (tiles <= 256) return launch_tile_w<H, COLS, WM, 4 / WM, MODE, 6, 6, true>(a, lda, w, ldw, out, ldc, m, n, k, splits, split_stride, stream);
        }
        return launch_tile_w<H, COLS, WM, 4 / WM, MODE, 4, 4, true>(a, lda, w, ldw, out, ldc, m, n, k, splits, split_stride, stream);
    } else {
        if (tiles <= 256) return launch_tile_w<H, COLS, WM, 4 / WM, MODE, 4, 4, true>(a, lda, w, ldw, out, ldc, m, n, k, splits, split_stride, stream);
        if (tiles > kSkinnySlots && (last == 0 || last >= kSkinnySlots * 3 / 4))
            return launch_tile_w<H, COLS, WM, 4 / WM, MODE, 2, 3, true>(a, lda, w, ldw, out, ldc, m, n, k, splits, split_stride, stream);
        return launch_tile_w<H, COLS, WM, 4 / WM, MODE, 3, 3, true>(a, lda, w, ldw, out, ldc, m, n, k, splits, split_stride, stream,
                                                                    tiles >= kAloneMinTiles && ldw * COLS * 2 != kNotAloneApart);
    }
}
int skinny_columns(int m, int n, int k, int mode, int splits);
// One band of 257..288 rows in store mode: tiles of 128 or of 192 columns, or whole rounds of 192 and a last one of 128.
enum class Tall { k128, k192, kMixed };
Tall tall_form(int m, int n, int splits);
int tall_mixed_cols(int n);

// Tile 6 up to 128 rows: 64 columns where half of the compute units would be without a tile of 128 and nearly all have one of 64.
// 360 products of 65 to 128 rows (profiles/gemm_65_to_128_rows.txt), planes read included: where it is picked, 0.91 of the best form
// without it on average, 0.78 to 1.00 (4096 x 4096 in four shares of k instead of eight: 80 rows 12.8 -> 10.8 us, 128 rows 14.9 ->
// 13.1).  Above 128 tiles two share a compute unit and 64 columns are always slower (1.03 to 1.43).  Below 113 they are faster in the
// same shares (0.7 to 0.8), but the fewer shares that the plan would then take are not always (0.77 to 1.25 of the best, 3584 x 5120 at 65 rows
// 12.2 -> 11.9); there the forms are as they were, unmeasured in a stage: no shape here has such a product at these rows.
bool half_width_deep(int m, int n, int splits) {
    const int64_t tiles = (int64_t)(n / 128) * splits;
    return m <= 128 && tiles > 112 && tiles <= 128;
}

// See gemm_bf16_tall_mixed_kernel.
template <bool THROUGH>
hipError_t launch_tall_mixed(const bf16_t* a, int64_t lda, const bf16_t* w, int64_t ldw, void* out, int64_t ldc, int m, int n, int k,
                             hipStream_t stream) {
    const int big_cols = tall_mixed_cols(n), small_cols = (n - big_cols * 192) / 128;
    constexpr size_t smem = 3 * (288 + 128) * BK * sizeof(bf16_t);  // (more than the 2 x 288 + 3 x 192 rows of the other width)
    auto kern = gemm_bf16_tall_mixed_kernel<THROUGH>;
    static bool configured = false;
    if (!configured) {
        hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(kern),
                                           hipFuncAttributeMaxDynamicSharedMemorySize, (int)smem);
        if (e != hipSuccess) return e;
        configured = true;
    }
    kern<<<big_cols + small_cols, 256, smem, stream>>>(a, lda, w, ldw, out, ldc, m, k, big_cols, small_cols);
    return hipGetLastError();
}

template <int MODE>
hipError_t launch_mode(const bf16_t* a, int64_t lda, const bf16_t* w, int64_t ldw, void* out, int64_t ldc, int m,
                       int n, int k, int tile, int splits, int64_t split_stride, hipStream_t stream) {
#define GLLM_TILE_ARGS a, lda, w, ldw, out, ldc, m, n, k, splits, split_stride, stream
    const int height = gemm_band_height(m, MODE);
    switch (tile) {
        case 0: return launch_tile<128, 128, 2, 2, MODE, 2, 3>(GLLM_TILE_ARGS);  // 80 KiB of LDS: two workgroups per compute unit
        case 1:
            if (gemm_low_bands(m)) return launch_tile<192, 128, 2, 2, MODE, 4>(GLLM_TILE_ARGS);
            return launch_tile<256, 128, 2, 2, MODE, 3>(GLLM_TILE_ARGS);
        case 8: case 12: return launch_tile<192, 256, 2, 2, MODE, 2, 3>(GLLM_TILE_ARGS);  // 257..384 rows
        case 14:
            if constexpr (MODE != GEMM_ADD_F32) {
                if (height == 160) return launch_tile<160, 256, 2, 2, MODE, kWideStages<160>, 3>(GLLM_TILE_ARGS);
                if (height == 192) return launch_tile<192, 256, 2, 2, MODE, kWideStages<192>, 3>(GLLM_TILE_ARGS);
                if (height == 224) return launch_tile<224, 256, 2, 2, MODE, kWideStages<224>, 3>(GLLM_TILE_ARGS);
            }
            return launch_tile<256, 256, 2, 2, MODE, 2, 3>(GLLM_TILE_ARGS);
        case 15:
            if constexpr (MODE != GEMM_ADD_F32) {
                if (height == 160) return launch_tile<160, 128, 2, 2, MODE, 4>(GLLM_TILE_ARGS);
                if (height == 192) return launch_tile<192, 128, 2, 2, MODE, 4>(GLLM_TILE_ARGS);
                if (height == 224) return launch_tile<224, 128, 2, 2, MODE, 3>(GLLM_TILE_ARGS);
            }
            return launch_tile<256, 128, 2, 2, MODE, 3>(GLLM_TILE_ARGS);
        case 2: case 3: case 10: return launch_tile<256, 256, 2, 2, MODE, 2, 3>(GLLM_TILE_ARGS);
        case 6:
            if constexpr (MODE == GEMM_STORE_F32) {
                if (half_width_deep(m, n, splits)) return m <= 96 ? launch_tile_w<96, 64, 2, 2, MODE, 4, 4, true>(GLLM_TILE_ARGS) : launch_tile_w<128, 64, 2, 2, MODE, 4, 4, true>(GLLM_TILE_ARGS);
            }
            // (a quarter of the rows less to load, read and multiply: 0.99 of the time on average, 0.94 to 1.05)
            if (m <= 96) return launch_tile_w<96, 128, 2, 2, MODE, 3, 3, true>(GLLM_TILE_ARGS);
            return launch_tile<128, 128, 2, 2, MODE, 4>(GLLM_TILE_ARGS);
        case 7:  // (up to 32 rows half the activations to load and to read from LDS: one row of the 8B shape 785 -> 770 us)
            if constexpr (MODE == GEMM_STORE_F32) {
                if (m <= 64 && skinny_columns(m, n, k, MODE, splits) == 64)
                    return m <= 32 ? launch_skinny<MODE, 32, 64>(GLLM_TILE_ARGS) : launch_skinny<MODE, 64, 64>(GLLM_TILE_ARGS);
            }
            if (m <= 32) return launch_skinny<MODE, 32, 128>(GLLM_TILE_ARGS);
            if (m <= 64) return launch_skinny<MODE, 64, 128>(GLLM_TILE_ARGS);
            return launch_tile_w<64, 128, 2, 2, MODE, 3, 3, false>(GLLM_TILE_ARGS);
        case 13:  // one band of 257..384 rows
            if constexpr (MODE == GEMM_STORE_F32) {
                const Tall form = tall_form(m, n, splits);
                if (form == Tall::k192) return launch_tile_w<288, 192, 2, 2, MODE, 2, 3, true>(GLLM_TILE_ARGS);
                if (form == Tall::kMixed)
                    return write_through(kThroughMinTiles, m, n, 1, ldc) ? launch_tall_mixed<true>(a, lda, w, ldw, out, ldc, m, n, k, stream)
                                                                         : launch_tall_mixed<false>(a, lda, w, ldw, out, ldc, m, n, k, stream);
            }
            if constexpr (MODE != GEMM_ADD_F32) {
                if (m <= 288) return launch_tile<288, 128, 2, 2, MODE, 3>(GLLM_TILE_ARGS);
                if (m <= 320) return launch_tile<320, 128, 2, 2, MODE, 2, 3>(GLLM_TILE_ARGS);
                if (m <= 352) return launch_tile<352, 128, 2, 2, MODE, 2, 3>(GLLM_TILE_ARGS);
                return launch_tile<384, 128, 2, 2, MODE, 2, 3>(GLLM_TILE_ARGS);
            }
            return launch_tile<256, 128, 2, 2, MODE, 3>(GLLM_TILE_ARGS);
        case 5:
            if constexpr (MODE != GEMM_SWIGLU_BF16) return launch_tile<256, 192, 2, 2, MODE, 2, 3>(GLLM_TILE_ARGS);
            else return hipErrorInvalidValue;
        case 9:  // (six waves on four SIMDs, before: 24768 x 4096 at 264 rows 90 -> 74 us, 74304 x 4096 188 -> 163)
            if constexpr (MODE != GEMM_SWIGLU_BF16) return launch_tile_w<288, 192, 2, 2, MODE, 2, 3, true>(GLLM_TILE_ARGS);
            else return hipErrorInvalidValue;
        default: return hipErrorInvalidValue;
    }
#undef GLLM_TILE_ARGS
}

// Weights whose k extent is so large that the row blocks of a tile span 4 GiB: 64-column tiles, which every n allows.
template <int MODE>
hipError_t launch_far(const bf16_t* a, int64_t lda, const bf16_t* w, int64_t ldw, void* out, int64_t ldc, int m,
                      int n, int k, int splits, int64_t split_stride, hipStream_t stream) {
    return launch_tile_w<128, 64, 4, 1, MODE, 4, 4, false, true>(a, lda, w, ldw, out, ldc, m, n, k, splits, split_stride, stream);
}

constexpr size_t kWideTileLds = (2 * 256 + 3 * 256) * BK * sizeof(bf16_t);  // 256x256 tile: all 160 KiB

// Mixed launch (see gemm_bf16_mixed_kernel); rem_cols 256-wide tile columns are turned into 2*rem_cols 128-wide ones.
template <int MODE, int H, bool W_ONCE, bool THROUGH = false>
hipError_t launch_mixed_h(const bf16_t* a, int64_t lda, const bf16_t* w, int64_t ldw, void* out, int64_t ldc, int m,
                          int n, int k, int rem_cols, hipStream_t stream) {
    if constexpr (MODE == GEMM_STORE_F32 && W_ONCE && !THROUGH) {
        if (write_through(kThroughMinTiles, m, n, 1, ldc))
            return launch_mixed_h<MODE, H, W_ONCE, true>(a, lda, w, ldw, out, ldc, m, n, k, rem_cols, stream);
    }
    const int tiles_m = (int)ceil_div(m, H), big_cols = n / 256 - rem_cols, small_cols = 2 * rem_cols;
    const size_t smem = std::max(kWideStages<H> * H + 3 * 256, 3 * H + 3 * 128) * BK * sizeof(bf16_t);
    auto kern = gemm_bf16_mixed_kernel<MODE, H, W_ONCE, THROUGH>;
    static bool configured = false;
    if (!configured) {
        hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(kern),
                                           hipFuncAttributeMaxDynamicSharedMemorySize, (int)smem);
        if (e != hipSuccess) return e;
        configured = true;
    }
    kern<<<tiles_m * (big_cols + small_cols), 256, smem, stream>>>(a, lda, w, ldw, out, ldc, m, k, tiles_m, big_cols, small_cols);
    return hipGetLastError();
}

template <int MODE>
hipError_t launch_mixed(const bf16_t* a, int64_t lda, const bf16_t* w, int64_t ldw, void* out, int64_t ldc, int m,
                        int n, int k, int rem_cols, hipStream_t stream) {
#define GLLM_MIXED(H_) (m <= H_ ? launch_mixed_h<MODE, H_, true>(a, lda, w, ldw, out, ldc, m, n, k, rem_cols, stream)   \
                                : launch_mixed_h<MODE, H_, false>(a, lda, w, ldw, out, ldc, m, n, k, rem_cols, stream))
    if constexpr (MODE != GEMM_ADD_F32) {
        const int height = band_height(m, (int)ceil_div(m, 256));
        if (height == 160) return GLLM_MIXED(160);
        if (height == 192) return GLLM_MIXED(192);
        if (height == 224) return GLLM_MIXED(224);
    }
    return GLLM_MIXED(256);
#undef GLLM_MIXED
}

// Row-mixed launch (see gemm_bf16_rowmix_kernel); BMR is 64 or 128.
template <int MODE, int BMR>
hipError_t launch_rowmix(const bf16_t* a, int64_t lda, const bf16_t* w, int64_t ldw, void* out, int64_t ldc, int m,
                         int n, int k, int splits, int64_t split_stride, hipStream_t stream) {
    const int bands = m / 256, tiles_n = n / 256;
    auto kern = gemm_bf16_rowmix_kernel<MODE, BMR>;
    static bool configured = false;
    if (!configured) {
        hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(kern),
                                           hipFuncAttributeMaxDynamicSharedMemorySize, (int)kWideTileLds);
        if (e != hipSuccess) return e;
        configured = true;
    }
    kern<<<dim3((bands + 1) * tiles_n, splits), 256, kWideTileLds, stream>>>(a, lda, w, ldw, out, ldc, m, k, bands, tiles_n, split_stride);
    return hipGetLastError();
}

}  // namespace

// Whether bands of 192 rows cover m rows with less padding than bands of 256.
bool gemm_low_bands(int m) { return round_up(m, 192) < round_up(m, 256); }

// Height of the last row band for a row-mixed launch (64 or 128), or 0 when the shape does not call for one: at
// least one whole band of 256 rows and at most 128 rows left over.
int gemm_rowmix_rem_rows(int m, int n) {
    if (n % 256 != 0 || m <= 256) return 0;
    const int r = m % 256;
    return r == 0 || r > 128 ? 0 : r <= 64 ? 64 : 128;
}

// Number of 256-wide tile columns to split in two for a mixed launch, or 0 when a plain launch is as good:
// worth it when the last round of 256x256 tiles would occupy at most half of the compute units.
int gemm_mixed_rem_cols(int m, int n) {
    if (n % 256 != 0) return 0;
    const int tiles_m = (int)ceil_div(m, 256), cols = n / 256;
    const int tiles = tiles_m * cols, rem = tiles % 256;
    if (tiles < 256 || rem == 0 || rem > 128 || rem % tiles_m != 0) return 0;
    return rem / tiles_m;
}

namespace {

// Cost of a launch of one tile shape in us, fitted to measurements on MI355X with operands streaming from HBM (weights
// are cold in the stage; four stage shapes and two vocabularies, 65 to 4160 rows, every tile and split: 3036 products, forms in
// random order, median of three runs): fixed + rounds * (step * k_steps + per_tile) + plane * (us to read the fp32 result at
// 6 TB/s).  A round is one tile per compute unit (two for a shape of which two share one).  Rounds count between the work (tiles
// / tiles in a round) and the span (when the last tile ends), the span with the weight `lone`: a last round that is not full
// takes less than a whole one, because fewer tiles run faster -- the chip is power- and bandwidth-limited -- but how much less
// depends on whether whole rounds run in front of it.  No launch is faster than its loads: the weights at `stream` TB/s and
// the activations, once per tile column, at kCacheRate TB/s from the caches, both slower by as much as the last round is short
// of tiles.
// The picks are 0.37 % behind the fastest forms on average, at most 10 % (profiles/gemm_plan_sweep.txt); fitted to three quarters
// of the products, 0.44 % and 14 % on the rest, of other row counts.  Before, with one `lone` for all and the low tiles of a
// row-mixed launch in a round of their own: 1.2 %, at most 28 % (28672 x 4096 at 1050 rows 240 -> 192 us, 4096 x 4096 at 800
// rows 41 -> 35).  All that was measured before results were written through and before 288x192 tiles of four waves and of both
// widths; with these, of 78 vocabulary products at 65 to 384 rows the pick is the fastest in 74, 3 % behind at most
// (profiles/gemm_vocabulary_by_tile.txt).  Tile 6 of 96 rows goes by the costs of 128 rows (0.99 of the time), that of 64 columns by costs set by hand: of
// the products where it is in question 4.6 % behind the fastest form on average, 2.5 % from 2048 columns on (360 products of 65 to 128
// rows, profiles/gemm_65_to_128_rows.txt).
struct TileCost {
    int slots, width;  // tiles in a round, columns of a tile
    double step, fixed, lone[3];  // lone: no whole round in front of the last one, one, more
    double per_tile, plane, stream;
};
constexpr double kCacheRate = 121;
constexpr TileCost kCost128x128{512, 128, 0.867, 7.42, {0.3, 0.77, 0.26}, 2.05, 0.24, 4.61}, kCost128x128Deep{256, 128, 0.454, 3.05, {0.99, 1, 1}, 1.15, 1.55, 6.72}, kCost128x64Deep{256, 64, 0.37, 2.9, {0.99, 1, 1}, 0.9, 0.5, 6.72},
    kCost256x192{256, 192, 0.996, 6.74, {0.34, 0.82, 0.92}, 0, 1.09, 6.87}, kCost288x192{256, 192, 1.134, 3, {0.8, 0.58, 0.58}, 7.1, 0.4, 6.5};
// tiles of 160, 192, 224 and 256 rows x 128 and x 256 columns, and of 288, 320, 352 and 384 rows x 128
constexpr TileCost narrow_cost(double step) { return {256, 128, step, 3.5, {0.67, 0.86, 0.66}, 2.89, 0.58, 6.15}; }
constexpr TileCost tall_cost(double step) { return {256, 128, step, 4.89, {0.87, 0.63, 0.17}, 1.34, 0.61, 5.73}; }
constexpr TileCost wide_cost(double step) { return {256, 256, step, 3.5, {0.66, 0.62, 0.59}, 2.14, 0.62, 6.74}; }
constexpr TileCost kCostNarrow[4] = {narrow_cost(0.594), narrow_cost(0.641), narrow_cost(0.746), narrow_cost(0.759)},
                   kCostWide[4] = {wide_cost(1.021), wide_cost(1.117), wide_cost(1.296), wide_cost(1.37)},
                   kCostTall[4] = {tall_cost(0.874), tall_cost(0.902), tall_cost(0.943), tall_cost(1.113)};
const TileCost& narrow_cost_of(int height) { return kCostNarrow[(height - 160) / 32]; }
const TileCost& wide_cost_of(int height) { return kCostWide[(height - 160) / 32]; }

// Rounds that a launch counts as: `work` of them are filled, its last tile ends after `span`.
double counted_rounds(const TileCost& c, double span, double work) {
    const double lone = c.lone[(int)std::min(work + 1e-9, 2.0)];
    return lone * span + (1.0 - lone) * work;
}
double rounds_of(const TileCost& c, double tiles) { return counted_rounds(c, std::ceil(tiles / c.slots - 1e-9), tiles / c.slots); }

// The same for a row-mixed launch: `big` tiles of 256 rows, then `low` tiles of the last band, which take kLowShare of a big
// one's time each (of 64 and of 128 rows alike: fitted one by one 0.78 and 0.75) and start as compute units become free.
constexpr double kLowShare = 0.75;
double rowmix_span(double big, double low) {
    const double full = std::floor(big / 256), rest = big - full * 256, free = 256 - rest;  // compute units free after `full` rounds
    double early = 0, late = 1;  // since then: when the free units end their next tile, and the others
    double end = rest > 0 ? 1 : 0;
    const double later = std::max(0.0, std::floor(low / 256) - 2);  // once all units take low tiles, 256 of them end every kLowShare
    low -= later * 256;
    while (low > 0) {
        if (rest == 0 || early <= late) {
            early += kLowShare;
            low -= free;
            end = std::max(end, early);
        } else {
            late += kLowShare;
            low -= rest;
            end = std::max(end, late);
        }
    }
    return full + end + later * kLowShare;
}

// us of a launch whose rounds count as `rounds` and would be `full` if the last one were as good as the others.
double launch_us(const TileCost& c, int m, int n, int k, double steps, double plane, double rounds, double full) {
    const double work = c.fixed + rounds * (c.step * steps + c.per_tile) + c.plane * plane;
    const double loads = (double)n * k * 2e-6 * (1.0 / c.stream + m / (kCacheRate * c.width)) * rounds / full;
    return std::max(work, loads) + plane + 1e-3 * work;  // of two that their loads bound, the lighter one
}
double plane_us(int m, int n, int mode, int splits) { return mode == GEMM_STORE_F32 ? (double)m * n * 4.0 * splits / 6e6 : 0.0; }

// Up to 64 rows: tiles of 128 or 64 columns, a round of one per compute unit (a second one on it halves the pace of both), so
// that the tiles should come to just under a multiple of 256: 40 x 6 for 5120 x 27648, not 40 x 8 (64 rows 62.3 -> 46.1 us), 64
// x 4 of half the width for 4096 x 4096, not 32 x 8 (64 rows 11.1 -> 9.2, one row 8.0 -> 7.1: half the planes too).  Fitted to
// products of 1024 to 12288 columns and k of 1024 to 28672, and the vocabularies, at 1 to 64 rows (700, every factor and width,
// profiles/gemm_plan_up_to_64_rows.txt): 0.45 % behind the fastest form on average, more than 5 % in 18, 14 % at most (12288 x
// 8192, one row); fitted to three quarters 0.53 % on the rest.  Factors of 1, 2, 4 and 8 and 128 columns alone: 9.5 % behind.
constexpr TileCost kCostSkinny128[2] = {{256, 128, 0.544, 2.756, {0.374, 0.449, 1}, 0.646, 2.319, 7.97}, {256, 128, 0.556, 3.181, {0.536, 0.648, 1}, 0.091, 1.997, 7.789}},
                   kCostSkinny64[2] = {{256, 64, 0.29, 2.625, {0.467, 0.414, 0.618}, 0.166, 3.244, 9}, {256, 64, 0.319, 2.257, {0.856, 0.629, 0.616}, 0, 3.343, 9}};
double skinny_us(const TileCost& c, int m, int n, int k, int mode, int splits) {
    const double tiles = (double)(n / c.width) * splits;
    return launch_us(c, m, n, k, (double)(k / BK) / splits, plane_us(m, n, mode, splits), rounds_of(c, tiles), tiles / c.slots);
}

// 64 or 128: the columns of tile 7 up to 64 rows (n a multiple of 128).
int skinny_columns(int m, int n, int k, int mode, int splits) {
    const int h = m > 32;
    return mode == GEMM_STORE_F32 && skinny_us(kCostSkinny64[h], m, n, k, mode, splits) < skinny_us(kCostSkinny128[h], m, n, k, mode, splits) ? 64 : 128;
}

// 288x192 tiles in the whole rounds of a launch of both widths (as many as leave whole 288x128 ones), or 0 where there is none.
int tall_mixed_cols(int n) {
    for (int big = n / (256 * 192) * 256; big > 0; big -= 256)
        if (n > big * 192 && (n - big * 192) % 128 == 0) return big;
    return 0;
}

// 257..288 rows in one share of k (n a multiple of 128).  A wider tile loads a fifth less for a result; tiles are one to a compute unit and
// end together, so that a round that is begun counts in full, one of 192 columns 1.3 of one of 128.  Norm, projection and sampling of 257
// to 288 rows, us, by 128 / 192 / both: 49152 x 4096 137 / 111 / -, 65664 x 4096 201 / 176 / 160, 89856 x 4096 218 / 201 / 227, 100352 x 8192 475 / - /
// 448, 128256 x 4096 308 / 295 / 282, 152064 x 4096 354 / 366 / 346, 196608 x 8192 845 / 789 / 831.  At 13 column counts, k of 4096, 5120
// and 8192 and three row counts the form picked so is the fastest one each time (profiles/gemm_288_rows_by_width.txt); by the costs of the
// planner, which decided before, it was up to 27 % behind (65664 x 4096).  In more shares 128 columns are better (6144 x 4096 in four, 264 rows 26 and 31).
constexpr double kRoundOf192 = 1.3;
Tall tall_form(int m, int n, int splits) {
    if (m <= 256 || m > 288 || splits != 1) return Tall::k128;
    const double rounds128 = (double)ceil_div(n / 128, 256);
    double best = rounds128;
    Tall form = Tall::k128;
    if (n % 192 == 0 && kRoundOf192 * ceil_div(n / 192, 256) < best) {
        best = kRoundOf192 * ceil_div(n / 192, 256);
        form = Tall::k192;
    }
    if (const int big = tall_mixed_cols(n); big > 0 && kRoundOf192 * (big / 256) + ceil_div((n - big * 192) / 128, 256) < best) form = Tall::kMixed;
    return form;
}

// What the planner takes them to cost beside other tiles.  The costs of 192 columns are fitted to 14 products of one to four shares of k, with
// the share of a lone round raised by hand to that of 20160 x 4096; from two rounds on those of all widths are about a tenth
// too low (the power limit).
double tall_us(int m, int n, int k, int splits) {
    const TileCost &c128 = kCostTall[0], &c192 = kCost288x192;
    const double steps = (double)(k / BK) / splits, plane = plane_us(m, n, GEMM_STORE_F32, splits);
    auto cost_of = [&](const TileCost& c, double rounds, double full) { return launch_us(c, m, n, k, steps, plane, rounds, full); };
    const double tiles = (double)(n / 128) * splits;
    double best = cost_of(c128, rounds_of(c128, tiles), tiles / 256);
    if (splits == 1) {
        if (n % 192 == 0) best = std::min(best, cost_of(c192, rounds_of(c192, n / 192), n / 192 / 256.0));
        if (const int big = tall_mixed_cols(n); big > 0) {
            const double whole = big / 256, low = rounds_of(c128, (n - big * 192) / 128) * (c128.step * steps + c128.per_tile) / (c192.step * steps + c192.per_tile);
            best = std::min(best, cost_of(c192, whole + low, n / 192.0 / 256.0));
        }
    }
    return best;
}

// Tile shape and split-K factor (a divisor of the k-steps from min_splits to max_splits) of the lowest cost.  Up to 64 rows the
// product is a stream of the weights and tile 7 the only candidate.  A result plane is read back by the next kernel, so a product that is
// split less is worth the time of that.
GemmPlan cheapest(int m, int n, int k, int mode, int min_splits, int max_splits, bool row_mixed) {
    const int its = k / BK;
    GemmPlan best{0, min_splits};
    double best_cost = 1e30;
    if (mode != GEMM_STORE_F32) max_splits = 1;
    for (int s = min_splits; s <= std::max(min_splits, std::min(max_splits, its / 8)); ++s) {  // (at least 8 k-steps a share)
        if (its % s != 0) continue;
        const double steps = (double)its / s;
        const double plane = plane_us(m, n, mode, s);
        if (m <= 64 && n % 128 == 0) {
            const double cost = skinny_us(skinny_columns(m, n, k, mode, s) == 64 ? kCostSkinny64[m > 32] : kCostSkinny128[m > 32], m, n, k, mode, s);
            if (cost < best_cost) { best_cost = cost; best = GemmPlan{7, s}; }
            continue;
        }
        auto round_us = [&](const TileCost& c) { return c.step * steps + c.per_tile; };
        // `rounds` as they count, `full` if the last one were as good as the others
        auto consider_rounds = [&](int tile, const TileCost& c, double rounds, double full) {
            const double cost = launch_us(c, m, n, k, steps, plane, rounds, full);
            if (cost < best_cost) { best_cost = cost; best = GemmPlan{tile, s}; }
        };
        auto consider = [&](int tile, const TileCost& c, double tiles) {
            consider_rounds(tile, c, rounds_of(c, tiles * s), tiles * s / c.slots);
        };
        const int height = gemm_band_height(m, mode);
        const double bands = (double)ceil_div(m, height), b128 = (double)ceil_div(m, 128), b256 = (double)ceil_div(m, 256);
        if (n % 256 == 0) {
            const double cols = n / 256;
            if (row_mixed && m > 384 && gemm_rowmix_rem_rows(m, n) > 0) {
                const TileCost& c = wide_cost_of(256);
                const double big = (double)(m / 256) * cols * s, low = cols * s, work = (big + kLowShare * low) / c.slots;
                consider_rounds(8, c, counted_rounds(c, rowmix_span(big, low), work), work);
            }
            if (s == 1 && gemm_mixed_rem_cols(m, n) > 0) {  // whole rounds of big tiles and one of half-width ones
                const int h = mode == GEMM_ADD_F32 ? 256 : band_height(m, (int)b256);
                const TileCost &big = wide_cost_of(h), &low = narrow_cost_of(h);
                const double tiles = b256 * cols, whole = std::floor(tiles / 256), half = rounds_of(low, 2 * (tiles - whole * 256));
                consider_rounds(4, big, whole + half * round_us(low) / round_us(big), tiles / 256);
            }
            consider(3, wide_cost_of(256), b256 * cols);
            if (height < 256) consider(14, wide_cost_of(height), bands * cols);
        }
        if (n % 192 == 0 && mode != GEMM_SWIGLU_BF16) {
            consider(5, kCost256x192, b256 * (n / 192));
            if (m > 256 && m <= 288 && n % 128 != 0) consider(9, kCost288x192, n / 192);
        }
        if (n % 128 == 0) {
            const double cols = n / 128;
            consider(15, narrow_cost_of(height), bands * cols);
            // as few bands as cover the rows, where those of equal height are one more (600 rows of 5120 x 5120: 47 -> 41 us)
            const int h1 = gemm_low_bands(m) ? 192 : 256;
            if (h1 != height) consider(1, narrow_cost_of(h1), (double)ceil_div(m, h1) * cols);
            if (m > 256 && m <= 288 && mode == GEMM_STORE_F32) {
                const double us = tall_us(m, n, k, s);
                if (us < best_cost) { best_cost = us; best = GemmPlan{13, s}; }
            } else if (m > 256 && m <= 384 && mode != GEMM_ADD_F32) consider(13, kCostTall[(m - 257) / 32], cols);
            if (mode == GEMM_STORE_F32 && half_width_deep(m, n, s)) consider(6, kCost128x64Deep, 2 * cols);
            else consider(6, kCost128x128Deep, b128 * cols);
            consider(0, kCost128x128, b128 * cols);
        }
    }
    return best;
}

}  // namespace

GemmPlan gemm_plan(int m, int n, int k, int mode, int max_splits, bool row_mixed) {
    return cheapest(m, n, k, mode, 1, max_splits, row_mixed);
}

namespace {

// Whether launches of this tile id cover a product of these sizes (the rule is the same whatever path addresses it).
bool tile_fits(int tile, int m, int n, int mode, int splits) {
    switch (tile) {
        case 0: case 1: case 6: case 7: return n % 128 == 0;
        case 2: case 3: case 10: return n % 256 == 0;
        case 4: case 11: return splits == 1 && gemm_mixed_rem_cols(m, n) > 0;
        case 5: return n % 192 == 0 && mode != GEMM_SWIGLU_BF16;
        case 8: case 12: return gemm_rowmix_rem_rows(m, n) > 0;
        case 9: return m > 256 && m <= 288 && n % 192 == 0 && mode != GEMM_SWIGLU_BF16;
        case 13: return m > 256 && m <= 384 && n % 128 == 0;
        case 14: return n % 256 == 0;
        case 15: return n % 128 == 0;
        default: return false;
    }
}

}  // namespace

int gemm_tile_columns(int m, int n, int k, int mode, int tile, int splits) {
    if (!tile_fits(tile, m, n, mode, splits)) return -1;
    if (tile == 9 && n % 128 == 0 && mode != GEMM_ADD_F32) tile = 13;
    const bool store = mode == GEMM_STORE_F32;
    switch (tile) {
        case 0: case 1: case 15: return 128;
        case 5: case 9: return 192;
        case 4: case 11: return 0;
        case 6: return store && half_width_deep(m, n, splits) ? 64 : 128;
        case 7: return store && m <= 64 ? skinny_columns(m, n, k, mode, splits) : 128;
        case 13: {
            const Tall form = store ? tall_form(m, n, splits) : Tall::k128;
            return form == Tall::k192 ? 192 : form == Tall::kMixed ? 0 : 128;
        }
        default: return 256;
    }
}

hipError_t launch_gemm_bf16(const bf16_t* a, int64_t lda, const bf16_t* w, int64_t ldw, void* out, int64_t ldc,
                            int m, int n, int k, int mode, int tile, int splits, int64_t split_stride,
                            hipStream_t stream) {
    if (m <= 0) return hipSuccess;
    if (n <= 0 || k <= 0 || n % 64 != 0 || k % BK != 0) return hipErrorInvalidValue;
    if (lda * 16 >= (int64_t)1 << 31 || ldw % kWBlock != 0 || ldw < k) return hipErrorInvalidValue;
    if (splits < 1 || (k / BK) % splits != 0) return hipErrorInvalidValue;
    if (splits > 1 && mode != GEMM_STORE_F32) return hipErrorInvalidValue;
    if (tile < 0) {
        tile = cheapest(m, n, k, splits == 1 ? mode : GEMM_STORE_F32, splits, splits, true).tile;
    }
    if (!tile_fits(tile, m, n, mode, splits)) return hipErrorInvalidValue;
    if (tile == 9 && n % 128 == 0 && mode != GEMM_ADD_F32) tile = 13;
    if ((((uintptr_t)a | (uintptr_t)w) & 3) || (m > 1 && lda % 2 != 0)) {
        const int cols = mode == GEMM_SWIGLU_BF16 ? n / 2 : n;
        const int64_t blocks = ceil_div((int64_t)m * cols, 256);
        if (blocks > 0x7FFFFFFF) return hipErrorInvalidValue;
        const dim3 grid((unsigned)blocks, splits);
        if (mode == GEMM_STORE_F32) gemm_any_address_kernel<GEMM_STORE_F32><<<grid, 256, 0, stream>>>(a, lda, w, ldw, out, ldc, m, cols, k, split_stride);
        else if (mode == GEMM_ADD_F32) gemm_any_address_kernel<GEMM_ADD_F32><<<grid, 256, 0, stream>>>(a, lda, w, ldw, out, ldc, m, cols, k, split_stride);
        else if (mode == GEMM_SWIGLU_BF16) gemm_any_address_kernel<GEMM_SWIGLU_BF16><<<grid, 256, 0, stream>>>(a, lda, w, ldw, out, ldc, m, cols, k, split_stride);
        else return hipErrorInvalidValue;
        return hipGetLastError();
    }
    // the kernels address the rows of a tile by 32-bit byte offsets: rows too far apart for that are multiplied in bands of
    // fewer rows, each with the tile the planner picks for it (a forced one need not fit a band)
    const int64_t rows32 = (((int64_t)1 << 32) - 1) / (2 * std::max<int64_t>(lda, 1));
    if (m > rows32 && rows32 < kMaxTileM) {
        const int elem = mode == GEMM_SWIGLU_BF16 ? 2 : 4;
        for (int64_t r = 0; r < m; r += rows32) {
            const hipError_t e = launch_gemm_bf16(a + r * lda, lda, w, ldw, (char*)out + r * ldc * elem, ldc, (int)std::min<int64_t>(rows32, m - r),
                                                  n, k, mode, -1, splits, split_stride, stream);
            if (e != hipSuccess) return e;
        }
        return hipSuccess;
    }
    if (ldw >= (int64_t)1 << 23) {  // (256 columns of W, the widest tile, are 4 GiB)
        switch (mode) {
            case GEMM_STORE_F32: return launch_far<GEMM_STORE_F32>(a, lda, w, ldw, out, ldc, m, n, k, splits, split_stride, stream);
            case GEMM_ADD_F32: return launch_far<GEMM_ADD_F32>(a, lda, w, ldw, out, ldc, m, n, k, splits, split_stride, stream);
            case GEMM_SWIGLU_BF16: return launch_far<GEMM_SWIGLU_BF16>(a, lda, w, ldw, out, ldc, m, n, k, splits, split_stride, stream);
            default: return hipErrorInvalidValue;
        }
    }
    if (tile == 8 || tile == 12) {
        if (m > 384) {  // up to 384 rows: two bands of 192, see launch_mode
            const int rem_rows = gemm_rowmix_rem_rows(m, n);
#define GLLM_ROWMIX_MODE(MODE_)                                                                                              \
    (rem_rows == 64 ? launch_rowmix<MODE_, 64>(a, lda, w, ldw, out, ldc, m, n, k, splits, split_stride, stream)              \
                    : launch_rowmix<MODE_, 128>(a, lda, w, ldw, out, ldc, m, n, k, splits, split_stride, stream))
            switch (mode) {
                case GEMM_STORE_F32: return GLLM_ROWMIX_MODE(GEMM_STORE_F32);
                case GEMM_ADD_F32: return GLLM_ROWMIX_MODE(GEMM_ADD_F32);
                case GEMM_SWIGLU_BF16: return GLLM_ROWMIX_MODE(GEMM_SWIGLU_BF16);
                default: return hipErrorInvalidValue;
            }
#undef GLLM_ROWMIX_MODE
        }
    }
    if (tile == 4 || tile == 11) {
        const int rem_cols = gemm_mixed_rem_cols(m, n);
        switch (mode) {
            case GEMM_STORE_F32: return launch_mixed<GEMM_STORE_F32>(a, lda, w, ldw, out, ldc, m, n, k, rem_cols, stream);
            case GEMM_ADD_F32: return launch_mixed<GEMM_ADD_F32>(a, lda, w, ldw, out, ldc, m, n, k, rem_cols, stream);
            case GEMM_SWIGLU_BF16: return launch_mixed<GEMM_SWIGLU_BF16>(a, lda, w, ldw, out, ldc, m, n, k, rem_cols, stream);
            default: return hipErrorInvalidValue;
        }
    }
    switch (mode) {
        case GEMM_STORE_F32:
            return launch_mode<GEMM_STORE_F32>(a, lda, w, ldw, out, ldc, m, n, k, tile, splits, split_stride, stream);
        case GEMM_ADD_F32:
            return launch_mode<GEMM_ADD_F32>(a, lda, w, ldw, out, ldc, m, n, k, tile, splits, split_stride, stream);
        case GEMM_SWIGLU_BF16:
            return launch_mode<GEMM_SWIGLU_BF16>(a, lda, w, ldw, out, ldc, m, n, k, tile, splits, split_stride, stream);
        default: return hipErrorInvalidValue;
    }
}
