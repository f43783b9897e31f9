// Ragged paged attention for decode rows and prefill chunks on the CDNA4 matrix cores.
//
// Both kernels run the same inner step on a block of 32 keys (two pages) and one or more groups
// of 16 "columns" (for a decode row: the query heads that share a KV head; for a prefill chunk:
// 16 consecutive query rows of one head), in transposed form so that nothing has to be moved
// between lanes:
//     S^T[key][col]  = K[key][:] . Q[col][:]          two 16x16x32 MFMA chains (16 of the 32 keys each)
//     O^T[dim][col] += V^T[dim][key] . P^T[key][col]  one 16x16x32 MFMA per 16 dims
// A 16x16x32 MFMA takes, per lane (r = lane % 16, G = lane / 16), 8 consecutive k-values of row r
// (A operand) or column r (B operand), k-slots 8G..8G+7, and returns for column r the rows
// 4G..4G+3.  The 4 + 4 results a lane holds for its column are the 8 k-slots 8G..8G+7 it must supply as the B operand of
// the P.V product: which keys they are is a matter of how the keys are dealt to the rows of the two S^T tiles, as long as
// the V operand holds the same ones.
//   prefill (operands from LDS): 8 consecutive keys 8G..8G+7 of the block (tile t, row i = slot 8((i>>2)&1) + 4t + (i&3)
//     of page i>>3), so V is one 16-byte piece, slots 8(G&1)..+7 of dim 16b + r of page G>>1 in the V page [d][16 slots];
//   decode (operands from HBM): tile t is page t, so every load instruction takes whole lines of the K page
//     [d/8][16 slots][8], and V is two 8-byte pieces, slots 4G..4G+3 of dim 16b + r of either page.
// Softmax is the running-reference form in base 2 (exponent s*log2(e)/sqrt(d) - m, see update_group);
// all reductions follow logical key order, so the result does not depend on which physical pages
// hold the keys.
#include "common.h"

#include <type_traits>
#include <utility>

namespace {

constexpr float kNegBig = -1.0e30f;

// K and V operands of one block of 32 keys (two pages) for a decode row.  Score tile t is page t, so a lane of group G ends
// up with keys 4G .. 4G+3 of either page, and its V operand is those slots of both.
template <int D>
struct KvFrag {
    u32x4 k[2][D / 32];  // [page][k-step]: operand row r = slot r
    u32x4 v[D / 16];     // [16-dim block]: slots 4G .. 4G+3 of dim r, first page in the low half
};

// Every instruction takes whole 128-byte lines: with lane groups owning 8 consecutive keys (as in the prefill kernel) a
// K line is split over two instructions, and a line loaded with the non-temporal hint is fetched for each (4 % more
// traffic: 512 rows of 1024 .. 8192 keys, 3 layers 4313 -> 4216 us; 251 rows of 64 .. 1100 keys, 8 layers 2224 -> 2182 us).
// The hint itself: a decode row's K and V are read once and never again, and without it the stream is allocated in the
// caches on its way (5.78 -> 6.20 TB/s on 256 rows of 512 .. 4096 keys; a bare streaming read without the hint sustains
// 5.9 - 6.2, with it 6.5).
template <int D>
__device__ __forceinline__ void load_kv(KvFrag<D>& f, const bf16_t* __restrict__ kp, const bf16_t* __restrict__ vp,
                                        int64_t page0, int64_t page1, int n_kv, int kvh, int lane) {
    constexpr int64_t PH = (int64_t)D * kPage;  // elements of one (page, head)
    const int r = lane & 15, G = lane >> 4;
    // K page layout [d/8 groups][16 slots][8]: 16 bytes per (group, slot); V page layout [d][16 slots]
    const bf16_t* k0 = kp + (page0 * n_kv + kvh) * PH + (G * kPage + r) * 8;
    const bf16_t* k1 = kp + (page1 * n_kv + kvh) * PH + (G * kPage + r) * 8;
    const bf16_t* v0 = vp + (page0 * n_kv + kvh) * PH + r * kPage + G * 4;
    const bf16_t* v1 = vp + (page1 * n_kv + kvh) * PH + r * kPage + G * 4;
#pragma unroll
    for (int s = 0; s < D / 32; ++s) {
        f.k[0][s] = __builtin_nontemporal_load(reinterpret_cast<const u32x4*>(k0 + s * 512));
        f.k[1][s] = __builtin_nontemporal_load(reinterpret_cast<const u32x4*>(k1 + s * 512));
    }
#pragma unroll
    for (int b = 0; b < D / 16; ++b) {
        const u32x2 lo = __builtin_nontemporal_load(reinterpret_cast<const u32x2*>(v0 + b * 256));
        const u32x2 hi = __builtin_nontemporal_load(reinterpret_cast<const u32x2*>(v1 + b * 256));
        f.v[b] = u32x4{lo[0], lo[1], hi[0], hi[1]};
    }
}

// State of NB column groups across the key loop.
template <int D, int NB>
struct AttnState {
    f32x4 o[NB][D / 16];
    float m[NB];
    float l[NB];
};

// Masks the V fragments of keys >= valid_end (slots that hold no data yet may contain any bit pattern,
// also NaN, and 0 * NaN would poison the P.V product).  v[b] holds this lane's keys key0 .. key0+3 and key1 .. key1+3 of
// dims block b, two per register.
template <int D>
__device__ __forceinline__ void mask_unwritten_v(u32x4 (&v)[D / 16], int key0, int key1, int valid_end) {
    uint32_t m[4];
#pragma unroll
    for (int w = 0; w < 4; ++w) {
        const int nv = valid_end - ((w < 2 ? key0 : key1) + 2 * (w & 1));
        m[w] = nv >= 2 ? 0xFFFFFFFFu : (nv == 1 ? 0x0000FFFFu : 0u);
    }
#pragma unroll
    for (int b = 0; b < D / 16; ++b)
#pragma unroll
        for (int w = 0; w < 4; ++w) v[b][w] &= m[w];
}

// One column group against one block of 32 keys, in two phases so that callers
// can fetch the V fragments only after the K fragments are dead.
// Phase 1: raw scores q.k of this lane's 8 keys (not yet scaled).  Lane group G receives rows 4G .. 4G+3 of both operand
// fragments; the caller's choice of the keys in those rows decides which keys these are (key0 .. key0+3 from fragment 0,
// key1 .. key1+3 from fragment 1), and the V operand of the P.V product has to hold the same ones.
template <int D>
__device__ __forceinline__ void score_group(float (&sc)[8], const u32x4 (&kf)[2][D / 32], const bf16x8 (&qf)[D / 32]) {
    f32x4 s0 = {0.f, 0.f, 0.f, 0.f}, s1 = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int s = 0; s < D / 32; ++s) {
        s0 = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, kf[0][s]), qf[s], s0, 0, 0, 0);
        s1 = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, kf[1][s]), qf[s], s1, 0, 0, 0);
    }
#pragma unroll
    for (int v = 0; v < 4; ++v) {
        sc[v] = s0[v];
        sc[4 + v] = s1[v];
    }
}
// Scores of keys past `limit` (the last key visible to this lane's column) become a huge negative.
__device__ __forceinline__ void mask_scores(float (&sc)[8], int key0, int key1, int limit) {
#pragma unroll
    for (int v = 0; v < 4; ++v) {
        if (key0 + v > limit) sc[v] = kNegBig;
        if (key1 + v > limit) sc[4 + v] = kNegBig;
    }
}

// Phase 2, for all NB column groups of a wave at once: softmax update in base 2 and O^T += V^T P^T.
//
// m is the reference exponent of a column (identical in the four lanes that share the column); p =
// 2^(s*c - m) with c = log2(e)/sqrt(d).  Softmax does not care which reference is used as long as nothing
// overflows.  DEFER = true lets the reference lag: it is only moved (to the exact running maximum: two
// cross-lane exchanges per group, then m, l and the accumulators are rescaled) when some lane sees a score
// more than 64 above it -- always in a wave's first block, where the reference is still the huge negative
// start value, and practically never afterwards -- so p stays below 2^64, sums of 2^13 of them stay finite,
// and the common path has no cross-lane traffic and no rescaling at all: a lane-local maximum, one wave vote,
// the exponentials, the MFMAs.  DEFER = false moves the reference whenever a lane's maximum exceeds it (the
// textbook order): the memory-bound decode kernel, with one group per wave, gains nothing from deferring.
constexpr float kRefSlack = 64.0f;

// issue_v() is called before the exponentials (a caller that fetches V from LDS starts its reads there),
// get_v() after them (it returns the fragments, waiting for them if need be).
template <int D, int NB, bool DEFER, typename IssueV, typename GetV>
__device__ __forceinline__ void update_groups(AttnState<D, NB>& st, const float (&sc)[NB][8], float scale_log2,
                                              IssueV&& issue_v, GetV&& get_v) {
    float lm[NB];
    bool low = false;
#pragma unroll
    for (int c = 0; c < NB; ++c) {
        float x = sc[c][0];
#pragma unroll
        for (int v = 1; v < 8; ++v) x = fmaxf(x, sc[c][v]);
        lm[c] = x * scale_log2;
        low |= DEFER ? lm[c] > st.m[c] + kRefSlack : lm[c] > st.m[c];
    }
    if (__any(low)) {  // wave-uniform
#pragma unroll
        for (int c = 0; c < NB; ++c) {
            float bm = fmaxf(lm[c], __shfl_xor(lm[c], 16));
            bm = fmaxf(bm, __shfl_xor(bm, 32));
            const float m_new = fmaxf(st.m[c], bm);
            const float alpha = __builtin_amdgcn_exp2f(st.m[c] - m_new);
            st.l[c] *= alpha;
#pragma unroll
            for (int b = 0; b < D / 16; ++b)
#pragma unroll
                for (int v = 0; v < 4; ++v) st.o[c][b][v] *= alpha;
            st.m[c] = m_new;
        }
    }
    issue_v();
    bf16x8 pb[NB];
#pragma unroll
    for (int c = 0; c < NB; ++c) {
        f32x8 p;
        float psum = 0.f;
#pragma unroll
        for (int v = 0; v < 8; ++v) {
            p[v] = __builtin_amdgcn_exp2f(fmaf(sc[c][v], scale_log2, -st.m[c]));
            psum += p[v];
        }
        st.l[c] += psum;
        pb[c] = __builtin_convertvector(p, bf16x8);
    }
    const u32x4 (&vf)[D / 16] = get_v();
#pragma unroll
    for (int b = 0; b < D / 16; ++b)
#pragma unroll
        for (int c = 0; c < NB; ++c)
            st.o[c][b] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, vf[b]), pb[c], st.o[c][b], 0, 0, 0);
}

// One block of 32 keys for NB column groups, K/V fragments in registers.
//   limit[c]   : last key visible to this lane's column in group c
//   valid_end  : keys >= valid_end hold no data yet
template <int D, int NB>
__device__ __forceinline__ void attend_block(AttnState<D, NB>& st, KvFrag<D>& f, const bf16x8 (&qf)[NB][D / 32],
                                             int tb, const int (&limit)[NB], int min_limit, int valid_end,
                                             float scale_log2, int lane) {
    const int key0 = tb + (lane >> 4) * 4, key1 = key0 + kPage;
    if (tb + 32 > valid_end) mask_unwritten_v<D>(f.v, key0, key1, valid_end);  // wave-uniform
    const bool need_mask = tb + 31 > min_limit;                                // wave-uniform
    float sc[NB][8];
#pragma unroll
    for (int c = 0; c < NB; ++c) {
        score_group<D>(sc[c], f.k, qf[c]);
        if (need_mask) mask_scores(sc[c], key0, key1, limit[c]);
    }
    update_groups<D, NB, false>(st, sc, scale_log2, []() {}, [&]() -> const u32x4 (&)[D / 16] { return f.v; });
}

// Walks key blocks [blk_begin, blk_end) (units of 32 keys) of one sequence.  Page ids are fetched 64
// at a time, one per lane, and handed out with readlane.  last_page is the last page index of the
// sequence that holds keys to be read, and no page id past it is taken from the table; page0 and page1 are the ids of the first
// block's pages, so that its loads need not wait for the table.  (page1 may be the page behind last_page that the new token starts,
// which the same launch then writes: what is read there is masked, like all keys from valid_end on.)
// prepare() fills qf; every wave calls it once, when the loads of its first block are on their way.
template <int D, int NB, typename Prepare>
__device__ __forceinline__ void attend_range(AttnState<D, NB>& st, const bf16x8 (&qf)[NB][D / 32],
                                             const bf16_t* __restrict__ kp, const bf16_t* __restrict__ vp,
                                             const int32_t* __restrict__ bt, int blk_begin, int blk_end, int page0, int page1,
                                             int last_page, const int (&limit)[NB], int min_limit, int valid_end,
                                             int n_kv, int kvh, float scale_log2, int lane, Prepare&& prepare) {
    if (blk_begin >= blk_end) {
        prepare();
        return;
    }
    int ids_base = blk_begin * 2;  // page index held by lane 0
    int ids = bt[min(ids_base + lane, last_page)];
    auto page_of = [&](int pi) -> int64_t {  // pi wave-uniform, within [ids_base, ids_base + 64)
        return (int64_t)__builtin_amdgcn_readlane(ids, pi - ids_base);
    };
    auto load_block = [&](KvFrag<D>& f, int blk) {
        int p0 = min(blk * 2, last_page), p1 = min(blk * 2 + 1, last_page);
        load_kv<D>(f, kp, vp, page_of(p0), page_of(p1), n_kv, kvh, lane);
    };
    KvFrag<D> fa, fb;
    load_kv<D>(fa, kp, vp, page0, page1, n_kv, kvh, lane);
    prepare();
    for (int blk = blk_begin; blk < blk_end; blk += 2) {
        // blocks blk and blk+1 use pages 2blk .. 2blk+3; refill the id window when it runs out
        const bool has_b = blk + 1 < blk_end;
        if (has_b) load_block(fb, blk + 1);
        attend_block<D, NB>(st, fa, qf, blk * 32, limit, min_limit, valid_end, scale_log2, lane);
        if (blk + 2 < blk_end) {
            if ((blk + 2) * 2 + 3 >= ids_base + 64) {
                ids_base = (blk + 2) * 2;
                ids = bt[min(ids_base + lane, last_page)];
            }
            load_block(fa, blk + 2);
        }
        if (has_b) attend_block<D, NB>(st, fb, qf, (blk + 1) * 32, limit, min_limit, valid_end, scale_log2, lane);
    }
}

template <int D, int NB>
__device__ __forceinline__ void init_state(AttnState<D, NB>& st) {
#pragma unroll
    for (int c = 0; c < NB; ++c) {
        st.m[c] = kNegBig;
        st.l[c] = 0.f;
#pragma unroll
        for (int b = 0; b < D / 16; ++b) st.o[c][b] = f32x4{0.f, 0.f, 0.f, 0.f};
    }
}

// ------------------------------------------------------------------------------------------
// Decode: one workgroup of 4 waves per (item, kv head).  The item's key partition is cut into four runs of
// 32-key blocks, one per wave; the waves' partial results are merged through LDS and written as
// one partial (running max, sum, unnormalised output) per query head of the KV head.
//
// FROM_QKV (batches of decode rows only): the queries and the row's new key and value come straight from the QKV projection.
// Every workgroup of a row sums the split-K planes of its heads and rotates (a few KiB from the caches, under the latency of
// the first keys); the one that owns the last position takes the new token as a fifth partial beside those of its waves (its
// score, weight 1, its value), so nothing waits for the pool.  Workgroups of their own, one per row, write the new keys and
// values there (write_new_token).  Against a RoPE kernel of its own in front: 64 rows of 1500 .. 3500 keys, eight layers, 1676
// -> 1656 us, 512 rows of 1024 .. 8192 keys, three layers, 4203 -> 4170.
constexpr int kMaxGroup = 16;  // query heads per KV head
template <int D, bool FROM_QKV>
struct DecodeLds {
    float o[4][16][D + 4];
    float m[4][16], l[4][16];
};
template <int D>
struct DecodeLds<D, true> : DecodeLds<D, false> {
    float s_new[16];  // score of the new token per query head
    __attribute__((aligned(16))) float sum[kMaxGroup + 2][D + 4];  // q heads of the group, k, v: summed planes (rows shifted by a bank group)
};

// The four columns e .. e+3 of head row h of the group (h = g: the key, g + 1: the value): all planes, not yet summed.
template <int D>
__device__ __forceinline__ int64_t qkv_column(const RopeKvArgs& r, int kvh, int g, int i) {
    const int h = i / (D / 4), e = i % (D / 4) * 4;
    return (int64_t)(h < g ? kvh * g + h : h == g ? r.n_q + kvh : r.n_q + r.n_kv + kvh) * D + e;
}
__device__ __forceinline__ void load_planes(f32x4 (&part)[kMaxPlanes], const RopeKvArgs& r, const float* __restrict__ at) {
#pragma unroll
    for (int p = 0; p < kMaxPlanes; ++p)
        if (p < r.planes) part[p] = *reinterpret_cast<const f32x4*>(at + p * r.plane_stride);
}
__device__ __forceinline__ f32x4 sum_planes(const f32x4 (&part)[kMaxPlanes], const RopeKvArgs& r, int64_t col) {
    f32x4 v = part[0];
#pragma unroll
    for (int p = 1; p < kMaxPlanes; ++p)
        if (p < r.planes) v += part[p];
    if (r.bias) v += __builtin_convertvector(*reinterpret_cast<const bf16x4*>(r.bias + col), f32x4);
    return v;
}

template <int D, bool FROM_QKV>
__device__ __forceinline__ void decode_workgroup(const AttnArgs& a, const DecodeArgs& dec, int wg, DecodeLds<D, FROM_QKV>& lds) {
    const DecodeItem* __restrict__ items = dec.items;
    float* __restrict__ part_o = a.part_o;
    float* __restrict__ part_ml = a.part_ml;
    // the KV heads of one item are neighbouring workgroups: they run at the same time and read
    // neighbouring 4 KiB pieces of the same pages
    const int kvh = wg % a.n_kv;
    // (the items lie in launch order and name the pages of each wave's first block: keys are asked for after one trip to memory, not
    // three -- order, item, page table.  Share of the batch's time, five runs of each side: 200 rows of 16 .. 600 keys 0.991 to 0.995, 500
    // of 16 .. 100 0.993, long rows 0.998 to 0.999, 32 rows of 100 .. 300 1.004)
    const DecodeItem& item = items[wg / a.n_kv];
    const DecodeItem it = item;
    const int g = a.n_q / a.n_kv;
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int r = lane & 15, G = lane >> 4;
    const int page0 = item.first_pages[wave][0], page1 = item.first_pages[wave][1];

    bf16x8 qf[1][D / 32];
    f32x4 part[kMaxPlanes], cs[D / 64][4];
    const int pieces = (g + 2) * (D / 4);  // of four columns: one per thread and pass
    const RopeKvArgs& rp = dec.rope;
    const float* qkv_row = nullptr;
    const f32x4* cs_row = nullptr;
    if constexpr (FROM_QKV) {
        qkv_row = rp.qkv + (int64_t)it.row * rp.ld_qkv;
        cs_row = reinterpret_cast<const f32x4*>(rp.rope_cs + (int64_t)it.pos * D);
        if ((int)threadIdx.x < pieces) load_planes(part, rp, qkv_row + qkv_column<D>(rp, kvh, g, threadIdx.x));
#pragma unroll
        for (int s = 0; s < D / 64; ++s)
#pragma unroll
            for (int i = 0; i < 4; ++i) cs[s][i] = cs_row[(s * 4 + G) * 4 + i];
        __builtin_amdgcn_sched_barrier(0);  // these loads go first: they come from the caches, the keys behind them from HBM
    } else {
        const bf16_t* qrow = a.q + (int64_t)it.row * a.ld_q + (int64_t)(kvh * g + r) * D;
#pragma unroll
        for (int s = 0; s < D / 32; ++s) {
            u32x4 z = {0u, 0u, 0u, 0u};
            if (r < g) z = *reinterpret_cast<const u32x4*>(qrow + (s * 4 + G) * 8);
            qf[0][s] = __builtin_bit_cast(bf16x8, z);
        }
    }
    const bool owns_new = FROM_QKV && it.kv_end == it.pos + 1;  // (the same for all threads)
    const int kv_end = owns_new ? it.pos : it.kv_end;           // keys to be read from the pool
    auto prepare = [&]() {
        if constexpr (FROM_QKV) {
            for (int i = threadIdx.x; i < pieces; i += 256) {
                const int64_t col = qkv_column<D>(rp, kvh, g, i);
                if (i >= 256) load_planes(part, rp, qkv_row + col);
                *reinterpret_cast<f32x4*>(&lds.sum[i / (D / 4)][i % (D / 4) * 4]) = sum_planes(part, rp, col);
            }
            __syncthreads();
            const int h = min(r, g - 1);
#pragma unroll
            for (int s = 0; s < D / 64; ++s) {  // dims (s*4+G)*8 .. +7 and their partners D/2 further
                bf16x4 lo[2], hi[2];
#pragma unroll
                for (int i = 0; i < 2; ++i) {
                    const int e = (s * 4 + G) * 8 + i * 4;
                    rope_rotate(*reinterpret_cast<const f32x4*>(&lds.sum[h][e]), *reinterpret_cast<const f32x4*>(&lds.sum[h][e + D / 2]),
                                cs[s][2 * i], cs[s][2 * i + 1], lo[i], hi[i]);
                }
                bf16x8 ql = __builtin_shufflevector(lo[0], lo[1], 0, 1, 2, 3, 4, 5, 6, 7), qh = __builtin_shufflevector(hi[0], hi[1], 0, 1, 2, 3, 4, 5, 6, 7);
                const u32x4 zero = {0u, 0u, 0u, 0u};
                qf[0][s] = r < g ? ql : __builtin_bit_cast(bf16x8, zero);
                qf[0][s + D / 64] = r < g ? qh : __builtin_bit_cast(bf16x8, zero);
            }
            if (owns_new) {  // the score of the new token: this lane's dims of key and queries, then the sum over the lane groups
                float dot = 0.f;
#pragma unroll
                for (int s = 0; s < D / 64; ++s) {
                    bf16x4 lo[2], hi[2];
#pragma unroll
                    for (int i = 0; i < 2; ++i) {
                        const int e = (s * 4 + G) * 8 + i * 4;
                        rope_rotate(*reinterpret_cast<const f32x4*>(&lds.sum[g][e]), *reinterpret_cast<const f32x4*>(&lds.sum[g][e + D / 2]),
                                    cs[s][2 * i], cs[s][2 * i + 1], lo[i], hi[i]);
#pragma unroll
                        for (int v = 0; v < 4; ++v)
                            dot += (float)lo[i][v] * (float)qf[0][s][i * 4 + v] + (float)hi[i][v] * (float)qf[0][s + D / 64][i * 4 + v];
                    }
                }
                dot += __shfl_xor(dot, 16);
                dot += __shfl_xor(dot, 32);
                if (wave == 0 && G == 0) lds.s_new[r] = dot * a.scale_log2;
            }
        }
    };
    const int blk0 = it.kv_begin / 32;
    const int nblk = (kv_end - it.kv_begin + 31) / 32;  // (one less than the item's where the new token starts a block)
    const int b_begin = blk0 + decode_wave_first(it, wave);
    const int b_end = blk0 + min(decode_wave_first(it, wave + 1), nblk);
    const int limit[1] = {kv_end - 1};
    AttnState<D, 1> st;
    init_state<D, 1>(st);
    attend_range<D, 1>(st, qf, a.k_pool, a.v_pool, a.bt_flat + it.bt_off, b_begin, b_end, page0, page1, (kv_end - 1) / kPage,
                       limit, kv_end - 1, kv_end, a.n_kv, kvh, a.scale_log2, lane, prepare);
    float l = st.l[0];
    l += __shfl_xor(l, 16);
    l += __shfl_xor(l, 32);
    if (G == 0) {
        lds.m[wave][r] = st.m[0];
        lds.l[wave][r] = l;
    }
#pragma unroll
    for (int b = 0; b < D / 16; ++b)
        *reinterpret_cast<f32x4*>(&lds.o[wave][r][b * 16 + G * 4]) = st.o[0][b];
    __syncthreads();
    // merge: thread -> (head j, 4-dim group)
    for (int idx = threadIdx.x; idx < g * (D / 4); idx += 256) {
        const int j = idx / (D / 4), e = (idx % (D / 4)) * 4;
        float mw[4], ms = kNegBig;
        if constexpr (FROM_QKV) {
            if (owns_new) ms = lds.s_new[j];
        }
#pragma unroll
        for (int w = 0; w < 4; ++w) {
            mw[w] = lds.m[w][j];
            ms = fmaxf(ms, mw[w]);
        }
        f32x4 acc = {0.f, 0.f, 0.f, 0.f};
        float ls = 0.f;
        if constexpr (FROM_QKV) {
            if (owns_new) {
                ls = __builtin_amdgcn_exp2f(lds.s_new[j] - ms);
                const bf16x4 v = __builtin_convertvector(*reinterpret_cast<const f32x4*>(&lds.sum[g + 1][e]), bf16x4);
#pragma unroll
                for (int u = 0; u < 4; ++u) acc[u] = (float)v[u] * ls;
            }
        }
#pragma unroll
        for (int w = 0; w < 4; ++w) {
            const float sc = __builtin_amdgcn_exp2f(mw[w] - ms);
            const f32x4 ov = *reinterpret_cast<const f32x4*>(&lds.o[w][j][e]);
#pragma unroll
            for (int v = 0; v < 4; ++v) acc[v] += ov[v] * sc;
            ls += lds.l[w][j] * sc;
        }
        if (it.single) {  // same arithmetic as the merge kernel applies to a row with one partial
            const float inv = 1.0f / ls;
#pragma unroll
            for (int v = 0; v < 4; ++v) acc[v] *= inv;
            *reinterpret_cast<bf16x4*>(a.out + (int64_t)it.row * a.ld_o + (kvh * g + j) * D + e) =
                __builtin_convertvector(acc, bf16x4);
            continue;
        }
        const int64_t slot = ((int64_t)it.slot * a.n_q + kvh * g + j);
        *reinterpret_cast<f32x4*>(part_o + slot * D + e) = acc;
        if (e == 0) {
            part_ml[slot * 2] = ms;
            part_ml[slot * 2 + 1] = ls;
        }
    }
}

// New key and value of token row t, all heads, into the pool: the same sums, rotation and rounding as rope_kv_write, a
// thread per four rotated pairs of K or four dims of V.
template <int D>
__device__ __forceinline__ void write_new_token(const RopeKvArgs& r, int t) {
    const int pos = r.tok_pos[t], slot = pos % kPage;
    const int64_t page = (int64_t)r.tok_page[t] * r.n_kv * (D * kPage);
    const float* row = r.qkv + (int64_t)t * r.ld_qkv;
    const f32x4* cs = reinterpret_cast<const f32x4*>(r.rope_cs + (int64_t)pos * D);
    const int k_units = r.n_kv * (D / 8), units = k_units + r.n_kv * (D / 4);
    for (int i = threadIdx.x; i < units; i += 256) {
        f32x4 part[kMaxPlanes];
        if (i < k_units) {
            const int hd = i / (D / 8), e = i % (D / 8) * 4;
            const int64_t col = (int64_t)(r.n_q + hd) * D + e;
            f32x4 part_hi[kMaxPlanes];
            load_planes(part, r, row + col);
            load_planes(part_hi, r, row + col + D / 2);
            const f32x4 c01 = cs[e / 2], c23 = cs[e / 2 + 1];
            bf16x4 lo, hi;
            rope_rotate(sum_planes(part, r, col), sum_planes(part_hi, r, col + D / 2), c01, c23, lo, hi);
            bf16_t* kb = r.k_pool + page + hd * (D * kPage) + slot * 8;
            *reinterpret_cast<bf16x4*>(kb + (e >> 3) * (kPage * 8) + (e & 7)) = lo;
            *reinterpret_cast<bf16x4*>(kb + ((e + D / 2) >> 3) * (kPage * 8) + (e & 7)) = hi;
        } else {
            const int hd = (i - k_units) / (D / 4), e = (i - k_units) % (D / 4) * 4;
            const int64_t col = (int64_t)(r.n_q + r.n_kv + hd) * D + e;
            load_planes(part, r, row + col);
            const bf16x4 v = __builtin_convertvector(sum_planes(part, r, col), bf16x4);
            bf16_t* vb = r.v_pool + page + hd * (D * kPage) + e * kPage + slot;
#pragma unroll
            for (int u = 0; u < 4; ++u) vb[u * kPage] = v[u];
        }
    }
}

// FROM_QKV: the workgroups that write the new tokens come last, into the slots that the shortest rows leave.  512 rows of 1024
// .. 8192 keys, three layers: 4170 us so, 4265 with them in front (all slots held while the memory idles), 4312 with every
// attention workgroup writing its own token (4127 without any writes: spread over the launch they break up the stream of
// reads), 4203 with a RoPE kernel before the launch.
template <int D, bool FROM_QKV>
__global__ __launch_bounds__(256, 2) void decode_attention_kernel(AttnArgs a, DecodeArgs dec) {
    __shared__ DecodeLds<D, FROM_QKV> lds;
    if constexpr (FROM_QKV) {
        const int t = (int)blockIdx.x - dec.num_items * a.n_kv;
        if (t >= 0) {
            write_new_token<D>(dec.rope, t);
            return;
        }
    }
    decode_workgroup<D, FROM_QKV>(a, dec, blockIdx.x, lds);
}

// grid (rows, query heads), D/4 threads: merges the partials of a row in partition order.
template <int D>
__global__ void decode_combine_kernel(AttnArgs a, const DecodeRow* __restrict__ rows) {
    const float* __restrict__ part_o = a.part_o;
    const float* __restrict__ part_ml = a.part_ml;
    const DecodeRow rw = rows[blockIdx.x];
    const int hq = blockIdx.y, e = threadIdx.x * 4;
    // The kernel is all latency.  Up to kFewParts partials, a row's usual number, are asked for at one time, references and sums
    // beside the outputs; of more the references are read first and then all of them, eight at a time.  Partition order either way.
    // Few against that order: one row of 2500 keys (ten partials), eight layers 736 -> 726 us, 32 chunk rows behind 6000 keys
    // 887 -> 874, 300 rows of the 14B shape behind 3000, three layers 772 -> 759; 118 partials are 1 % slower in sixteens.
    constexpr int kFewParts = 16;
    const int64_t slot0 = (int64_t)rw.first_item * a.n_q + hq, slot_step = a.n_q;
    float ms = kNegBig, ls = 0.f;
    f32x4 acc = {0.f, 0.f, 0.f, 0.f};
    if (rw.num_items <= kFewParts) {
        float m[kFewParts], l[kFewParts];
        f32x4 ov[kFewParts];
#pragma unroll
        for (int u = 0; u < kFewParts; ++u) {
            m[u] = kNegBig;
            if (u < rw.num_items) {
                const int64_t slot = slot0 + u * slot_step;
                const f32x2 ml = *reinterpret_cast<const f32x2*>(part_ml + slot * 2);
                m[u] = ml[0];
                l[u] = ml[1];
                ov[u] = *reinterpret_cast<const f32x4*>(part_o + slot * D + e);
            }
        }
#pragma unroll
        for (int u = 0; u < kFewParts; ++u) ms = fmaxf(ms, m[u]);
#pragma unroll
        for (int u = 0; u < kFewParts; ++u) {
            if (u < rw.num_items) {
                const float sc = __builtin_amdgcn_exp2f(m[u] - ms);
#pragma unroll
                for (int v = 0; v < 4; ++v) acc[v] += ov[u][v] * sc;
                ls += l[u] * sc;
            }
        }
    } else {
        constexpr int U = 8;
        for (int i0 = 0; i0 < rw.num_items; i0 += U) {
            float m[U];
#pragma unroll
            for (int u = 0; u < U; ++u) m[u] = i0 + u < rw.num_items ? part_ml[(slot0 + (i0 + u) * slot_step) * 2] : kNegBig;
#pragma unroll
            for (int u = 0; u < U; ++u) ms = fmaxf(ms, m[u]);
        }
        for (int i0 = 0; i0 < rw.num_items; i0 += U) {
            float m[U], l[U];
            f32x4 ov[U];
#pragma unroll
            for (int u = 0; u < U; ++u) {
                if (i0 + u < rw.num_items) {
                    const int64_t slot = slot0 + (i0 + u) * slot_step;
                    m[u] = part_ml[slot * 2];
                    l[u] = part_ml[slot * 2 + 1];
                    ov[u] = *reinterpret_cast<const f32x4*>(part_o + slot * D + e);
                }
            }
#pragma unroll
            for (int u = 0; u < U; ++u) {
                if (i0 + u < rw.num_items) {
                    const float sc = __builtin_amdgcn_exp2f(m[u] - ms);
#pragma unroll
                    for (int v = 0; v < 4; ++v) acc[v] += ov[u][v] * sc;
                    ls += l[u] * sc;
                }
            }
        }
    }
    const float inv = 1.0f / ls;
#pragma unroll
    for (int v = 0; v < 4; ++v) acc[v] *= inv;
    *reinterpret_cast<bf16x4*>(a.out + (int64_t)rw.row * a.ld_o + hq * D + e) = __builtin_convertvector(acc, bf16x4);
}

// One 16-byte LDS read at addr + 512*B (dims block B of a V page).  Written as assembly so that the reads can be
// issued early and awaited late: the result is valid only after await_lds().
template <int B>
__device__ __forceinline__ void read_v_operand(u32x4& v, uint32_t addr) {
    asm volatile("ds_read_b128 %0, %1 offset:%2" : "=v"(v) : "v"(addr), "n"(B * 512) : "memory");
}
template <int N, int... Bs>
__device__ __forceinline__ void read_v_operands(u32x4 (&v)[N], uint32_t addr, std::integer_sequence<int, Bs...>) {
    (read_v_operand<Bs>(v[Bs], addr), ...);
}
// Waits for all outstanding LDS reads; the registers are passed through the statement so that no use of them
// can be scheduled before it.
template <int N>
__device__ __forceinline__ void await_lds(u32x4 (&v)[N]) {
    static_assert(N % 4 == 0, "fragments are awaited four at a time");
#pragma unroll
    for (int b = 0; b < N; b += 4)
        asm volatile("s_waitcnt lgkmcnt(0)" : "+v"(v[b]), "+v"(v[b + 1]), "+v"(v[b + 2]), "+v"(v[b + 3])::"memory");
}

// ------------------------------------------------------------------------------------------
// Prefill: one workgroup of 4 waves per (item, group of HW query heads of one KV head).  An item is up
// to 64*NB/HW consecutive query rows of a chunk, so the workgroup owns 4*NB column groups of 16 (NB per wave)
// that all share the same K/V: every 32-key block is brought into LDS once (global_load_lds into a ring
// of 3 stages, two blocks in flight while one is processed: a block is only ~0.5 us of work, far less
// than the memory latency) and read by all 4 waves.
// A lane owns 8 consecutive keys of the block (the K operand rows are permuted accordingly),
// so a V operand is one 16-byte LDS read of 8 slots of one page; LDS holds the pages as the pool does, except
// that the second K page is shifted by four slots (see issue_block).
// Column group cb = NB*wave + c covers head (cb % HW) and query rows 16*(cb / HW) .. +15 of the item.
// The keys of a tile may be cut into parts, an item each: what the waves hold at the end then goes out as partial results, which
// decode_combine_kernel merges like those of decode rows.  The cuts lie where every row of the tile sees all keys, so that no
// part is wholly masked for any of them.
// ------------------------------------------------------------------------------------------
typedef const __attribute__((address_space(1))) void* gptr_t;
typedef __attribute__((address_space(3))) void* lptr_t;

constexpr int kPrefillStages = 3;
template <int D>
struct PrefillLds {
    __attribute__((aligned(1024))) unsigned char stage[kPrefillStages][4][D * kPage * 2];  // [stage][K0,K1,V0,V1]
};

template <int D, int HW, int NB>
__device__ __forceinline__ void prefill_workgroup(const AttnArgs& a, const PrefillItem* __restrict__ items, int wg, PrefillLds<D>& shared) {
    constexpr int PAGE_BYTES = D * kPage * 2;  // one (page, head) of K or of V
    constexpr int NS = kPrefillStages;
    constexpr int IPB = PAGE_BYTES / 1024;     // load instructions per wave and block
    auto& lds = shared.stage;
    const int groups = a.n_q / HW;
    const PrefillItem it = items[wg / groups];
    const int head0 = (wg % groups) * HW;
    const int kvh = head0 / (a.n_q / a.n_kv);
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int r = lane & 15, G = lane >> 4;

    // (only items of half the rows are cut; whole ones, which fill the chip, have no registers to spare for it)
    constexpr bool CUT = NB == 1;
    // Keys, pages and positions are counted from the first key of the part, so that the loop is the same as without parts (counted
    // from that of the sequence, with the first block subtracted for the ring's stage, it took 172 instead of 155 us at 512 workgroups
    // of uncut tiles).
    const int blk0 = CUT ? it.blk_begin : 0, pos0 = it.pos0 - 32 * blk0;
    bf16x8 qf[NB][D / 32];
    int limit[NB], wave_min = 0x7FFFFFFF, wave_max = -1;
#pragma unroll
    for (int c = 0; c < NB; ++c) {
        const int cb = wave * NB + c, qb = cb / HW;
        const int qi = min(qb * 16 + r, it.n_rows - 1);  // rows past the item repeat its last row (never stored)
        limit[c] = pos0 + qi;
        wave_min = min(wave_min, pos0 + min(qb * 16, it.n_rows - 1));
        wave_max = max(wave_max, pos0 + min(qb * 16 + 15, it.n_rows - 1));
        const bf16_t* qrow = a.q + (int64_t)(it.row0 + qi) * a.ld_q + (int64_t)(head0 + cb % HW) * D;
#pragma unroll
        for (int s = 0; s < D / 32; ++s)
            qf[c][s] = __builtin_bit_cast(bf16x8, *reinterpret_cast<const u32x4*>(qrow + (s * 4 + G) * 8));
    }
    const int last_pos = pos0 + it.n_rows - 1;
    const int nblk = CUT ? it.blk_end - blk0 : last_pos / 32 + 1, last_page = last_pos / kPage;
    const int32_t* bt = a.bt_flat + it.bt_off + 2 * blk0;
    // wave w brings in piece w of a block: K page 0, K page 1, V page 0, V page 1 (4 x 1 KiB per page at d=128)
    const bf16_t* pool = (wave < 2) ? a.k_pool : a.v_pool;
    auto page_id = [&](int blk) -> int { return bt[min(blk * 2 + (wave & 1), last_page)]; };
    auto issue_block = [&](int64_t page, int stage) {
        // K page 0 and the V pages are copied as they are, K page 1 with slot s at the place of slot s ^ 4.  A 16-byte
        // LDS read is served 16 lanes at a time -- measured: lanes 0-7 together with lanes 24-31, 8-15 with 16-23,
        // and likewise in the upper half of the wave -- and is free of bank conflicts when those 16 lanes hit 16
        // different 16-byte columns of the 256-byte bank line.  The K operand rows of such a group are slots
        // {0-3, 8-11} (or {4-7, 12-15}) of page 0 and of page 1: the shift by four slots separates the two pages.
        // The V operand of such a group is one half (16 bytes) of dims 0-7 and the other half of dims 8-15 of a
        // 16-dim block: 16 different columns as stored.  A lane picks the source piece for its LDS position.
        const int src_lane = wave == 1 ? lane ^ 4 : lane;
        const char* src = reinterpret_cast<const char*>(pool + (page * a.n_kv + kvh) * (int64_t)(D * kPage)) + src_lane * 16;
#pragma unroll
        for (int i = 0; i < IPB; ++i)
            __builtin_amdgcn_global_load_lds((gptr_t)(src + i * 1024), (lptr_t)(&lds[stage][wave][i * 1024]), 16, 0, 0);
    };

    AttnState<D, NB> st;
    init_state<D, NB>(st);
    auto block_step = [&](int stage, int tb, auto masked) {
        constexpr bool MASKED = decltype(masked)::value;
        float sc[NB][8];
        {
            // fragment t, row r of the operand = slot 8 ((r >> 2) & 1) + 4 t + (r & 3) of page r >> 3: lane group G gets the
            // 8 consecutive keys 8G .. 8G+7 of the block
            u32x4 kf[2][D / 32];
            const int kpage = r >> 3, kslot = ((r >> 2) & 1) * 8 + (r & 3);
#pragma unroll
            for (int t = 0; t < 2; ++t)
#pragma unroll
                for (int s = 0; s < D / 32; ++s)
                    kf[t][s] = *reinterpret_cast<const u32x4*>(
                        &lds[stage][kpage][((s * 4 + G) * 16 + ((kslot + 4 * t) ^ (4 * kpage))) * 16]);
#pragma unroll
            for (int c = 0; c < NB; ++c) {
                score_group<D>(sc[c], kf, qf[c]);
                if (MASKED) mask_scores(sc[c], tb + G * 8, tb + G * 8 + 4, limit[c]);
            }
        }
        // V^T operands: dims block b needs this lane's 8 consecutive keys of one dim: the 16 bytes of slots 0-7 or
        // 8-15 of page G >> 1.  The reads are issued before the exponentials and awaited after them.
        u32x4 vf[D / 16];
        update_groups<D, NB, true>(
            st, sc, a.scale_log2,
            [&]() {
                const uint32_t addr = (uint32_t)(uintptr_t)(&lds[stage][2 + (G >> 1)][r * 32 + (G & 1) * 16]);
                read_v_operands(vf, addr, std::make_integer_sequence<int, D / 16>{});
            },
            [&]() -> const u32x4 (&)[D / 16] {
                await_lds(vf);
                if (MASKED) mask_unwritten_v<D>(vf, tb + G * 8, tb + G * 8 + 4, last_pos + 1);
                return vf;
            });
    };
    // every wave always issues its piece (indices past the end re-read the last page into a stage nobody
    // reads), so the count of outstanding loads is the same in every iteration
#pragma unroll
    for (int i = 0; i < NS - 1; ++i) issue_block(page_id(i), i);
    int pid_next = page_id(NS - 1);  // page of block blk + NS - 1, fetched one iteration ahead
    auto ring_advance = [&](int blk) {
        // blocks blk+1 .. blk+NS-2 may still be in flight
        asm volatile("s_waitcnt vmcnt(%0)" ::"n"((NS - 2) * IPB) : "memory");
        __syncthreads();  // block blk has landed; nobody reads stage (blk-1) % NS any more
        issue_block(pid_next, (blk + NS - 1) % NS);
        pid_next = page_id(blk + NS);
    };
    // Two loops with one barrier per block each (every wave passes the same number of barriers in total): first the
    // blocks wholly visible to every row of this wave -- no masks at all, the common case -- then the
    // blocks at the causal edge / the end of the written keys (masked) and the wholly invisible ones (skipped).
    const int n_full = min((wave_min + 1) / 32, nblk);
    for (int blk = 0; blk < n_full; ++blk) {
        ring_advance(blk);
        block_step(blk % NS, blk * 32, std::false_type{});
    }
    for (int blk = n_full; blk < nblk; ++blk) {
        ring_advance(blk);
        if (blk * 32 <= wave_max) block_step(blk % NS, blk * 32, std::true_type{});
    }
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");  // no LDS fill may outlive the workgroup
#pragma unroll
    for (int c = 0; c < NB; ++c) {
        float l = st.l[c];
        l += __shfl_xor(l, 16);
        l += __shfl_xor(l, 32);
        const int cb = wave * NB + c;
        const int qi = (cb / HW) * 16 + r;
        if (CUT && qi < it.n_rows && it.parts > 1) {
            const int64_t slot = (int64_t)(it.slot0 + qi * it.parts) * a.n_q + head0 + cb % HW;
#pragma unroll
            for (int b = 0; b < D / 16; ++b) *reinterpret_cast<f32x4*>(a.part_o + slot * D + b * 16 + G * 4) = st.o[c][b];
            if (G == 0) {
                a.part_ml[slot * 2] = st.m[c];
                a.part_ml[slot * 2 + 1] = l;
            }
        } else if (qi < it.n_rows) {
            const float inv = 1.0f / l;
            bf16_t* orow = a.out + (int64_t)(it.row0 + qi) * a.ld_o + (int64_t)(head0 + cb % HW) * D;
#pragma unroll
            for (int b = 0; b < D / 16; ++b) {
                f32x4 o = st.o[c][b];
#pragma unroll
                for (int v = 0; v < 4; ++v) o[v] *= inv;
                *reinterpret_cast<bf16x4*>(orow + b * 16 + G * 4) = __builtin_convertvector(o, bf16x4);
            }
        }
    }
}

template <int D, int HW, int NB>
__global__ __launch_bounds__(256, 3) void prefill_attention_kernel(AttnArgs a, const PrefillItem* __restrict__ items) {
    __shared__ PrefillLds<D> lds;
    prefill_workgroup<D, HW, NB>(a, items, blockIdx.x, lds);
}

// Both kinds in one launch: the first workgroups take the prefill items, the others the decode items.  For batches with so
// few prefill workgroups that they would run on a nearly empty chip (kHybridPrefillMax).
template <int D, int HW, int NB>
__global__ __launch_bounds__(256, 2) void hybrid_attention_kernel(AttnArgs a, const PrefillItem* __restrict__ items, int prefill_wgs,
                                                                   DecodeArgs dec) {
    __shared__ union Lds {
        PrefillLds<D> prefill;
        DecodeLds<D, false> decode;
    } lds;
    if ((int)blockIdx.x < prefill_wgs) prefill_workgroup<D, HW, NB>(a, items, blockIdx.x, lds.prefill);
    else decode_workgroup<D, false>(a, dec, blockIdx.x - prefill_wgs, lds.decode);
}

}  // namespace

hipError_t launch_decode_attention(const AttnArgs& a, const DecodeArgs& dec, hipStream_t stream) {
    if (dec.num_items <= 0) return hipSuccess;
    const dim3 grid(dec.num_items * a.n_kv + (dec.from_qkv ? dec.rope.T : 0));
    if (a.n_q / a.n_kv > kMaxGroup || (dec.from_qkv && (dec.rope.planes < 1 || dec.rope.planes > kMaxPlanes))) return hipErrorInvalidValue;
    if (a.d != 128 && a.d != 64) return hipErrorInvalidValue;
    if (a.d == 128 && dec.from_qkv) decode_attention_kernel<128, true><<<grid, 256, 0, stream>>>(a, dec);
    else if (a.d == 128) decode_attention_kernel<128, false><<<grid, 256, 0, stream>>>(a, dec);
    else if (dec.from_qkv) decode_attention_kernel<64, true><<<grid, 256, 0, stream>>>(a, dec);
    else decode_attention_kernel<64, false><<<grid, 256, 0, stream>>>(a, dec);
    return hipGetLastError();
}

hipError_t launch_decode_combine(const AttnArgs& a, const DecodeRow* rows, int num_rows, hipStream_t stream) {
    if (num_rows <= 0) return hipSuccess;
    dim3 grid(num_rows, a.n_q);
    if (a.d == 128) decode_combine_kernel<128><<<grid, 32, 0, stream>>>(a, rows);
    else if (a.d == 64) decode_combine_kernel<64><<<grid, 16, 0, stream>>>(a, rows);
    else return hipErrorInvalidValue;
    return hipGetLastError();
}

// Query heads of a KV head that share a workgroup, and rows of an item: a workgroup has four waves of NB column groups of 16
// (16 rows of one head), eight groups, or four (`half`).
int prefill_heads_per_workgroup(int n_q, int n_kv, bool half) {
    const int g = n_q / n_kv;
    if (g == 8 && half) return 4;
    return (g == 1 || g == 2 || g == 4 || g == 8) ? g : 1;
}

int prefill_item_rows(int n_q, int n_kv, bool half) { return (half ? 64 : 128) / prefill_heads_per_workgroup(n_q, n_kv, half); }

#define GLLM_BY_HEADS(LAUNCH, D_)                                       \
    do {                                                                \
        if (half) {                                                     \
            if (hw == 4) LAUNCH(D_, 4, 1); else if (hw == 2) LAUNCH(D_, 2, 1); else LAUNCH(D_, 1, 1);                               \
        } else {                                                        \
            if (hw == 8) LAUNCH(D_, 8, 2); else if (hw == 4) LAUNCH(D_, 4, 2); else if (hw == 2) LAUNCH(D_, 2, 2); else LAUNCH(D_, 1, 2); \
        }                                                               \
    } while (0)

hipError_t launch_prefill_attention(const AttnArgs& a, const PrefillItem* items, int num_items, bool half, hipStream_t stream) {
    if (num_items <= 0) return hipSuccess;
    const int hw = prefill_heads_per_workgroup(a.n_q, a.n_kv, half);
    const dim3 grid(num_items * (a.n_q / hw));
#define GLLM_PREFILL(D_, HW_, NB_) prefill_attention_kernel<D_, HW_, NB_><<<grid, 256, 0, stream>>>(a, items)
    if (a.d == 128) GLLM_BY_HEADS(GLLM_PREFILL, 128);
    else if (a.d == 64) GLLM_BY_HEADS(GLLM_PREFILL, 64);
    else return hipErrorInvalidValue;
#undef GLLM_PREFILL
    return hipGetLastError();
}

// Up to 64 prefill workgroups (a quarter of the compute units; twice as many of half the rows) share the launch of the decode items: with 4 of them (52
// rows, one layer) a batch takes 43 instead of 46 us, with 32 (71 prompt rows beside 251 decode rows, eight layers) 2220
// instead of 2306 us, against two launches one after the other.  Counted are whole tiles: where the decode rows are too few to hide
// a tile's keys these are cut (see the stage), into up to 768 workgroups.
// More tiles gain nothing beside the key stream of the decode items (160: +0.5 % of the batch, 448: +0.5 %): their own
// loads then wait in the same queues, they hold their slots five times as long, and the sum of the two times is what
// comes out -- from one launch, in either order or interleaved, and from two streams (whose events cost 13 us on top).
constexpr int kHybridPrefillMax = 64;

bool attention_in_one_launch(int n_q, int n_kv, int64_t num_tiles, bool half, int num_decode_rows) {
    return num_tiles > 0 && num_decode_rows > 0 &&
           num_tiles * (n_q / prefill_heads_per_workgroup(n_q, n_kv, half)) <= (half ? 2 : 1) * kHybridPrefillMax;
}

hipError_t launch_hybrid_attention(const AttnArgs& a, const PrefillItem* items, int num_items, bool half, const DecodeArgs& dec, hipStream_t stream) {
    const int hw = prefill_heads_per_workgroup(a.n_q, a.n_kv, half);
    const int prefill_wgs = num_items * (a.n_q / hw);
    if (num_items <= 0 || dec.num_items <= 0) return hipErrorInvalidValue;
    if (dec.from_qkv) return hipErrorInvalidValue;
    const dim3 grid(prefill_wgs + dec.num_items * a.n_kv);
#define GLLM_HYBRID(D_, HW_, NB_) hybrid_attention_kernel<D_, HW_, NB_><<<grid, 256, 0, stream>>>(a, items, prefill_wgs, dec)
    if (a.d == 128) GLLM_BY_HEADS(GLLM_HYBRID, 128);
    else if (a.d == 64) GLLM_BY_HEADS(GLLM_HYBRID, 64);
    else return hipErrorInvalidValue;
#undef GLLM_HYBRID
    return hipGetLastError();
}
#undef GLLM_BY_HEADS
