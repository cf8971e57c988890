// Paged grouped-query decode attention (Sec. 2.3: one query token per request against all of its cached keys; a
// memory-bound sweep over the KV cache), split over the context, plus the merge of the split results.
//
// A request's keys are cut into spans by a rule on its own context (and on whether the batch is a small one), and a span is
// reduced by one wavefront from its first key to its last: a request's result does not depend on which requests share the
// batch, on how tight the context hint is or on the CU share.  The spans of the batch, request by request, kv head by kv
// head, are dealt to the wavefronts in runs of equal length, whatever requests and heads a run touches: ragged contexts
// leave no wavefront with much more to do than another.  The wavefront serves all G query heads of its kv head at once, so every
// K/V byte is fetched once per kv head.  K and V pages are read straight from global memory into MFMA operand registers: the private page
// layouts make each load instruction cover contiguous runs of memory with 16 bytes per lane, and no LDS is needed because
// nothing is shared between wavefronts.  S^T = K Q^T and O^T += V^T P^T with the 16x16x32 bf16 MFMA: one column per
// query head, softmax running max / sum kept per column, and the score registers of two consecutive 16-row tiles
// are exactly the 8 probabilities the matching V^T operand needs (no transpose between the products).
//
// Queries are the rotated bf16 rows written by the rotary kernel; the new token's K/V is already in the pools
// (appended by the same kernel), so a request with c cached tokens attends to c+1 keys.
#pragma once
#include "common.hpp"

namespace nexus {

// Wavefronts the spans are dealt to: one per SIMD, so that all run at once and end together.  A wavefront
// pays a fixed chain of latencies (context lengths, page ids, first pages: 3 us on an idle chip, 7 us in the queue of a
// loaded one) per stretch of one request's keys; runs of equal length have few of them.  256 requests with contexts up to
// 8192, 8B shape: a wavefront per 256-key span 815 us, runs 768 (512, 2048 and 4096 of them instead of 1024: 2 to 3 % more);
// without regard to spans, cut at any pair, runs took 750, but then a request's cuts, and its rounding, follow from its
// neighbours' contexts.  Three or four pairs in flight per wavefront instead of two gain nothing.  The number of runs
// changes no result, so it follows the CU share: on up to 64 CUs two per SIMD, as many as it holds (four wavefronts do not keep
// enough in flight for a CU's 50 GB/s).  64 requests up to 4096, steps of two layers, 1024 runs / these: on 96 CUs 712 / 685 us,
// on 160 538 / 527, on 224 473 / 455; four layers next to a 512-token chunk on 192 CUs 1946 / 1922 (one per SIMD 1944).
//
// Spans, in pairs of pages (32 keys).  Where 256 keys hold a context it is one span, and nothing is to be merged.  Otherwise a
// long span costs balance (a run is longer or shorter by up to one) and parallelism (a batch of few requests has fewer
// spans than the chip has SIMDs), a short one costs stores and merging.  Up to 32 requests: 2 pairs up to 1024 keys (one
// request of 800 keys, 8B shape: 6.4 us; 8 pairs 8.5), 4 up to 4096 (23 requests up to 2500, a step of four layers of the 14B
// shape: 601 us, 604 with 2 pairs up to 2048), 8 beyond (one of 8000, a step of two layers: 233 us, 246 with 2 pairs).  More
// requests: 8 pairs (64 up to 4096: 828 us for a step of four layers, 830 with 4 pairs), and 16 beyond 4096 keys if there are
// more than 64 (the 256 requests above 768 us, 781 with 8 pairs).  The bounds 32 and 64 are those at which the projections
// change their order of summation, too.
constexpr int kDecWorkers = 1024, kDecMinPairs = 2, kDecWholeCtx = 256;
// log2 of the pairs of pages in a span of a context of `len` keys; decode_spans: its spans
__host__ __device__ __forceinline__ int decode_span_shift(int n_reqs, int len) {
    if (len <= kDecWholeCtx) return 3;
    if (n_reqs > 64 && len > 4096) return 4;
    if (n_reqs > 32 || len > 4096) return 3;
    return len > 1024 ? 2 : 1;
}
__host__ __device__ __forceinline__ int decode_pairs(int len) { return (len + 31) >> 5; }
__host__ __device__ __forceinline__ int decode_spans(int n_reqs, int len) {
    const int sh = decode_span_shift(n_reqs, len);
    return (decode_pairs(len) + (1 << sh) - 1) >> sh;
}
// Largest number of spans of a context of at most max_ctx keys.
inline int decode_max_spans(int n_reqs, int max_ctx) {
    int n = decode_spans(n_reqs, max_ctx);
    for (int top : {kDecWholeCtx, 1024, 4096})
        if (max_ctx > top) n = std::max(n, decode_spans(n_reqs, top));
    return n;
}
// Keys of a context that a batch with this hint attends to.  The hint is at least every context with its new token; one that
// is too small (the scheduler states contexts without the new token) costs no keys up to the next multiple of 256.
inline int decode_ctx_bound(int max_ctx) { return round_up(max_ctx, 256); }
inline int decode_workers(int cus) { return std::min(kDecWorkers, (cus <= 64 ? 8 : 4) * cus); }
inline int decode_grid(int n_reqs, int n_kv_heads, int max_ctx, int workers) {
    const long seqs = (long)n_reqs * n_kv_heads;
    if (max_ctx <= kDecWholeCtx) return (int)seqs;
    const long runs = (seqs * ((max_ctx + 31) / 32) + kDecMinPairs - 1) / kDecMinPairs;
    return (int)(runs < workers ? runs : workers);
}

struct AttnDecodeArgs {
    const bf16_t *q;  // row-major [B][Hq*hd], rotated
    const int32_t *ctx_len, *page_table;
    int n_reqs, max_pages, max_ctx;  // max_ctx: decode_ctx_bound of the hint; <= kDecWholeCtx: outputs go straight to `out`
    int max_spans;  // decode_max_spans of max_ctx
    int workers;    // decode_workers of the CUs it runs on
    const bf16_t *k_pool, *v_pool;
    int n_pages, Hq, Hkv;
    float scale_log2e;
    f16_t *part_o;   // [B][Hkv][max_spans][G][hd]: each span's output normalised by its own sum, half
    float *part_ml;  // [B][Hkv][max_spans][G][2]  (running max in the log2 domain, sum)
    f16_t *out;      // merge output: half, P32 [B rows][Hq*hd]
    // Decode requests riding in a chunked-prefill batch (the fused single-batch step): their queries sit in the
    // prefill layout -- P32, every request on a 32-row boundary, request j of the decode part in the row tile that
    // follows the tiles of the n_lead leading requests -- and their outputs go to rows out_row0 + j.  lead_cu is
    // null for the plain decode phase (q row-major [B][Hq*hd], output row j).
    const int32_t *lead_cu;  // cu_chunk of the batch the requests ride in
    int n_lead, out_row0;
};

// Keys of request j (contexts past the bound are cut: it bounds the work, the page table its reads), and their pairs.
__device__ __forceinline__ int decode_len(const AttnDecodeArgs &a, int j) {
    const int c = a.ctx_len[min(j, a.n_reqs - 1)];  // no branch around the load: the four of a lane are in flight together
    return j < a.n_reqs ? max(0, min(c + 1, a.max_ctx)) : 0;
}

// Inclusive sum over the lanes of a wavefront, by lane moves of the vector ALU (no trip through LDS).
__device__ __forceinline__ int wave_inclusive_sum(int v) {
    v += __builtin_amdgcn_update_dpp(0, v, 0x111, 0xf, 0xf, true);  // row_shr:1, 2, 4, 8: sums inside the rows of 16 lanes
    v += __builtin_amdgcn_update_dpp(0, v, 0x112, 0xf, 0xf, true);
    v += __builtin_amdgcn_update_dpp(0, v, 0x114, 0xf, 0xf, true);
    v += __builtin_amdgcn_update_dpp(0, v, 0x118, 0xf, 0xf, true);
    v += __builtin_amdgcn_update_dpp(0, v, 0x142, 0xa, 0xf, true);  // row_bcast:15 into rows 1 and 3
    v += __builtin_amdgcn_update_dpp(0, v, 0x143, 0xc, 0xf, true);  // row_bcast:31 into rows 2 and 3
    return v;
}

template <int HD, int G>
__global__ __launch_bounds__(64, 2) void attn_decode_kernel(AttnDecodeArgs a) {
    constexpr int KK = HD / 32;   // k-steps of QK^T
    constexpr int RT = HD / 16;   // 16-row tiles of O^T
    constexpr int BLK = kPage * HD;  // elements per (page, kv head) block
    // Results of finished spans, written out at the end of the run or when the stage is full (20 KB, an eighth of a CU's LDS: as
    // many wavefronts as its registers hold).  A store counts like a load, and the loads behind it are waited for in order: the 256 requests
    // above, in spans of 8 pairs, took 821 us with every result stored between the pairs, 808 staged per request and kv
    // head, 781 staged per run (731 with the stores left out); in spans of 16 pairs a run fits the stage whole (19 spans, 4 heads).
    constexpr int kStage = 20480 / (G * (2 * HD + 8) + 4), CPS = G * HD / 8;  // spans, 16-byte chunks of a span
    __shared__ uint4 stage_o[kStage * CPS];
    __shared__ float2 stage_ml[kStage * G];
    __shared__ int stage_slot[kStage];
    const int lane = threadIdx.x & 63;
    const int col = lane & 15, g4 = lane >> 4;
    const int w = blockIdx.x;

    // This wavefront's run: the spans whose first pairs are among the pairs [run_begin, run_begin + per) of the batch's pairs in
    // (request, kv head) order.  A lane counts the pairs of 4 consecutive requests, a wavefront scan places 256.
    int j = 0, kvh = 0, pair = 0, todo = 0, len = 0;
    const bool whole = a.max_ctx <= kDecWholeCtx;
    if (whole) {
        j = w / a.Hkv, kvh = w % a.Hkv;
        len = decode_len(a, j);
        todo = decode_pairs(len);
        if (todo == 0) return;
    } else {
        int lens[4], mine = 0, incl = 0, total = 0;
        auto scan = [&](int base) {  // incl: pairs per kv head of the requests base .. base + 4 lane + 3
#pragma unroll
            for (int e = 0; e < 4; ++e) lens[e] = decode_len(a, base + 4 * lane + e);
            mine = decode_pairs(lens[0]) + decode_pairs(lens[1]) + decode_pairs(lens[2]) + decode_pairs(lens[3]);
            incl = wave_inclusive_sum(mine);
            return __builtin_amdgcn_readlane(incl, 63);
        };
        for (int base = 0; base < a.n_reqs; base += 256) total += scan(base);
        total *= a.Hkv;
        const int per = max(kDecMinPairs, (total + a.workers - 1) / a.workers);
        const int run_begin = w * per;
        if (run_begin >= total) return;
        todo = min(per, total - run_begin);
        int before = 0, base = 0;  // pairs of the requests before `base`, then before j
        if (a.n_reqs > 256) {
            int t;
            while (run_begin >= before + (t = scan(base)) * a.Hkv) before += t * a.Hkv, base += 256;
        }
        const int hit = __builtin_ctzll(__builtin_amdgcn_ballot_w64(run_begin < before + incl * a.Hkv));
        before += __builtin_amdgcn_readlane(incl - mine, hit) * a.Hkv;
        j = base + 4 * hit;
        len = __builtin_amdgcn_readlane(lens[0], hit);
#pragma unroll
        for (int e = 1; e < 4; ++e) {
            const int c = decode_pairs(len) * a.Hkv;
            if (j == base + 4 * hit + e - 1 && run_begin >= before + c) before += c, ++j, len = __builtin_amdgcn_readlane(lens[e], hit);
        }
        const int np = decode_pairs(len), rest = run_begin - before;
        kvh = rest / np, pair = rest % np;
        const int span = 1 << decode_span_shift(a.n_reqs, len), skip = min((span - pair % span) % span, np - pair);
        pair += skip, todo -= skip;
    }
    j = __builtin_amdgcn_readfirstlane(j), kvh = __builtin_amdgcn_readfirstlane(kvh), len = __builtin_amdgcn_readfirstlane(len);
    pair = __builtin_amdgcn_readfirstlane(pair), todo = __builtin_amdgcn_readfirstlane(todo);

    const int half_off = (col & 7) * 8 + g4 * 128;  // elements: slot (col % 8) of a tile's half, k-group g4
    int lead_tiles = 0;
    if (a.lead_cu)
        for (int i = 0; i < a.n_lead; ++i) lead_tiles += (a.lead_cu[i + 1] - a.lead_cu[i] + 31) >> 5;

    int staged = 0;
    auto write_staged = [&]() {
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");  // what other lanes wrote
        for (int i = lane; i < staged * CPS; i += 64) ((uint4 *)a.part_o)[(size_t)stage_slot[i / CPS] * CPS + i % CPS] = stage_o[i];
        for (int i = lane; i < staged * G; i += 64) ((float2 *)a.part_ml)[(size_t)stage_slot[i / G] * G + i % G] = stage_ml[i];
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        staged = 0;
    };

    // one stretch of spans of a (request, kv head) after another
    while (todo > 0) {
    const int np = decode_pairs(len), sh = decode_span_shift(a.n_reqs, len), span = 1 << sh;
    const int n_pairs = min((todo + span - 1) & -span, np - pair);
    if (n_pairs > 0) {
    // Page ids of a span, one per lane, fetched a span ahead: no key/value load waits on a page-table read.  Ids that are out
    // of range or belong to pages past the end of the context are replaced by page 0: every load below then has a valid
    // address and no branch, and what it fetches for such a page is masked out.
    auto page_ids = [&](int lp0) {
        const int lp = lp0 + lane;
        int id = 0;
        if (lp * 16 < len && lp < a.max_pages) id = a.page_table[(size_t)j * a.max_pages + lp];
        return (unsigned)id < (unsigned)a.n_pages ? id : 0;
    };
    int ids = page_ids(2 * pair);

    const int q_row = (lead_tiles + j) * 32;
    bf16x8 qf[KK];
#pragma unroll
    for (int kk = 0; kk < KK; ++kk) {
        u32x4 v = {0, 0, 0, 0};
        if (col < G) {
            const int k = (kvh * G + col) * HD + (kk * 4 + g4) * 8;
            v = *(const u32x4 *)(a.q + (a.lead_cu ? p32_offset(q_row, k, a.Hq * HD) : (size_t)j * a.Hq * HD + k));
        }
        qf[kk] = *(bf16x8 *)&v;
    }
    f32x4 o_acc[RT];
#pragma unroll
    for (int i = 0; i < RT; ++i)
#pragma unroll
        for (int e = 0; e < 4; ++e) o_acc[i][e] = 0.f;
    float m_run = -INFINITY, l_run = 0.f;

    // One pair = two pages (A, B) = 32 keys.  S^T is computed as two 16-row tiles: tile 1 takes slots 0..7 of page
    // A and of page B (tokens {0..3, 8..11}), tile 2 slots 8..15 (tokens {4..7, 12..15}); lane (col = query head,
    // g4) then holds the scores of tokens 8*(g4 % 2) .. +7 of page g4 / 2, exactly the 8 tokens of the V^T operand
    // it reads with one 16-byte load.
    struct PairRegs {
        u32x4 k1[KK], k2[KK], v[RT];
    };
    auto load_pair = [&](PairRegs &r, int ids, int pp) {  // pair pp of the span whose page ids are given
        const int pageA = __builtin_amdgcn_readlane(ids, 2 * pp), pageB = __builtin_amdgcn_readlane(ids, 2 * pp + 1);
        // K operand row (lane % 16): rows 0..7 from page A, 8..15 from page B
        const bf16_t *kp = a.k_pool + ((size_t)(col < 8 ? pageA : pageB) * a.Hkv + kvh) * BLK + half_off;
        // V operand: lane group g4 reads page g4 / 2, token group g4 % 2, hd rows 16 i + col
        const bf16_t *vp = a.v_pool + ((size_t)(g4 < 2 ? pageA : pageB) * a.Hkv + kvh) * BLK + ((g4 & 1) * HD + col) * 8;
#pragma unroll
        for (int kk = 0; kk < KK; ++kk) {
            // K/V pages are read once per kv head: non-temporal loads, so the stream does not evict what the prefill
            // phase shares through L2
            r.k1[kk] = __builtin_nontemporal_load((const u32x4 *)(kp + kk * 512));
            r.k2[kk] = __builtin_nontemporal_load((const u32x4 *)(kp + kk * 512 + 64));
        }
#pragma unroll
        for (int i = 0; i < RT; ++i) r.v[i] = __builtin_nontemporal_load((const u32x4 *)(vp + i * 128));
    };
    auto compute_pair = [&](PairRegs &r, int p) {  // pair p of the request
        f32x4 s1 = {0, 0, 0, 0}, s2 = {0, 0, 0, 0};
#pragma unroll
        for (int kk = 0; kk < KK; ++kk) {
            s1 = __builtin_amdgcn_mfma_f32_16x16x32_bf16(*(bf16x8 *)&r.k1[kk], qf[kk], s1, 0, 0, 0);
            s2 = __builtin_amdgcn_mfma_f32_16x16x32_bf16(*(bf16x8 *)&r.k2[kk], qf[kk], s2, 0, 0, 0);
        }
        // register e of s1 is key key0 + e, of s2 key key0 + 4 + e
        const int key0 = 32 * p + 16 * (g4 >> 1) + 8 * (g4 & 1);
        float sv[8];
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            sv[e] = s1[e] * a.scale_log2e;
            sv[4 + e] = s2[e] * a.scale_log2e;
        }
        const bool tail = 32 * p + 32 > len;  // uniform: only the last pair of a context
        if (tail) {
#pragma unroll
            for (int e = 0; e < 8; ++e) sv[e] = key0 + e < len ? sv[e] : -INFINITY;
            // values past the end of the context may hold anything; their weight is 0 but 0 * NaN is not
#pragma unroll
            for (int i = 0; i < RT; ++i)
#pragma unroll
                for (int e = 0; e < 8; ++e)
                    if (key0 + e >= len) r.v[i][e >> 1] &= (e & 1) ? 0x0000ffffu : 0xffff0000u;
        }
        float mx = m_run;
#pragma unroll
        for (int e = 0; e < 8; ++e) mx = fmaxf(mx, sv[e]);
        mx = fmaxf(mx, __shfl_xor(mx, 16));
        mx = fmaxf(mx, __shfl_xor(mx, 32));
        // the first key of a pair is always valid, so mx is finite
        const float alpha = __builtin_amdgcn_exp2f(m_run - mx);
        m_run = mx;
        float rs = 0.f;
        bf16x8 pf;
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            const float p = __builtin_amdgcn_exp2f(sv[e] - mx);
            rs += p;
            pf[e] = (__bf16)p;
        }
        l_run = l_run * alpha + rs;
#pragma unroll
        for (int i = 0; i < RT; ++i) {
#pragma unroll
            for (int e = 0; e < 4; ++e) o_acc[i][e] *= alpha;
            o_acc[i] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(*(bf16x8 *)&r.v[i], pf, o_acc[i], 0, 0, 0);
        }
    };

    // The running span's result, and the start of the next one's.  Register e of o_acc[i] is hd = 16 i + 4 g4 + e.  Stored
    // normalised (an average of value rows, inside half's range whenever the values are) and in half: half the bytes of an
    // fp32 partial, at a rounding 4x finer than the bf16 the values came in; a span is never empty.
    auto sum_lanes = [&]() {
        l_run += __shfl_xor(l_run, 16);
        l_run += __shfl_xor(l_run, 32);
        return 1.0f / l_run;
    };
    auto row = [&](int i, float inv_l) {
        return uint2{packh2(o_acc[i][0] * inv_l, o_acc[i][1] * inv_l), packh2(o_acc[i][2] * inv_l, o_acc[i][3] * inv_l)};
    };
    auto stage_span = [&](int s) {
        const float inv_l = sum_lanes();
        if (lane == 0) stage_slot[staged] = (j * a.Hkv + kvh) * a.max_spans + s;
        if (col < G) {
            f16_t *so = (f16_t *)stage_o + (staged * G + col) * HD + 4 * g4;
#pragma unroll
            for (int i = 0; i < RT; ++i) *(uint2 *)(so + 16 * i) = row(i, inv_l);
            if (g4 == 0) stage_ml[staged * G + col] = float2{m_run, l_run};
        }
#pragma unroll
        for (int i = 0; i < RT; ++i)
#pragma unroll
            for (int e = 0; e < 4; ++e) o_acc[i][e] = 0.f;
        m_run = -INFINITY, l_run = 0.f;
        if (++staged == kStage) write_staged();
    };

    // Two register sets: the loads of the next pair are in flight while the current pair is computed.  The steady
    // state loop has no branch around a prefetch: with one, the paths with and without the extra loads in flight
    // merge, and the compiler can only wait as if they had not been issued, i.e. for the prefetch itself.
    PairRegs r0, r1;
    load_pair(r0, ids, 0);
    int p0 = pair;  // first pair of the running span
    for (; pair + n_pairs - p0 > span; p0 += span) {
        const int next_ids = page_ids(2 * (p0 + span));
        load_pair(r1, ids, 1);
        if (p0 > pair) stage_span((p0 - 1) >> sh);
        compute_pair(r0, p0);
        load_pair(r0, span > 2 ? ids : next_ids, span > 2 ? 2 : 0);
        compute_pair(r1, p0 + 1);
        for (int pp = 2; pp < span; pp += 2) {
            load_pair(r1, ids, pp + 1);
            compute_pair(r0, p0 + pp);
            load_pair(r0, pp + 2 < span ? ids : next_ids, pp + 2 < span ? pp + 2 : 0);
            compute_pair(r1, p0 + pp + 1);
        }
        ids = next_ids;
    }
    if (p0 > pair) stage_span((p0 - 1) >> sh);
    {
        const int left = pair + n_pairs - p0;
        int pp = 0;
        for (; pp + 2 < left; pp += 2) {
            load_pair(r1, ids, pp + 1);
            compute_pair(r0, p0 + pp);
            load_pair(r0, ids, pp + 2);
            compute_pair(r1, p0 + pp + 1);
        }
        if (pp + 1 < left) {
            load_pair(r1, ids, pp + 1);
            compute_pair(r0, p0 + pp);
            compute_pair(r1, p0 + pp + 1);
        } else {
            compute_pair(r0, p0 + pp);
        }
    }
    if (np > span) {
        stage_span(p0 >> sh);
    } else {  // a single span, nothing to merge: the output row itself, P32
        const float inv_l = sum_lanes();
        if (col < G)
#pragma unroll
            for (int i = 0; i < RT; ++i)
                *(uint2 *)(a.out + p32_offset(a.out_row0 + j, (kvh * G + col) * HD + 16 * i + 4 * g4, a.Hq * HD)) = row(i, inv_l);
    }
    }
    todo -= n_pairs, pair = 0;
    if (++kvh == a.Hkv) kvh = 0, ++j, len = todo > 0 ? __builtin_amdgcn_readfirstlane(decode_len(a, j)) : 0;
    }
    if (staged) write_staged();
}

// Merge of the partial results of one (request, query head): with w_s = 2^(m_s - m) l_s and o_s the normalised output of
// its s-th span, o = sum_s w_s o_s / sum_s w_s, in order.  One wavefront per (request, query head); output in P32 order for
// the O projection.  A request of a single span has its output already.
template <int HD, int G>
__global__ __launch_bounds__(64) void attn_merge_kernel(AttnDecodeArgs a) {
    const int j = blockIdx.x / a.Hq, hq = blockIdx.x % a.Hq;
    const int kvh = hq / G, col = hq % G, lane = threadIdx.x;
    const int n_spans = decode_spans(a.n_reqs, decode_len(a, j));
    if (n_spans <= 1) return;
    const size_t item0 = ((size_t)j * a.Hkv + kvh) * a.max_spans;
    constexpr int EPL = HD / 64;
    float acc[EPL], m = -INFINITY, denom = 0.f;
#pragma unroll
    for (int e = 0; e < EPL; ++e) acc[e] = 0.f;
    // spans are taken 64 at a time: lane s holds the statistics of span base + s, so the loads of the partial
    // outputs do not wait on one another
    for (int base = 0; base < n_spans; base += 64) {
        const int s = base + lane;
        float2 ml = {-INFINITY, 0.f};
        if (s < n_spans) ml = *(const float2 *)(a.part_ml + ((item0 + s) * G + col) * 2);
        float cm = ml.x;
#pragma unroll
        for (int o = 32; o > 0; o >>= 1) cm = fmaxf(cm, __shfl_xor(cm, o));
        const float m_new = fmaxf(m, cm);
        const float rescale = exp2f(m - m_new);  // 0 on the first chunk (m = -inf), spans are never empty
        const float wl = s < n_spans ? exp2f(ml.x - m_new) * ml.y : 0.f;  // weight of the span's normalised output
        float part = wl;
#pragma unroll
        for (int o = 32; o > 0; o >>= 1) part += __shfl_xor(part, o);
        denom = denom * rescale + part;
#pragma unroll
        for (int e = 0; e < EPL; ++e) acc[e] *= rescale;
        const int cnt = min(64, n_spans - base);
        // eight spans' rows at a time, fetched by loads that do not wait on one another; summed in span order
        for (int k0 = 0; k0 < cnt; k0 += 8) {
            uint32_t pv[8];
#pragma unroll
            for (int u = 0; u < 8; ++u) {
                pv[u] = 0;
                if (k0 + u < cnt) {
                    const f16_t *po = a.part_o + ((item0 + base + k0 + u) * G + col) * HD + lane * EPL;
                    pv[u] = EPL == 2 ? *(const uint32_t *)po : (uint32_t)po[0];
                }
            }
#pragma unroll
            for (int u = 0; u < 8; ++u) {
                const float wk = __shfl(wl, (k0 + u) & 63);  // rows past cnt were read as zero
                acc[0] += wk * h2f((f16_t)(pv[u] & 0xffffu));
                if (EPL == 2) acc[EPL - 1] += wk * h2f((f16_t)(pv[u] >> 16));
            }
        }
        m = m_new;
    }
    const float inv = 1.0f / denom;
    const int QKp = a.Hq * HD;
    f16_t *dst = a.out + p32_offset(a.out_row0 + j, hq * HD + lane * EPL, QKp);
    if (EPL == 2) {
        *(uint32_t *)dst = packh2(acc[0] * inv, acc[EPL - 1] * inv);
    } else {
        dst[0] = f2h(acc[0] * inv);
    }
}

}  // namespace nexus
