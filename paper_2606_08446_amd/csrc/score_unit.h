// Page scoring of one (sequence, KV head) unit by one workgroup, the scores staying on chip
// as top-k keys in LDS (internal to libsparrow, not part of the ABI), and the pieces of the
// page score that the split scoring kernel shares with it.
//
// The score of page p (Sec. 3.3 of arXiv 2606.08446) is one dot product of the page's
// 512-byte landmark row with a weight vector fixed per unit (see score_topk.hip).  A lane
// multiplies 16 bytes of the row by its weights in a fixed FMA chain and a 32-lane
// butterfly adds the lanes' parts, in the same order wherever the page is scored, so every
// path gives the same bits.
#pragma once

#include "common.h"
#include "topk.h"

namespace sparrow {

// Sum of 8 per-lane values over the 32 lanes of a half-wave: afterwards lane i holds the
// total of value (i & 7).  Butterfly: each xor step halves the number of values a lane
// keeps.  Every value is summed by the same tree of commutative pairwise additions, so
// identical inputs give identical sums wherever they sit in the batch.
__device__ __forceinline__ float butterfly8(const float (&v)[8], int li)
{
    const bool b0 = li & 1, b1 = li & 2, b2 = li & 4;
    float v1[4], v2[2];
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        const float keep = b0 ? v[2 * j + 1] : v[2 * j];
        const float send = b0 ? v[2 * j] : v[2 * j + 1];
        v1[j] = keep + __shfl_xor(send, 1, 64);
    }
#pragma unroll
    for (int j = 0; j < 2; ++j) {
        const float keep = b1 ? v1[2 * j + 1] : v1[2 * j];
        const float send = b1 ? v1[2 * j] : v1[2 * j + 1];
        v2[j] = keep + __shfl_xor(send, 2, 64);
    }
    const float keep = b2 ? v2[1] : v2[0];
    const float send = b2 ? v2[0] : v2[1];
    float r = keep + __shfl_xor(send, 4, 64);
    r += __shfl_xor(r, 8, 64);
    r += __shfl_xor(r, 16, 64);
    return r;
}

// One lane's share of a page's dot product: its 8 metadata elements against its 8 weights,
// in a fixed FMA order.
__device__ __forceinline__ float lane_dot(const float (&w)[8], u32x4_t v)
{
    float acc = 0.f;
#pragma unroll
    for (int t = 0; t < 4; ++t) {
        acc = fmaf(w[2 * t], bf16_lo(v[t]), acc);
        acc = fmaf(w[2 * t + 1], bf16_hi(v[t]), acc);
    }
    return acc;
}

// Mean landmark: 4 fp32 key sums against the lane's 4 weights, in a fixed FMA order.
__device__ __forceinline__ float lane_dot4(const float (&w)[8], u32x4_t v)
{
    float acc = 0.f;
#pragma unroll
    for (int t = 0; t < 4; ++t)
        acc = fmaf(w[t], __uint_as_float(v[t]), acc);
    return acc;
}

// Valid tokens of logical page p of a sequence of L tokens.
__device__ __forceinline__ int page_tokens(int p, int L, int ps)
{
    const int left = L - p * ps;
    return left < ps ? left : ps;
}

// Adds up to 8 query rows g0 .. of a group of G to a lane's weights, in head order: Q- (the
// mn half of the row) or Q+ (the mx half) of its 8 channels, or with the mean landmark the
// plain sums of its 4 channels.  `qh` points at the lane's channels of the group's row 0.
template <bool kMean>
__device__ __forceinline__ void add_query_rows(float (&w)[8], const uint16_t *qh, int g0, int G,
                                               bool neg)
{
    u32x4_t v[8];
#pragma unroll
    for (int u = 0; u < 8; ++u) {
        v[u] = (u32x4_t){0u, 0u, 0u, 0u};
        if (g0 + u < G) {
            if (kMean) {
                const u32x2_t x = *reinterpret_cast<const u32x2_t *>(qh + (g0 + u) * kHeadDim);
                v[u][0] = x[0];
                v[u][1] = x[1];
            } else {
                v[u] = ld16(qh + (g0 + u) * kHeadDim);
            }
        }
    }
#pragma unroll
    for (int u = 0; u < 8; ++u) {
        if (!(g0 + u < G))
            continue;
        if (kMean) {
            w[0] += bf16_lo(v[u][0]);
            w[1] += bf16_hi(v[u][0]);
            w[2] += bf16_lo(v[u][1]);
            w[3] += bf16_hi(v[u][1]);
        } else {
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                const float x0 = bf16_lo(v[u][j]), x1 = bf16_hi(v[u][j]);
                w[2 * j] += neg ? fminf(x0, 0.f) : fmaxf(x0, 0.f);
                w[2 * j + 1] += neg ? fminf(x1, 0.f) : fmaxf(x1, 0.f);
            }
        }
    }
}

struct ScoreArgs {
    const uint16_t *q;
    uint16_t *meta;
    const int32_t *block_table;
    const int32_t *seq_lens;
    Sched sched;
    AppendArgs app;
    int k_max, num_q_heads, num_kv_heads, ps, max_pages;
    int64_t num_phys;
};

// The token being decoded appended by a half-wave (lane li: elements 8 li .. of the [mn | mx]
// row): its K and V rows written to slot `tok` of physical page `phys`, the page's landmark
// row updated.  Returns the lane's updated 16 bytes.
template <bool kMean>
__device__ __forceinline__ u32x4_t append_token(const ScoreArgs &a, int b, int hh, int64_t phys,
                                                int tok, int li)
{
    const int e0 = 8 * li;
    const int i0 = e0 & (kHeadDim - 1);
    const int64_t nrow = ((int64_t)b * a.num_kv_heads + hh) * kHeadDim + i0;
    const u32x4_t kn = ld16(static_cast<const uint16_t *>(a.app.k_new) + nrow);
    const int64_t crow = ((phys * a.num_kv_heads + hh) * a.ps + tok) * kHeadDim + i0;
    if (e0 < kHeadDim)
        st16(static_cast<uint16_t *>(a.app.k_cache) + crow, kn);
    else
        st16(static_cast<uint16_t *>(a.app.v_cache) + crow,
             ld16(static_cast<const uint16_t *>(a.app.v_new) + nrow));
    uint16_t *mrow = a.meta + (phys * a.num_kv_heads + hh) * 2 * kHeadDim + e0;
    u32x4_t upd = {0u, 0u, 0u, 0u};
    if (kMean) {
        const u32x2_t k4 = *reinterpret_cast<const u32x2_t *>(
            static_cast<const uint16_t *>(a.app.k_new) + nrow - i0 + 4 * li);
        upd = sums_with_key(tok == 0, tok == 0 ? upd : ld16(mrow), k4);
    } else {
        upd = meta_with_key(tok == 0 ? kn : ld16(mrow), kn, e0 >= kHeadDim, tok == 0);
    }
    st16(mrow, upd);
    return upd;
}

// A unit's scoring pass, in the order a workgroup's code runs it.
//
// A wave takes every kWaves-th batch of 16 pages; a load instruction reads the rows of two
// pages (lanes 0-31 one of the batch's first eight, 32-63 one of its last eight), 512
// contiguous bytes each, and the next batch's eight loads are always in flight (they are
// unconditional, so the compiled loop waits for exactly the current ones).  The physical
// pages of four batches come with one block-table load, a group ahead.  Every page index is
// clamped to the cache where it is loaded: an entry outside it (an absent page, score 0) or
// past the sequence reads page 0, whose value is not used.
template <bool kAppend, bool kMean, int kThreads>
struct UnitScorer {
    static constexpr int kWaves = kThreads / 64;
    static constexpr int kBatch = 16;  // pages per batch of a wave

    const ScoreArgs &a;
    const int32_t *bt;   // the sequence's block-table row
    const uint16_t *mrow;  // the lane's 16 bytes of the unit's row of physical page 0
    int b, h, wave, lane, half, li;
    int btv, btn;       // lane i: physical page (or -1) of page i of this group / the next
    uint64_t absent;    // bit i: page i of the group is absent
    float w[8];

    __device__ __forceinline__ UnitScorer(const ScoreArgs &args, int b_, int h_)
        : a(args), b(b_), h(h_)
    {
        wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
        lane = threadIdx.x & 63;
        half = lane >> 5;
        li = lane & 31;
        bt = a.block_table + (int64_t)b * a.max_pages;
        mrow = a.meta + (int64_t)h * 2 * kHeadDim + 8 * li;
    }

    // The page of lane `l` of block-table group g (four batches of this wave).
    __device__ __forceinline__ int group_page(int g, int l) const
    {
        return (wave + kWaves * (4 * g + (l >> 4))) * kBatch + (l & 15);
    }

    __device__ __forceinline__ int load_group(int g) const
    {
        const int p = group_page(g, lane);
        const int e = bt[p < a.max_pages ? p : a.max_pages - 1];
        return p < a.max_pages && e >= 0 && e < a.num_phys ? e : -1;
    }

    // Whether this half-wave appends the token: there is one (its position inside what the
    // block table addresses), and the half-wave scores its page n - 1.
    __device__ __forceinline__ bool append_here(int L_raw, int n) const
    {
        return L_raw >= 1 && L_raw <= a.ps * a.max_pages &&
               ((n - 1) / kBatch) % kWaves == wave && half == (((n - 1) & 15) >> 3);
    }

    // Requests what does not depend on the length: the first block-table groups and the
    // group's queries.
    __device__ __forceinline__ void start()
    {
        btv = load_group(0);
        const int G = a.num_q_heads / a.num_kv_heads;
        const uint16_t *qh = a.q + ((int64_t)b * a.num_q_heads + (int64_t)h * G) * kHeadDim +
                             (kMean ? 4 * li : (8 * li) & (kHeadDim - 1));
#pragma unroll
        for (int j = 0; j < 8; ++j)
            w[j] = 0.f;
        add_query_rows<kMean>(w, qh, 0, G, li < 16);
        for (int g0 = 8; g0 < G; g0 += 8)
            add_query_rows<kMean>(w, qh, g0, G, li < 16);
        absent = __ballot(btv < 0);
        btn = load_group(1);
    }

    // Loads of batch i of this wave (its pages sit in btv), and which of its pages are absent.
    __device__ __forceinline__ void issue(int i, u32x4_t (&v)[8], uint32_t &ab) const
    {
        const int base = (i & 3) * kBatch;
        const int64_t page_elems = (int64_t)a.num_kv_heads * 2 * kHeadDim;
#pragma unroll
        for (int j = 0; j < 8; ++j) {
            const int p0 = __builtin_amdgcn_readlane(btv, base + j);
            const int p1 = __builtin_amdgcn_readlane(btv, base + 8 + j);
            const int ph = half ? p1 : p0;
            v[j] = ld16_nt(mrow + (int64_t)(ph < 0 ? 0 : ph) * page_elems);
        }
        ab = (uint32_t)(absent >> base) & 0xffffu;
    }

    // Keys of the pages 0 .. n-1 of a sequence of L tokens into keys[]; `last` is the page the
    // token was appended to (-1: none), whose updated slice is `upd`.  kmin and kmax take the
    // thread's own keys.
    __device__ __forceinline__ void run(u32x4_t (&nxt)[8], uint32_t ab, int L, int n, int last,
                                        u32x4_t upd, uint32_t *keys, uint32_t &kmin,
                                        uint32_t &kmax)
    {
        const int nb_all = (n + kBatch - 1) / kBatch;
        const int nb = (nb_all - wave + kWaves - 1) / kWaves;  // of this wave
        auto put = [&](int page, float total) {
            // forced pages (sinks, most recent pages) outrank every score
            const bool forced = page < a.sched.sink_pages || page >= n - a.sched.local_pages;
            const uint32_t key = forced ? 0xffffffffu : score_key(total);
            keys[page] = key;
            kmin = min(kmin, key);
            kmax = max(kmax, key);
        };
        auto process = [&](int i, const u32x4_t (&cur)[8], uint32_t abc) {
            float part[8];
#pragma unroll
            for (int j = 0; j < 8; ++j)
                part[j] = kMean ? lane_dot4(w, cur[j]) : lane_dot(w, cur[j]);
            const float total = butterfly8(part, li);
            const int page = (wave + kWaves * i) * kBatch + 8 * half + (li & 7);
            if (li < 8 && page < n && !(kAppend && page == last))
                put(page, (abc >> (8 * half + li)) & 1 ? 0.f
                          : kMean ? total / (float)page_tokens(page, L, a.ps)
                                  : total);
        };
        int i = 0;
        for (; i + 1 < nb; ++i) {
            u32x4_t cur[8];
#pragma unroll
            for (int j = 0; j < 8; ++j)
                cur[j] = nxt[j];
            const uint32_t abc = ab;
            if (((i + 1) & 3) == 0) {
                btv = btn;
                absent = __ballot(btv < 0);
                btn = load_group((i + 1) / 4 + 1);
            }
            issue(i + 1, nxt, ab);
            process(i, cur, abc);
        }
        if (i < nb)
            process(i, nxt, ab);
        // The appended page, from the updated slice: the same FMA chain and a 32-lane xor
        // reduction, the tree that butterfly8 applies to every page.
        if (kAppend && last >= 0) {  // only in the half-wave that owns the page
            float total = kMean ? lane_dot4(w, upd) : lane_dot(w, upd);
#pragma unroll
            for (int x = 1; x < 32; x <<= 1)
                total += __shfl_xor(total, x, 64);
            if (li == 0)
                put(last, kMean ? total / (float)page_tokens(last, L, a.ps) : total);
        }
    }
};

}  // namespace sparrow
