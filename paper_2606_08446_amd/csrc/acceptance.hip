// Per-token acceptance rate between the dense policy and the sparse rollout (Sec. 3.1,
// Eq. 1 of arXiv 2606.08446) and its lower-tail statistic per length bin (Sec. 3.1-3.2).
//
// k_acceptance: alpha_t = sum_x min(p(x), q(x)) with p, q the softmax of the target and draft
// logit rows at inverse temperature tau.  Two passes over a token's two rows: the log-sum-exp of
// both, then sum_x exp(min(tau a_x - P, tau b_x - Q)) - one exp per vocabulary entry, since
// min(e^u, e^v) = e^min(u, v).  A 512-thread workgroup per CU (8 waves, so a wave has 256
// registers) takes every gridDim.x-th token and keeps as much of the rows as fits on chip
// between the passes: 144 KiB in LDS, 21 (fp32) or 19 (bf16) vectors per thread and row in
// registers - 40 % of an fp32 row pair of Qwen3's vocabulary, three quarters of a bf16 one.
// The rest is read again, last part first, while the L2 may still hold it; where there is a
// rest and more than a few tokens, the kept vectors are read non-temporally to leave the caches
// to it.
//
// What bounds it: fp32 rows their traffic (the loads ask for 1.56 times the rows of Qwen3's
// vocabulary, at 7.5 TB/s, some of the second reading being served by the caches), bf16 rows
// the arithmetic and the turns between the passes.  The fp32 kernel spills 3 registers at 21
// kept vectors; with 20 it spills none and was 1-2 % slower on those rows.  With one token per workgroup the memory was
// idle while the second pass computed and the VALU idle while a new token's rows arrived;
// now the second pass replaces every kept vector by the next token's as soon as it is used,
// the other vectors roll through three slots per row, and one barrier a token joins the
// passes.  The running maximum went too (lse_add_fast): 4 instructions per entry and row in
// the first pass instead of 6.  4096 tokens of 151936 entries: bf16 569 -> 465 us, fp32 1050 ->
// 1026 us; 2000 tokens of 30011: bf16 94 -> 76 us, fp32 135 -> 113 us.
// Rows are read as 16-byte vectors; the elements before and after them (a row that does not
// start 16-byte aligned) are one element per thread at most.  Accumulation is fp32 per thread,
// tree reductions across the workgroup.
//
// k_acceptance_topk: the approximation from the top-K listed tokens' normalised
// log-probabilities, sum_i min(exp(lp_i), exp(lq_i)); one thread per token.
//
// k_tail_stats: one workgroup per position bin.  Count and fp64 sum of the bin's values,
// then the order statistics x_lo and x_lo+1 (lo = floor((N - 1) pct / 100)) by a radix
// select over order-preserving uint32 keys (8-bit digits), and the percentile x_lo + (h - lo)(x_lo+1 - x_lo) in fp64 with the multiply and
// the add rounded separately.
#include <type_traits>

#include "common.h"
#include "wave.h"

namespace sparrow {
namespace {

constexpr int kAccThreads = 512;
constexpr int kAccWaves = kAccThreads / 64;
constexpr int kAccLdsVecs = 9;  // 16-byte vectors of each row a thread keeps in LDS
constexpr int kAccBatch = 3;    // vectors of each row a thread has in flight beside the kept ones
constexpr int kAccFold = 8;     // groups of them after which a thread's partial sums are put aside
constexpr int kAccSmallVocab = 64;  // rows shorter than this: one wave per token
constexpr int kTailThreads = 1024;
constexpr int kTailWaves = kTailThreads / 64;

template <typename T> struct Logit;
template <> struct Logit<float> {
    static constexpr int kVec = 4;  // elements per 16-byte vector
    static constexpr int kKeep = 21;  // vectors of each row a thread keeps in registers
    __device__ static float at(const float *row, int64_t i) { return row[i]; }
    __device__ static void unpack(u32x4_t v, float (&x)[kVec])
    {
#pragma unroll
        for (int e = 0; e < 4; ++e)
            x[e] = __uint_as_float(v[e]);
    }
};
template <> struct Logit<uint16_t> {
    static constexpr int kVec = 8;
    static constexpr int kKeep = 19;
    __device__ static float at(const uint16_t *row, int64_t i)
    {
        return __uint_as_float((uint32_t)row[i] << 16);
    }
    __device__ static void unpack(u32x4_t v, float (&x)[kVec])
    {
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            x[2 * e] = bf16_lo(v[e]);
            x[2 * e + 1] = bf16_hi(v[e]);
        }
    }
};

// 2^x and log2 x on the VALU's transcendental unit (v_exp_f32 / v_log_f32).  The rate is
// computed in the base-2 domain with the scale ts = |tau| log2(e) folded into each
// exponent's FMA: 2^(ts x - m) is one v_fma_f32 and one v_exp_f32 per element, and the
// running maximum is taken on the unscaled values (ts >= 0 preserves their order; a
// negative tau is handled by negating the logits as they are read).
__device__ __forceinline__ float exp2_hw(float x) { return __builtin_amdgcn_exp2f(x); }
__device__ __forceinline__ float log2_hw(float x) { return __builtin_amdgcn_logf(x); }

// Running (max, sum of 2^(ts x - max)) of base-2-scaled logits (max on the scaled scale).
struct Lse {
    float m, s;
};

// A base-2 log-sum-exp m + log2 s as a rounded value and what the rounding left out.  The value
// is tens where its exponents' differences matter to 2^-23, so its rounding alone was most of
// the rate's error (4e-7); s is split into exponent and mantissa because log2 of the whole
// would round at the same place.
struct LogSum {
    float hi, lo;
};

__device__ __forceinline__ LogSum log_sum(Lse a)
{
    const int e = __builtin_amdgcn_frexp_expf(a.s);
    const float f = log2_hw(__builtin_amdgcn_frexp_mantf(a.s));  // in [-1, 0)
    // two exact sums (Knuth): m + e, then + f
    const float x = (float)e;
    const float s = a.m + x, xs = s - a.m;
    const float r = (a.m - (s - xs)) + (x - xs);
    const float t = s + f, ft = t - s;
    return {t, ((s - (t - ft)) + (f - ft)) + r};
}

// The factor that makes up for the roundings of both rows' log-sum-exps: exact where the two
// rows share the rate's mass evenly, as they do near 1, and at most the larger of the two roundings off.
__device__ __forceinline__ float rounding_factor(LogSum p, LogSum q)
{
    return exp2_hw(-0.5f * (p.lo + q.lo));
}

__device__ __forceinline__ Lse lse_merge(Lse a, Lse b)
{
    const float m = fmaxf(a.m, b.m);
    if (m == -INFINITY)
        return {m, 0.f};
    return {m, a.s * exp2_hw(a.m - m) + b.s * exp2_hw(b.m - m)};
}

// Moves the reference up to m (>= a.m).
__device__ __forceinline__ void lse_raise(Lse &a, float m)
{
    if (m > a.m) {
        a.s = a.m == -INFINITY ? 0.f : a.s * exp2_hw(a.m - m);
        a.m = m;
    }
}

// Adds the unscaled values x (scale ts >= 0) to the running log-sum-exp.
template <int N>
__device__ __forceinline__ void lse_add(Lse &r, const float (&x)[N], float ts)
{
    float mx = x[0];
#pragma unroll
    for (int e = 1; e < N; ++e)
        mx = fmaxf(mx, x[e]);
    mx *= ts;
    lse_raise(r, mx);
    // While every entry seen is -inf (masked vocabulary entries), the chunk adds nothing:
    // 2^(x - 0) = 0 for x = -inf, where x - r.m would be -inf - (-inf) = NaN.
    const float m = r.m == -INFINITY ? 0.f : r.m;
    float s = 0.f;
#pragma unroll
    for (int e = 0; e < N; ++e)
        s += exp2_hw(fmaf(ts, x[e], -m));
    r.s += s;
}

template <typename T>
__device__ __forceinline__ void row_split(const T *row, int V, int &head, int &nvec)
{
    constexpr int W = Logit<T>::kVec;
    const uintptr_t mis = reinterpret_cast<uintptr_t>(row) & 15u;
    head = mis == 0 ? 0 : (int)((16u - mis) / sizeof(T));
    if (head > V)
        head = V;
    nvec = (V - head) / W;
}

// The wave's log-sum-exp, in every lane.
__device__ __forceinline__ Lse wave_lse(Lse a)
{
    const float m = wave_max_f(a.m);
    const float s = wave_sum_f(a.m == -INFINITY ? 0.f : a.s * exp2_hw(a.m - m));
    return {m, s};
}

// Logit as read, negated when the inverse temperature is negative (so that the scale ts
// applied to it is >= 0).
template <bool kNeg>
__device__ __forceinline__ float oriented(float x)
{
    return kNeg ? -x : x;
}

// A vector's values (as read, scale ts >= 0) into the running log-sum-exp, without the
// running maximum: the sum is scale free, so the reference m only has to be near the largest
// terms (a term 2^u with large u carries u's rounding, so u stays below 8 to keep that under
// 2^-22).  While the vector's own sum is at most 2^8 its entries cost one FMA, one exp and
// one add each; a larger sum, an infinite one (nothing seen yet: m = -inf) or a NaN (only
// masked entries seen) takes lse_add, which moves the reference to the vector's maximum.
template <int N>
__device__ __forceinline__ void lse_add_fast(Lse &r, const float (&x)[N], float ts)
{
    float s = exp2_hw(fmaf(ts, x[0], -r.m));
#pragma unroll
    for (int e = 1; e < N; ++e)
        s += exp2_hw(fmaf(ts, x[e], -r.m));
    if (s <= 0x1p8f)
        r.s += s;
    else
        lse_add(r, x, ts);
}

template <typename T, bool kNeg>
__device__ __forceinline__ void lse_add_vec(Lse &a, Lse &b, u32x4_t va, u32x4_t vb, float ts)
{
    constexpr int W = Logit<T>::kVec;
    float xa[W], xb[W];
    Logit<T>::unpack(va, xa);
    Logit<T>::unpack(vb, xb);
#pragma unroll
    for (int e = 0; e < W; ++e) {
        xa[e] = oriented<kNeg>(xa[e]);
        xb[e] = oriented<kNeg>(xb[e]);
    }
    lse_add_fast(a, xa, ts);
    lse_add_fast(b, xb, ts);
}

// sum over the vector's entries of 2^min(ts a - P, ts b - Q)
template <typename T, bool kNeg>
__device__ __forceinline__ float min_sum_vec(u32x4_t va, u32x4_t vb, float ts, float P, float Q)
{
    constexpr int W = Logit<T>::kVec;
    float xa[W], xb[W];
    Logit<T>::unpack(va, xa);
    Logit<T>::unpack(vb, xb);
    float acc = 0.f;
#pragma unroll
    for (int e = 0; e < W; ++e)
        acc += exp2_hw(fminf(fmaf(ts, oriented<kNeg>(xa[e]), -P),
                             fmaf(ts, oriented<kNeg>(xb[e]), -Q)));
    return acc;
}

// One token's row pair as a thread sees it: 16-byte vectors v = tid + slot * kAccThreads of both
// rows, and at most one element of the unaligned head or tail.
template <typename T, bool kNeg>
struct RowPair {
    const u32x4_t *pv, *qv;
    int nvec;
    bool odd;      // this thread has an element outside the vectors
    float oa, ob;  // that element of both rows

    __device__ __forceinline__ void open(const T *target, const T *draft, int64_t t, int V)
    {
        const T *pr = target + t * V;
        const T *qr = draft + t * V;
        int head;
        row_split(pr, V, head, nvec);
        const int tail0 = head + nvec * Logit<T>::kVec;
        const int tid = threadIdx.x;
        const int i = tid < head ? tid : tail0 + tid - head;  // (head and tail: under 16 each)
        odd = i < V && (tid < head || i >= tail0);
        oa = ob = 0.f;
        if (odd) {
            oa = oriented<kNeg>(Logit<T>::at(pr, i));
            ob = oriented<kNeg>(Logit<T>::at(qr, i));
        }
        pv = reinterpret_cast<const u32x4_t *>(pr + head);
        qv = reinterpret_cast<const u32x4_t *>(qr + head);
    }
    __device__ __forceinline__ bool has(int slot) const
    {
        return (int)threadIdx.x + slot * kAccThreads < nvec;
    }
    // The slot's vectors of both rows.  Every load is unconditional: a thread past the row
    // repeats its last vector, a slot past it reads slot 0.  (The slot's start is uniform, so
    // a load needs one 32-bit register of its own for its address.)
    template <bool kOnce>
    __device__ __forceinline__ void load(int slot, u32x4_t &a, u32x4_t &b) const
    {
        int left = nvec - 1 - slot * kAccThreads;
        const int64_t start = left < 0 ? 0 : (int64_t)slot * kAccThreads;
        left = left < 0 ? nvec - 1 : left;
        const uint32_t off = 16u * (uint32_t)min((int)threadIdx.x, left);
        const char *pa = reinterpret_cast<const char *>(pv + start);
        const char *pb = reinterpret_cast<const char *>(qv + start);
        a = kOnce ? ld16_nt(pa + off) : ld16(pa + off);
        b = kOnce ? ld16_nt(pb + off) : ld16(pb + off);
    }
};

template <typename T, bool kNeg, bool kOnce>
__global__ __launch_bounds__(kAccThreads) void k_acceptance(const T *__restrict__ target,
                                                            const T *__restrict__ draft, int tokens,
                                                            int V, float ts,
                                                            float *__restrict__ alpha)
{
    extern __shared__ u32x4_t s_keep[];  // [2][kAccLdsVecs][kAccThreads]
    __shared__ Lse s_red[2][kAccWaves][2];
    __shared__ float s_sum[2][kAccWaves];
    constexpr int R = Logit<T>::kKeep, L = kAccLdsVecs, NB = kAccBatch;
    static_assert(L % NB == 0, "an LDS group is whole");
    const int tid = threadIdx.x;
    const int wave = tid >> 6;
    const int lane = tid & 63;

    RowPair<T, kNeg> x;
    u32x4_t ka[R], kb[R];          // slots L .. L + R - 1 of the current token
    u32x4_t na[NB], nb[NB];        // a group of the others, in flight
    // Group g of the slots that are not kept: slots g NB .., with the kept ones skipped.
    auto slot_of = [&](int g, int u) {
        const int i = g * NB + u;
        return i < L ? i : i + R;
    };
    auto load_loose = [&](const RowPair<T, kNeg> &r, int g, int u, auto again) {
        r.template load<decltype(again)::value>(slot_of(g, u), na[u], nb[u]);
    };
    auto load_kept = [&](const RowPair<T, kNeg> &r, int j) {
        r.template load<kOnce>(L + j, ka[j], kb[j]);
    };
    constexpr std::false_type kFirst{};
    constexpr std::true_type kAgain{};

    int t = blockIdx.x;
    x.open(target, draft, t, V);
#pragma unroll
    for (int j = 0; j < R; ++j)
        load_kept(x, j);
#pragma unroll
    for (int u = 0; u < NB; ++u)
        load_loose(x, 0, u, kFirst);

    for (int round = 0;; round ^= 1) {
        const int nslots = (x.nvec + kAccThreads - 1) / kAccThreads;
        const int loose = nslots <= L ? nslots : (nslots <= L + R ? L : nslots - R);
        const int groups = (loose + NB - 1) / NB;

        // ---- pass 1: log-sum-exp of both rows
        Lse a{-INFINITY, 0.f}, b{-INFINITY, 0.f};
#pragma unroll
        for (int j = 0; j < R; ++j) {
            if (x.has(L + j))
                lse_add_vec<T, kNeg>(a, b, ka[j], kb[j], ts);
            if (j == 0) {  // the reference of the whole wave, so few later vectors exceed it
                lse_raise(a, wave_max_f(a.m));
                lse_raise(b, wave_max_f(b.m));
            }
        }
        if (x.odd) {
            const float xa[1] = {x.oa}, xb[1] = {x.ob};
            lse_add(a, xa, ts);
            lse_add(b, xb, ts);
        }
        // The sums so far are put aside here and after every kAccFold groups: one sum of all of a
        // thread's vectors (74 of Qwen3's vocabulary in fp32) would be a chain whose roundings
        // show where one entry holds most of the mass.
        Lse pa = a, pb = b;
        a.s = b.s = 0.f;
        // The other slots roll through na, nb: each is replaced by its successor as soon as it
        // is used, and the last group stays for the second pass, which goes back to front.
        auto first_use = [&](int g, int u) {
            if (x.has(slot_of(g, u)))
                lse_add_vec<T, kNeg>(a, b, na[u], nb[u], ts);
            if (g < L / NB) {
                s_keep[(g * NB + u) * kAccThreads + tid] = na[u];
                s_keep[(L + g * NB + u) * kAccThreads + tid] = nb[u];
            }
        };
        for (int g = 0; g + 1 < groups; ++g) {
#pragma unroll
            for (int u = 0; u < NB; ++u) {
                first_use(g, u);
                load_loose(x, g + 1, u, kFirst);
            }
            if ((g + 1) % kAccFold == 0) {
                pa = lse_merge(pa, a);
                pb = lse_merge(pb, b);
                a.s = b.s = 0.f;
            }
        }
#pragma unroll
        for (int u = 0; u < NB; ++u)
            first_use(groups - 1, u);
        a = wave_lse(lse_merge(pa, a));
        b = wave_lse(lse_merge(pb, b));
        if (lane == 0) {
            s_red[round][wave][0] = a;
            s_red[round][wave][1] = b;
        }
        __syncthreads();  // (the rounds alternate buffers: one barrier per token)
        a = s_red[round][0][0];
        b = s_red[round][0][1];
#pragma unroll
        for (int w = 1; w < kAccWaves; ++w) {
            a = lse_merge(a, s_red[round][w][0]);
            b = lse_merge(b, s_red[round][w][1]);
        }
        const LogSum lp = log_sum(a), lq = log_sum(b);  // of the scaled rows
        const float P = lp.hi, Q = lq.hi;
        if (tid == 0 && t != (int)blockIdx.x) {  // the previous token's waves are all in
            float total = 0.f;
            for (int w = 0; w < kAccWaves; ++w)
                total += s_sum[round ^ 1][w];
            alpha[t - gridDim.x] = total;
        }

        // ---- pass 2: sum of 2^min(ts a - P, ts b - Q), the other slots first (the last group
        // is still here), then LDS, then the kept slots, each replaced by the next token's
        float acc = 0.f, aside = 0.f;  // (put aside as in the first pass)
        if (x.odd)
            acc += exp2_hw(fminf(fmaf(ts, x.oa, -P), fmaf(ts, x.ob, -Q)));
        auto second_use = [&](int g, int u) {
            if (x.has(slot_of(g, u)))
                acc += min_sum_vec<T, kNeg>(na[u], nb[u], ts, P, Q);
        };
        if (groups > L / NB) {
            for (int g = groups - 1; g > L / NB; --g) {
#pragma unroll
                for (int u = 0; u < NB; ++u) {
                    second_use(g, u);
                    load_loose(x, g - 1, u, kAgain);
                }
                if (g % kAccFold == 0) {
                    aside += acc;
                    acc = 0.f;
                }
            }
#pragma unroll
            for (int u = 0; u < NB; ++u)
                second_use(L / NB, u);
        }
#pragma unroll
        for (int u = 0; u < L; ++u)
            if (x.has(u))
                acc += min_sum_vec<T, kNeg>(s_keep[u * kAccThreads + tid],
                                            s_keep[(L + u) * kAccThreads + tid], ts, P, Q);
        aside += acc;
        acc = 0.f;
        const int64_t tn = (int64_t)t + gridDim.x;
        const bool more = tn < tokens;
        RowPair<T, kNeg> y = x;
        if (more) {
            y.open(target, draft, tn, V);
#pragma unroll
            for (int j = 0; j < R; ++j) {
                if (x.has(L + j))
                    acc += min_sum_vec<T, kNeg>(ka[j], kb[j], ts, P, Q);
                load_kept(y, j);
            }
#pragma unroll
            for (int u = 0; u < NB; ++u)
                load_loose(y, 0, u, kFirst);
        } else {
#pragma unroll
            for (int j = 0; j < R; ++j)
                if (x.has(L + j))
                    acc += min_sum_vec<T, kNeg>(ka[j], kb[j], ts, P, Q);
        }
        acc = wave_sum_f(acc + aside) * rounding_factor(lp, lq);
        if (lane == 0)
            s_sum[round][wave] = acc;
        if (!more)
            break;
        t = (int)tn;
        x = y;
    }
    __syncthreads();
    if (tid == 0) {
        float total = 0.f;
        // (the last round's buffer: rounds alternate from 0)
        const int last = ((tokens - 1 - (int)blockIdx.x) / (int)gridDim.x) & 1;
        for (int w = 0; w < kAccWaves; ++w)
            total += s_sum[last][w];
        alpha[t] = total;
    }
}

// Rows of fewer than kAccSmallVocab entries: one wave per token, one entry per lane.
template <typename T, bool kNeg>
__global__ __launch_bounds__(64) void k_acceptance_small(const T *__restrict__ target,
                                                         const T *__restrict__ draft, int V,
                                                         float ts, float *__restrict__ alpha)
{
    const int64_t t = blockIdx.x;
    const int i = threadIdx.x;
    Lse a{-INFINITY, 0.f}, b{-INFINITY, 0.f};
    float xa[1] = {0.f}, xb[1] = {0.f};
    if (i < V) {
        xa[0] = oriented<kNeg>(Logit<T>::at(target + t * V, i));
        xb[0] = oriented<kNeg>(Logit<T>::at(draft + t * V, i));
        lse_add(a, xa, ts);
        lse_add(b, xb, ts);
    }
    a = wave_lse(a);
    b = wave_lse(b);
    const LogSum lp = log_sum(a), lq = log_sum(b);
    const float acc =
        wave_sum_f(i < V ? exp2_hw(fminf(fmaf(ts, xa[0], -lp.hi), fmaf(ts, xb[0], -lq.hi)))
                         : 0.f) *
        rounding_factor(lp, lq);
    if (i == 0)
        alpha[t] = acc;
}

__global__ __launch_bounds__(256) void k_acceptance_topk(const float *__restrict__ lp_target,
                                                         const float *__restrict__ lp_draft,
                                                         int64_t T, int K,
                                                         float *__restrict__ alpha)
{
    for (int64_t t = blockIdx.x * 256ll + threadIdx.x; t < T; t += (int64_t)gridDim.x * 256) {
        float acc = 0.f;
        for (int i = 0; i < K; ++i)
            acc += __expf(fminf(lp_target[t * K + i], lp_draft[t * K + i]));
        alpha[t] = acc;
    }
}

// fp32 -> uint32 whose unsigned order is the order of the values (-0 == +0).
__device__ __forceinline__ uint32_t float_key(float s)
{
    uint32_t u = __float_as_uint(s);
    if (u == 0x80000000u)
        u = 0u;
    return (u & 0x80000000u) ? ~u : (u | 0x80000000u);
}

__device__ __forceinline__ float key_float(uint32_t k)
{
    return __uint_as_float((k & 0x80000000u) ? (k & 0x7fffffffu) : ~k);
}

__device__ __forceinline__ int bin_of(int32_t pos, int bin_tokens, int n_bins)
{
    if (pos < 0)
        return -1;
    const int b = pos / bin_tokens;
    return b > n_bins - 1 ? n_bins - 1 : b;
}

constexpr int kTailKeep = 8;  // tokens per thread whose keys stay in registers

// One workgroup per bin.  The first kTailKeep tokens of every thread (8192 in all) are loaded
// once, together; later ones are read again by every pass.  At these sizes the kernel is a
// chain of block-wide steps, so their number and length decide it: the radix select starts at
// the highest bit where the bin's keys differ, finds a digit with one wave scan, and the two
// order statistics come from one pass after it.  4096 tokens in 20 bins: 45 us with one thread
// walking each digit's 256 counts and six passes over the tokens in memory, 9 us now.
__global__ __launch_bounds__(kTailThreads) void k_tail_stats(
    const float *__restrict__ alpha, const int32_t *__restrict__ pos, int64_t T, int bin_tokens,
    int n_bins, double pct, double *__restrict__ quantile, double *__restrict__ mean,
    int64_t *__restrict__ count)
{
    __shared__ unsigned long long hist[2][256];  // (a bin may hold more than 2^32 tokens)
    __shared__ double s_sum[kTailWaves];
    __shared__ unsigned long long s_cnt[kTailWaves];
    __shared__ uint32_t s_min[kTailWaves], s_max[kTailWaves];
    __shared__ uint32_t s_first[kTailWaves], s_above[kTailWaves];
    __shared__ uint32_t s_digit;
    __shared__ int64_t s_rank;
    __shared__ int64_t s_in_digit;
    const int bin = blockIdx.x;
    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int wave = tid >> 6;

    // ---- count, sum (each thread's tokens in order) and the range of the keys
    float x[kTailKeep];
    uint32_t in = 0;  // bit j: the thread's j-th token belongs to the bin
    {
        int32_t p[kTailKeep];
#pragma unroll
        for (int j = 0; j < kTailKeep; ++j) {
            const int64_t t = tid + (int64_t)j * kTailThreads;
            p[j] = t < T ? pos[t] : -1;
            x[j] = t < T ? alpha[t] : 0.f;
        }
#pragma unroll
        for (int j = 0; j < kTailKeep; ++j)
            in |= (uint32_t)(bin_of(p[j], bin_tokens, n_bins) == bin) << j;
    }
    // f(value) for every token of this thread in the bin, in token order
    auto each = [&](auto f) {
#pragma unroll
        for (int j = 0; j < kTailKeep; ++j)
            if (in >> j & 1)
                f(x[j]);
        for (int64_t t = tid + (int64_t)kTailKeep * kTailThreads; t < T; t += kTailThreads)
            if (bin_of(pos[t], bin_tokens, n_bins) == bin)
                f(alpha[t]);
    };
    double sum = 0.0;
    unsigned long long cnt = 0;
    uint32_t kmin = 0xffffffffu, kmax = 0u;
    each([&](float v) {
        sum += (double)v;
        ++cnt;
        const uint32_t key = float_key(v);
        kmin = min(kmin, key);
        kmax = max(kmax, key);
    });
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
        sum += __shfl_xor(sum, o, 64);
        cnt += __shfl_xor(cnt, o, 64);
    }
    kmin = wave_min(kmin);
    kmax = wave_max(kmax);
    if (lane == 0) {
        s_sum[wave] = sum;
        s_cnt[wave] = cnt;
        s_min[wave] = kmin;
        s_max[wave] = kmax;
    }
    if (tid < 256)
        hist[0][tid] = 0;
    __syncthreads();
    double total = 0.0;
    int64_t N = 0;
    for (int w = 0; w < kTailWaves; ++w) {
        total += s_sum[w];
        N += (int64_t)s_cnt[w];
        kmin = min(kmin, s_min[w]);
        kmax = max(kmax, s_max[w]);
    }
    if (N == 0) {
        if (tid == 0) {
            count[bin] = 0;
            mean[bin] = __builtin_nan("");
            quantile[bin] = __builtin_nan("");
        }
        return;
    }

    // ---- rank lo: a radix select over 8-bit digits.  After a digit the candidates are the keys
    // in [prefix, prefix + 2^shift), `rank` of them below the wanted one; a single one ends it.
    const double h = (double)(N - 1) * pct / 100.0;
    int64_t lo = (int64_t)floor(h);
    if (lo > N - 1)
        lo = N - 1;
    int64_t rank = lo;
    int64_t in_digit = N;
    int hi = kmin == kmax ? -1 : 31 - __builtin_clz(kmin ^ kmax);  // highest undecided bit
    uint32_t prefix = hi < 0 ? kmin : kmin & ~(0xffffffffu >> (31 - hi));
    for (int cur = 0; hi >= 0 && in_digit > 1; cur ^= 1) {
        const int shift = hi >= 7 ? hi - 7 : 0;
        const uint32_t mask = 0xffffffffu >> (31 - hi);  // bits hi .. 0
        each([&](float v) {
            const uint32_t key = float_key(v);
            if ((key & ~mask) == prefix)
                atomicAdd(&hist[cur][(key & mask) >> shift], 1ull);
        });
        if (tid < 256)
            hist[cur ^ 1][tid] = 0;
        __syncthreads();
        if (wave == 0) {  // lane l owns digits 4l .. 4l + 3
            int64_t c[4];
            int64_t before = 0;
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                c[i] = (int64_t)hist[cur][4 * lane + i];
                before += c[i];
            }
            const int64_t own = before;
#pragma unroll
            for (int o = 1; o < 64; o <<= 1) {
                const int64_t up = __shfl_up((long long)before, o, 64);
                before += lane >= o ? up : 0;
            }
            before -= own;
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                if (rank >= before && rank < before + c[i]) {
                    s_digit = 4 * lane + i;
                    s_rank = rank - before;
                    s_in_digit = c[i];
                }
                before += c[i];
            }
        }
        __syncthreads();
        prefix |= s_digit << shift;
        rank = s_rank;
        in_digit = s_in_digit;
        hi = shift - 1;
    }

    // ---- x_lo is the smallest key from prefix on; x_hi the same key again if more than
    // rank + 1 candidates equal it, else the next larger key
    uint32_t first = prefix, above = 0xffffffffu;
    if (hi >= 0) {  // one candidate left, some of its bits unknown
        first = 0xffffffffu;
        each([&](float v) {
            const uint32_t key = float_key(v);
            if (key >= prefix && key < first) {
                above = first;
                first = key;
            } else if (key >= prefix && key < above) {
                above = key;  // (an equal key would be a second candidate)
            }
        });
    } else {
        each([&](float v) {
            const uint32_t key = float_key(v);
            if (key > prefix && key < above)
                above = key;
        });
    }
    const uint32_t own_first = first, own_above = above;
    first = wave_min(first);
    if (lane == 0)
        s_first[wave] = first;
    __syncthreads();
    for (int w = 0; w < kTailWaves; ++w)
        first = min(first, s_first[w]);
    // the thread that holds the smallest key offers its second one
    above = wave_min(own_first > first ? min(own_first, own_above) : own_above);
    if (lane == 0)
        s_above[wave] = above;
    __syncthreads();
    for (int w = 0; w < kTailWaves; ++w)
        above = min(above, s_above[w]);
    if (tid == 0) {
        // the definition's separate multiply and add (device code otherwise contracts to fma)
#pragma clang fp contract(off)
        const double x_lo = (double)key_float(first);
        const bool again = hi < 0 && rank + 1 < in_digit;
        const double x_hi = lo + 1 >= N || again ? x_lo : (double)key_float(above);
        count[bin] = N;
        mean[bin] = total / (double)N;
        quantile[bin] = x_lo + (h - (double)lo) * (x_hi - x_lo);
    }
}

}  // namespace

int device_cus()
{
    int dev = 0, cus = 0;
    if (hipGetDevice(&dev) != hipSuccess ||
        hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess ||
        cus < 1)
        cus = 256;
    return cus;
}

hipError_t launch_acceptance(int64_t T, int V, int dtype, const void *target, const void *draft,
                             float tau, float *alpha, hipStream_t stream)
{
    // The vectors kept in LDS between the passes (144 KiB: one workgroup per CU).
    constexpr size_t kKeep = 2 * (size_t)kAccLdsVecs * kAccThreads * sizeof(u32x4_t);
    const bool neg = tau < 0.f;
    const float ts = (neg ? -tau : tau) * 1.44269504088896340736f;  // |tau| log2(e)
    auto go = [&](auto type) {
        using L = decltype(type);
        const L *p = static_cast<const L *>(target), *q = static_cast<const L *>(draft);
        if (V < kAccSmallVocab) {
            hipLaunchKernelGGL((neg ? k_acceptance_small<L, true> : k_acceptance_small<L, false>),
                               dim3((unsigned)T), dim3(64), 0, stream, p, q, V, ts, alpha);
            return;
        }
        // Non-temporal loads of the kept vectors leave the caches to the others, which are read
        // again; a few tokens find all of theirs in the caches.  fp32, plain / non-temporal, us:
        // 16 tokens of 62000 entries 16.1 / 19.1, 16 of 151936 33.0 / 35.5, 64 of 65536 17.8 /
        // 20.2, 64 of 151936 42.2 / 40.5, 128 of 80000 28.1 / 26.5, 256 of 131072 65.4 / 60.4;
        // bf16 16 of 151936 28.6 / 30.4, 128 of 131072 29.8 / 29.6, 256 39.1 / 38.1.
        const int cus = device_cus();
        const bool once = T >= cus / 2 &&
                          V / Logit<L>::kVec > (Logit<L>::kKeep + kAccLdsVecs) * kAccThreads;
        auto kernel = once ? (neg ? k_acceptance<L, true, true> : k_acceptance<L, false, true>)
                           : (neg ? k_acceptance<L, true, false> : k_acceptance<L, false, false>);
        hipLaunchKernelGGL(kernel, dim3((unsigned)(T < cus ? T : cus)), dim3(kAccThreads), kKeep,
                           stream, p, q, (int)T, V, ts, alpha);
    };
    if (dtype == SPARROW_LOGITS_BF16)
        go(uint16_t{});
    else
        go(float{});
    return hipGetLastError();
}

hipError_t launch_acceptance_topk(int64_t T, int K, const float *lp_target, const float *lp_draft,
                                  float *alpha, hipStream_t stream)
{
    int64_t blocks = (T + 255) / 256;
    if (blocks > 65535)
        blocks = 65535;
    hipLaunchKernelGGL(k_acceptance_topk, dim3((unsigned)blocks), dim3(256), 0, stream, lp_target,
                       lp_draft, T, K, alpha);
    return hipGetLastError();
}

hipError_t launch_tail_stats(int64_t T, const float *alpha, const int32_t *pos, int bin_tokens,
                             int n_bins, double pct, double *quantile, double *mean,
                             int64_t *count, hipStream_t stream)
{
    hipLaunchKernelGGL(k_tail_stats, dim3(n_bins), dim3(kTailThreads), 0, stream, alpha, pos, T,
                       bin_tokens, n_bins, pct, quantile, mean, count);
    return hipGetLastError();
}

}  // namespace sparrow
