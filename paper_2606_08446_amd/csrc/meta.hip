// Per-page key metadata: channel-wise min and max of each page's keys (the page landmark
// that block top-k selection scores, Sec. 3.3 / Appendix C of arXiv 2606.08446).
//
// k_meta_minmax builds large caches of 16-token pages; k_meta_update does the rest:
// one workgroup per (sequence, logical page) when rebuilding, or per sequence when
// updating the pages touched by freshly written tokens.  A thread owns one (KV head,
// 8-channel slice): it streams the slice of every valid token of the page (16 bytes per
// token, the 16 threads of a head covering one contiguous 256-byte key row), keeps
// min/max in registers and writes two 16-byte rows.  Min/max run on an integer image of
// the bf16 bit pattern whose order is the total order of the values (-0 below +0), so
// the result is one of the input patterns, bit for bit.
//
// With the mean landmark the thread instead sums its 8 channels over the page's tokens in
// token order (fp32 adds of exactly converted bf16 keys) and writes 8 fp32 sums.
#include "common.h"
#include "wave.h"

namespace sparrow {
namespace {

constexpr int kMetaThreads = 128;

__device__ __forceinline__ void fold(u32x4_t v, int32_t (&mn)[8], int32_t (&mx)[8])
{
#pragma unroll
    for (int w = 0; w < 4; ++w) {
        const int32_t lo = order16(v[w] & 0xffffu);
        const int32_t hi = order16(v[w] >> 16);
        mn[2 * w] = min(mn[2 * w], lo);
        mx[2 * w] = max(mx[2 * w], lo);
        mn[2 * w + 1] = min(mn[2 * w + 1], hi);
        mx[2 * w + 1] = max(mx[2 * w + 1], hi);
    }
}

// Min/max of one (page, head, 8-channel slice) over `valid` tokens of a page of PS tokens.
template <int PS>
__device__ __forceinline__ void slice_minmax(const uint16_t *__restrict__ src, int valid,
                                             uint16_t *__restrict__ dst)
{
    int32_t mn[8], mx[8];
#pragma unroll
    for (int e = 0; e < 8; ++e) {
        mn[e] = 0x7fffffff;
        mx[e] = -0x7fffffff - 1;
    }
    // 16 tokens at a time: all loads of a batch are independent and issue together.
    for (int t0 = 0; t0 < PS; t0 += 16) {
        if (t0 >= valid)
            break;
        u32x4_t v[16];
        v[0] = ld16_nt(src + (size_t)t0 * kHeadDim);
#pragma unroll
        for (int t = 1; t < 16; ++t)
            v[t] = (t0 + t < valid) ? ld16_nt(src + (size_t)(t0 + t) * kHeadDim) : v[0];
        // token t0 is valid; re-folding it for slots past the length changes nothing.
#pragma unroll
        for (int t = 0; t < 16; ++t)
            fold(v[t], mn, mx);
    }
    u32x4_t lo, hi;
#pragma unroll
    for (int w = 0; w < 4; ++w) {
        lo[w] = unorder16(mn[2 * w]) | (unorder16(mn[2 * w + 1]) << 16);
        hi[w] = unorder16(mx[2 * w]) | (unorder16(mx[2 * w + 1]) << 16);
    }
    st16(dst, lo);
    st16(dst + kHeadDim, hi);
}

typedef short s16x2_t __attribute__((ext_vector_type(2)));

// order16 on the two bf16 patterns of a word, and back (the map is an involution).
__device__ __forceinline__ s16x2_t order16x2(uint32_t word)
{
    const s16x2_t s = __builtin_bit_cast(s16x2_t, word);
    return s ^ ((s >> (short)15) & (short)0x7fff);
}

__device__ __forceinline__ uint32_t unorder16x2(s16x2_t s)
{
    return __builtin_bit_cast(uint32_t, order16x2(__builtin_bit_cast(uint32_t, s)));
}

constexpr int kMinmaxThreads = 512;
constexpr int kMinmaxWaves = kMinmaxThreads / 64;
constexpr int kMinmaxRows = 256;  // landmark rows a workgroup holds in LDS (128 KiB)
constexpr int64_t kMinmaxBytes = 1ll << 30;  // key bytes from which the burst kernel is used
constexpr int kMinmaxBatch = 4096;  // sequences whose page offsets fit LDS beside the rows

// Min/max landmarks of 16-token pages in large builds, one workgroup per CU.  Memory-bound, and
// bound by its writes more than by its reads: landmark rows (512 B per 4 KiB of keys) trickling
// out between the key reads cost the reads a third of their rate.  So a workgroup keeps the rows
// of a chunk of pages (kMinmaxRows rows; one lane per page) in LDS and writes them in one burst
// of non-temporal stores, and the workgroups, which start together and work alike, stay in step
// so that bursts meet bursts (the first chunks staggered by halves, quarters or eighths: 3, 5
// and 6 % slower).  2.7 GB of keys in 64 sequences of 8K-32K tokens: 615 us page by page, 568 so.
//
// The batch's pages are laid end to end and every workgroup takes an equal, contiguous share of
// them, whatever the lengths.  With a workgroup per (sequence, chunk) the empty ones behind a
// wide block table each waited for a CU of their own, between the full ones: 64 sequences of 300
// pages behind 2049-page rows 236 us, page by page 131, now 122; 32 of 300 behind 4097 123, 69,
// 66; 64 of 8 pages behind 2049 12, 34, 7.
//
// A wave takes whole (page, head) blocks: a load instruction reads four consecutive key rows
// (1 KiB), four of them a block, and the next block is in flight while one is folded.  Lane
// (r, c) folds channels 8c .. 8c+7 of the rows r mod 4 on packed 16-bit integers; two lane
// exchanges join the four row classes.  Rows past the length repeat the last valid one.
__global__ __launch_bounds__(kMinmaxThreads) void k_meta_minmax(
    const uint16_t *__restrict__ k_cache, const int32_t *__restrict__ block_table,
    const int32_t *__restrict__ seq_lens, uint16_t *__restrict__ meta, int batch,
    int num_kv_heads, int max_pages, int64_t num_phys, int most)
{
    constexpr int PS = 16;  // a page is one batch of four loads
    extern __shared__ u32x4_t s_out[];  // [most][heads][32], then the page offsets
    int32_t *s_off = reinterpret_cast<int32_t *>(s_out + kMinmaxRows * 32);  // [batch + 1]
    __shared__ int32_t s_scan[kMinmaxWaves];
    const int h0 = blockIdx.y * (kMinmaxRows / most);
    const int nh = min(kMinmaxRows / most, num_kv_heads - h0);
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int lane = threadIdx.x & 63;
    const int r = lane >> 4;
    const int c = lane & 15;

    // ---- page offsets of the sequences, each thread scanning its own few
    const int per = (batch + kMinmaxThreads - 1) / kMinmaxThreads;
    const int b0 = min(batch, (int)threadIdx.x * per);
    const int b1 = min(batch, b0 + per);
    int mine = 0;
    for (int b = b0; b < b1; ++b) {
        s_off[b] = mine;
        mine += (clamp_len(seq_lens[b], PS, max_pages) + PS - 1) / PS;
    }
    const int incl = (int)wave_scan_add((uint32_t)mine);
    if (lane == 63)
        s_scan[wave] = incl;
    __syncthreads();
    int before = incl - mine;
    for (int w = 0; w < wave; ++w)
        before += s_scan[w];
    for (int b = b0; b < b1; ++b)
        s_off[b] += before;
    if (threadIdx.x == kMinmaxThreads - 1)
        s_off[batch] = before + mine;
    __syncthreads();

    // ---- this workgroup's pages [lo, hi), `most` at a time
    const int64_t total = __builtin_amdgcn_readfirstlane(s_off[batch]);
    const int lo = (int)(total * blockIdx.x / gridDim.x);
    const int hi = (int)(total * (blockIdx.x + 1) / gridDim.x);
    if (lo == hi)
        return;
    // lane i: the physical page of page p0 + i, or -1 (absent), and its valid tokens
    auto locate = [&](int p0, int &phys, int &valid) {
        const int f = min(p0 + lane, hi - 1);
        int b = 0;  // the sequence with s_off[b] <= f < s_off[b + 1]
        for (int end = batch; end - b > 1;) {
            const int mid = (b + end) >> 1;
            if (s_off[mid] <= f)
                b = mid;
            else
                end = mid;
        }
        const int page = f - s_off[b];
        const int e = block_table[(int64_t)b * max_pages + page];
        phys = e >= 0 && e < num_phys ? e : -1;
        valid = min(PS, clamp_len(seq_lens[b], PS, max_pages) - page * PS);
    };
    int phys, valid;
    auto issue = [&](int s, u32x4_t (&v)[4]) {
        const int it = wave + kMinmaxWaves * s;
        const int pg = it / nh;
        const int h = h0 + it - pg * nh;
        const int ph = __builtin_amdgcn_readlane(phys, pg);
        const int rows = __builtin_amdgcn_readlane(valid, pg);
        const uint16_t *src =  // (an absent page reads page 0)
            k_cache + ((int64_t)(ph < 0 ? 0 : ph) * num_kv_heads + h) * PS * kHeadDim + 8 * c;
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const int row = 4 * j + r;
            v[j] = ld16_nt(src + (row < rows ? row : rows - 1) * kHeadDim);
        }
    };
    auto fold = [&](int s, const u32x4_t (&v)[4]) {
        s16x2_t mn[4], mx[4];
#pragma unroll
        for (int w = 0; w < 4; ++w)
            mn[w] = mx[w] = order16x2(v[0][w]);
#pragma unroll
        for (int j = 1; j < 4; ++j)
#pragma unroll
            for (int w = 0; w < 4; ++w) {
                const s16x2_t x = order16x2(v[j][w]);
                mn[w] = __builtin_elementwise_min(mn[w], x);
                mx[w] = __builtin_elementwise_max(mx[w], x);
            }
        u32x4_t out;
#pragma unroll
        for (int w = 0; w < 4; ++w) {
#pragma unroll
            for (int x = 16; x < 64; x <<= 1) {
                const int lo16 = __shfl_xor(__builtin_bit_cast(int, mn[w]), x, 64);
                const int hi16 = __shfl_xor(__builtin_bit_cast(int, mx[w]), x, 64);
                mn[w] = __builtin_elementwise_min(mn[w], __builtin_bit_cast(s16x2_t, lo16));
                mx[w] = __builtin_elementwise_max(mx[w], __builtin_bit_cast(s16x2_t, hi16));
            }
            out[w] = unorder16x2(r & 1 ? mx[w] : mn[w]);
        }
        if (lane < 32)  // lanes 0-15 the min row, 16-31 the max row
            s_out[(wave + kMinmaxWaves * s) * 32 + lane] = out;
    };
    // (page, head) blocks of the chunk at p0, page-major, and this wave's share of them
    auto blocks_of = [&](int p0) { return min(most, hi - p0) * nh; };
    auto steps_of = [&](int items) { return (items - wave + kMinmaxWaves - 1) / kMinmaxWaves; };

    locate(lo, phys, valid);
    int items = blocks_of(lo);
    int steps = steps_of(items);
    u32x4_t nxt[4];
    if (steps > 0)
        issue(0, nxt);
    for (int p0 = lo; p0 < hi; p0 += most) {
        const bool more = p0 + most < hi;
        int phys2 = -1, valid2 = 1;
        if (more)
            locate(p0 + most, phys2, valid2);
        int s = 0;
        for (; s + 1 < steps; ++s) {
            u32x4_t cur[4];
#pragma unroll
            for (int j = 0; j < 4; ++j)
                cur[j] = nxt[j];
            issue(s + 1, nxt);
            fold(s, cur);
        }
        if (s < steps)
            fold(s, nxt);
        __syncthreads();
        // the burst: a wave writes two landmark rows (1 KiB) per instruction (every lane takes
        // part in the exchange of the page's entry, also past the last row)
        for (int it0 = 2 * wave; it0 < items; it0 += 2 * kMinmaxWaves) {
            const int it = it0 + (lane >> 5);
            const int pg = (it < items ? it : items - 1) / nh;
            const int ph = __shfl(phys, pg, 64);
            if (it < items && ph >= 0)
                __builtin_nontemporal_store(s_out[it * 32 + (lane & 31)],
                                            reinterpret_cast<u32x4_t *>(meta) + (lane & 31) +
                                                ((int64_t)ph * num_kv_heads + h0 + it - pg * nh) * 32);
        }
        if (more) {  // (its first loads behind this wave's stores: before them costs 1 %)
            phys = phys2;
            valid = valid2;
            items = blocks_of(p0 + most);
            steps = steps_of(items);
            if (steps > 0)
                issue(0, nxt);
        }
        __syncthreads();  // the rows are out of LDS before the next chunk's arrive
    }
}

// Key sums of one (page, head, 8-channel slice) over `valid` tokens, in token order.
template <int PS>
__device__ __forceinline__ void slice_sum(const uint16_t *__restrict__ src, int valid,
                                          float *__restrict__ dst)
{
    float acc[8];
#pragma unroll
    for (int e = 0; e < 8; ++e)
        acc[e] = 0.f;
    for (int t0 = 0; t0 < PS; t0 += 16) {
        if (t0 >= valid)
            break;
        const int nt = valid - t0 < 16 ? valid - t0 : 16;
        u32x4_t v[16];
#pragma unroll
        for (int t = 0; t < 16; ++t)
            v[t] = (t < nt) ? ld16_nt(src + (size_t)(t0 + t) * kHeadDim) : (u32x4_t){0u, 0u, 0u, 0u};
#pragma unroll
        for (int t = 0; t < 16; ++t) {
            if (t < nt) {
#pragma unroll
                for (int w = 0; w < 4; ++w) {
                    acc[2 * w] += bf16_lo(v[t][w]);
                    acc[2 * w + 1] += bf16_hi(v[t][w]);
                }
            }
        }
    }
    st16(dst, __builtin_bit_cast(u32x4_t, (f32x4_t){acc[0], acc[1], acc[2], acc[3]}));
    st16(dst + 4, __builtin_bit_cast(u32x4_t, (f32x4_t){acc[4], acc[5], acc[6], acc[7]}));
}

template <int PS, bool kMean>
__global__ __launch_bounds__(kMetaThreads) void k_meta_update(
    const uint16_t *__restrict__ k_cache, const int32_t *__restrict__ block_table,
    const int32_t *__restrict__ seq_lens, const int32_t *__restrict__ first_pos,
    void *__restrict__ meta, int num_kv_heads, int max_pages, int64_t num_phys, int rebuild)
{
    const int b = rebuild ? blockIdx.y : blockIdx.x;
    const int L = clamp_len(seq_lens[b], PS, max_pages);
    const int n = (L + PS - 1) / PS;
    int p_begin, p_end;
    if (rebuild) {
        p_begin = blockIdx.x;
        p_end = p_begin + 1 < n ? p_begin + 1 : n;
    } else {
        int f = first_pos[b];
        f = f < 0 ? 0 : f;
        if (f >= L)
            return;
        p_begin = f / PS;
        p_end = n;
    }
    const int slices = num_kv_heads * (kHeadDim / 8);
    for (int p = p_begin; p < p_end; ++p) {
        const int64_t phys = block_table[(int64_t)b * max_pages + p];
        if (phys < 0 || phys >= num_phys)
            continue;  // an entry outside the cache: an absent page, nothing to build
        const int valid = L - p * PS < PS ? L - p * PS : PS;
        for (int u = threadIdx.x; u < slices; u += kMetaThreads) {
            const int h = u >> 4;
            const int c = u & 15;
            const uint16_t *src = k_cache + ((phys * num_kv_heads + h) * PS) * kHeadDim + c * 8;
            if (kMean) {
                float *dst = static_cast<float *>(meta) + (phys * num_kv_heads + h) * kHeadDim + c * 8;
                slice_sum<PS>(src, valid, dst);
            } else {
                uint16_t *dst = static_cast<uint16_t *>(meta) +
                                ((phys * num_kv_heads + h) * 2) * kHeadDim + c * 8;
                slice_minmax<PS>(src, valid, dst);
            }
        }
    }
}

template <int PS>
hipError_t launch_ps(const sparrow_shape_t &s, const void *k_cache, const int32_t *bt,
                     const int32_t *lens, const int32_t *first_pos, void *meta, hipStream_t st)
{
    const int rebuild = first_pos == nullptr;
    const int64_t page_bytes = (int64_t)s.num_kv_heads * PS * kHeadDim * 2;
    // A large build by bursts: never slower from 1 GiB of possible keys on.  Below it the shorter
    // chain of the page-per-workgroup kernel can be: one sequence of 1000 pages 7.6 us against
    // 8.2, 4 of 250 7.9 against 9.4, 64 of 30 13.6 against 15.7.
    if (PS == 16 && rebuild && s.landmark == SPARROW_LANDMARK_MINMAX &&
        s.batch <= kMinmaxBatch && page_bytes * s.max_pages_per_seq * s.batch >= kMinmaxBytes) {
        int most = kMinmaxRows / (s.num_kv_heads < kMinmaxRows ? s.num_kv_heads : kMinmaxRows);
        most = most < 64 ? most : 64;  // one lane per page
        const int heads = kMinmaxRows / most;  // per workgroup
        const dim3 grid(device_cus(), (s.num_kv_heads + heads - 1) / heads);
        const size_t lds = (size_t)kMinmaxRows * 2 * kHeadDim * sizeof(uint16_t) +
                           (size_t)(s.batch + 1) * sizeof(int32_t);
        hipLaunchKernelGGL(k_meta_minmax, grid, dim3(kMinmaxThreads), lds, st,
                           static_cast<const uint16_t *>(k_cache), bt, lens,
                           static_cast<uint16_t *>(meta), s.batch, s.num_kv_heads,
                           s.max_pages_per_seq, s.num_phys_pages, most);
        return hipGetLastError();
    }
    const dim3 grid = rebuild ? dim3(s.max_pages_per_seq, s.batch) : dim3(s.batch);
    if (s.landmark == SPARROW_LANDMARK_MEAN)
        hipLaunchKernelGGL((k_meta_update<PS, true>), grid, dim3(kMetaThreads), 0, st,
                           static_cast<const uint16_t *>(k_cache), bt, lens, first_pos, meta,
                           s.num_kv_heads, s.max_pages_per_seq, s.num_phys_pages, rebuild);
    else
        hipLaunchKernelGGL((k_meta_update<PS, false>), grid, dim3(kMetaThreads), 0, st,
                           static_cast<const uint16_t *>(k_cache), bt, lens, first_pos, meta,
                           s.num_kv_heads, s.max_pages_per_seq, s.num_phys_pages, rebuild);
    return hipGetLastError();
}

}  // namespace

hipError_t launch_meta_update(const sparrow_shape_t &s, const void *k_cache,
                              const int32_t *block_table, const int32_t *seq_lens,
                              const int32_t *first_pos, void *meta, hipStream_t stream)
{
    switch (s.page_size) {
    case 16: return launch_ps<16>(s, k_cache, block_table, seq_lens, first_pos, meta, stream);
    case 32: return launch_ps<32>(s, k_cache, block_table, seq_lens, first_pos, meta, stream);
    case 64: return launch_ps<64>(s, k_cache, block_table, seq_lens, first_pos, meta, stream);
    default: return launch_ps<128>(s, k_cache, block_table, seq_lens, first_pos, meta, stream);
    }
}

}  // namespace sparrow
