// gfx950 kernels of the graph builder (Fig. 1 data structures): an int64
// scan for row pointers, random Bernoulli and fixed-fan-out rows, grouping of
// an edge list by source, per-row LDS sort by (target, weight), and slice
// pivots with plastic prefixes.
#include "snn_device.h"

#include <algorithm>

namespace snn {
namespace {

// ---------------------------------------------------------------------------
// inclusive scan of int64 in place: chunks of 4*kBlock, chunk totals, offsets

constexpr int kScanChunk = 4 * kBlock;

__device__ long long block_incl_scan_i64(long long v, long long *sh)
{
    const int lane = threadIdx.x % kWave, wave = threadIdx.x / kWave;
#pragma unroll
    for (int off = 1; off < kWave; off <<= 1) {
        const long long u = __shfl_up(v, off, kWave);
        if (lane >= off) v += u;
    }
    __syncthreads();
    if (lane == kWave - 1) sh[wave] = v;
    __syncthreads();
    for (int q = 0; q < wave; ++q) v += sh[q];
    return v;
}

__global__ __launch_bounds__(kBlock) void k_scan_local(int64_t *d, int64_t count, int64_t *bsum)
{
    __shared__ long long sh[kBlock / kWave];
    const int64_t base = (int64_t)blockIdx.x * kScanChunk + threadIdx.x * 4;
    long long x[4];
#pragma unroll
    for (int q = 0; q < 4; ++q) x[q] = base + q < count ? d[base + q] : 0;
    x[1] += x[0];
    x[2] += x[1];
    x[3] += x[2];
    const long long incl = block_incl_scan_i64(x[3], sh);
    const long long excl = incl - x[3];
#pragma unroll
    for (int q = 0; q < 4; ++q)
        if (base + q < count) d[base + q] = x[q] + excl;
    if (threadIdx.x == kBlock - 1) bsum[blockIdx.x] = incl;
}

__global__ __launch_bounds__(kBlock) void k_scan_bsum(int64_t *bsum, int64_t nb)
{
    __shared__ long long sh[kBlock / kWave];
    __shared__ long long carry;
    if (threadIdx.x == 0) carry = 0;
    __syncthreads();
    for (int64_t b0 = 0; b0 < nb; b0 += kBlock) {
        const int64_t i = b0 + threadIdx.x;
        const long long v = i < nb ? bsum[i] : 0;
        const long long incl = block_incl_scan_i64(v, sh);
        const long long c = carry;
        if (i < nb) bsum[i] = c + incl - v;  // exclusive offsets
        __syncthreads();
        if (threadIdx.x == kBlock - 1) carry = c + incl;
        __syncthreads();
    }
}

__global__ __launch_bounds__(kBlock) void k_scan_add(int64_t *d, int64_t count, const int64_t *bsum)
{
    const long long off = bsum[blockIdx.x];
    const int64_t base = (int64_t)blockIdx.x * kScanChunk;
    for (int q = threadIdx.x; q < kScanChunk; q += kBlock)
        if (base + q < count) d[base + q] += off;
}

// ---------------------------------------------------------------------------
// graph builder (Fig. 1 data structures)

// Bernoulli rows: count the pairs (k, j), j != k, whose stream-0 draw is
// below the threshold; row_ptr[k+1] = count (scanned afterwards).
__global__ __launch_bounds__(kBlock) void k_count_bernoulli(GraphArgs a)
{
    __shared__ long long sh[kBlock / kWave];
    const int k = blockIdx.x;
    long long c = 0;
    for (int j = threadIdx.x; j < a.n; j += kBlock)
        c += (j != k) && rng32(a.seed, 0, (uint64_t)k, (uint64_t)j) < a.thr;
    c = block_sum_i64(c, sh);
    if (threadIdx.x == 0) {
        a.row_ptr[k + 1] = c;
        if (k == 0) a.row_ptr[0] = 0;
    }
}

// Bernoulli rows: write the present targets in ascending order (ballot-rank
// within each wave, wave offsets through LDS) with the source's weight.
__global__ __launch_bounds__(kBlock) void k_fill_bernoulli(GraphArgs a)
{
    __shared__ int s_wc[kBlock / kWave];
    const int k = blockIdx.x, tid = threadIdx.x;
    const int wave = tid / kWave, lane = tid % kWave;
    const int64_t base = a.row_ptr[k];
    const float wk = k < a.n_exc ? a.w_exc : a.w_inh;
    const uint64_t below = lane == 0 ? 0ull : (~0ull >> (64 - lane));
    int64_t off = 0;
    for (int j0 = 0; j0 < a.n; j0 += kBlock) {
        const int j = j0 + tid;
        const bool f = j < a.n && j != k && rng32(a.seed, 0, (uint64_t)k, (uint64_t)j) < a.thr;
        const uint64_t m = ballot64(f);
        if (lane == 0) s_wc[wave] = __popcll(m);
        __syncthreads();
        int pre = 0, tot = 0;
#pragma unroll
        for (int q = 0; q < kBlock / kWave; ++q) {
            pre += q < wave ? s_wc[q] : 0;
            tot += s_wc[q];
        }
        if (f) {
            const int64_t pos = base + off + pre + __popcll(m & below);
            a.col[pos] = j;
            a.w[pos] = wk;
        }
        off += tot;
        __syncthreads();
    }
}

__global__ __launch_bounds__(kBlock) void k_rowptr_fanout(GraphArgs a)
{
    const int64_t k = (int64_t)blockIdx.x * kBlock + threadIdx.x;
    if (k <= a.n) a.row_ptr[k] = k * a.fanout;
}

// Fixed fan-out: edge (k, b) targets (u32 * n) >> 32 of stream 1 at (k, b).
__global__ __launch_bounds__(kBlock) void k_fill_fanout(GraphArgs a)
{
    const int64_t total = (int64_t)a.n * a.fanout;
    const int64_t stride = (int64_t)gridDim.x * kBlock;
    for (int64_t e = (int64_t)blockIdx.x * kBlock + threadIdx.x; e < total; e += stride) {
        const int64_t k = e / a.fanout, b = e - k * a.fanout;
        const uint32_t u = rng32(a.seed, 1, (uint64_t)k, (uint64_t)b);
        a.col[e] = (int32_t)(((uint64_t)u * (uint64_t)a.n) >> 32);
        a.w[e] = k < a.n_exc ? a.w_exc : a.w_inh;
    }
}

// Edge list: validate indices and count per source into row_ptr[src+1].
__global__ __launch_bounds__(kBlock) void k_edges_count(GraphArgs a, const int32_t *src,
                                                        const int32_t *dst, int64_t e)
{
    const int64_t stride = (int64_t)gridDim.x * kBlock;
    for (int64_t i = (int64_t)blockIdx.x * kBlock + threadIdx.x; i < e; i += stride) {
        const int32_t s = src[i], d = dst[i];
        if (s < 0 || s >= a.n || d < 0 || d >= a.n) {
            atomicOr(a.err, kErrIndex);
            continue;
        }
        atomicAdd((unsigned long long *)(a.row_ptr + s + 1), 1ull);
    }
}

__global__ __launch_bounds__(kBlock) void k_edges_scatter(GraphArgs a, const int32_t *src,
                                                          const int32_t *dst, const float *w,
                                                          int64_t e, int64_t *cursor)
{
    const int64_t stride = (int64_t)gridDim.x * kBlock;
    for (int64_t i = (int64_t)blockIdx.x * kBlock + threadIdx.x; i < e; i += stride) {
        const int32_t s = src[i], d = dst[i];
        if (s < 0 || s >= a.n || d < 0 || d >= a.n) continue;
        const int64_t pos = (int64_t)atomicAdd((unsigned long long *)(cursor + s), 1ull);
        a.col[pos] = d;
        a.w[pos] = w[i];
    }
}

// Edge lists by buckets of rows (BucketArgs). One global atomic per edge, to
// count and again to place it, is executed at the memory (about 20 per ns for
// the whole device), and a bitonic network sorts a row of 266 in 45 rounds of
// barriers; here a workgroup counts its stretch of the list per bucket of
// consecutive rows in LDS, reserves room for the whole stretch with one atomic
// per bucket, and drops the edges there (row in the bucket and target in one
// word, weight in another, in the arrays of the graph itself); then one
// workgroup per bucket sorts it in LDS. 8M edges of 30,011 rows: counting 391
// -> 18 us, placing 721 -> 197 us (bound by its scattered words), sorting 750 -> 108 us.
// A list with a bucket beyond the sort's LDS (rows of very different lengths) is
// built the general way, so placing it would be wasted: 66M edges in lognormal
// rows, one of them of 16,000: 21.1 -> 18.2 ms, as before there were buckets, and
// 15.6 with the shifts of k_row_sort (670,000 edges: 909 -> 824 us).
constexpr int kGroupBlock = 1024;
constexpr int kGroupU = 8;  // edges a thread loads at once

__device__ __forceinline__ bool edge_ok(const GraphArgs &a, int s, int d)
{
    return s >= 0 && s < a.n && d >= 0 && d < a.n;
}

__global__ __launch_bounds__(kGroupBlock) void k_bucket_count(GraphArgs a, BucketArgs b)
{
    extern __shared__ int s_n[];  // nb
    for (int x = threadIdx.x; x < b.nb; x += kGroupBlock) s_n[x] = 0;
    __syncthreads();
    const int64_t e0 = blockIdx.x * b.stretch, e1 = min(e0 + b.stretch, b.e);
    bool bad = false;
    for (int64_t i0 = e0 + threadIdx.x; i0 < e1; i0 += kGroupBlock * kGroupU) {
        int s[kGroupU], d[kGroupU];
#pragma unroll
        for (int u = 0; u < kGroupU; ++u) {
            const int64_t i = min(i0 + u * kGroupBlock, e1 - 1);
            s[u] = b.src[i];
            d[u] = b.dst[i];
        }
#pragma unroll
        for (int u = 0; u < kGroupU; ++u) {
            if (i0 + u * kGroupBlock >= e1) break;
            if (edge_ok(a, s[u], d[u]))
                atomicAdd(&s_n[s[u] >> b.shift], 1);
            else
                bad = true;
        }
    }
    if (bad) atomicOr(a.err, kErrIndex);
    __syncthreads();
    for (int x = threadIdx.x; x < b.nb; x += kGroupBlock)
        if (s_n[x]) atomicAdd((unsigned long long *)(b.start + x + 1), (unsigned long long)s_n[x]);
}

__global__ __launch_bounds__(kGroupBlock) void k_bucket_place(GraphArgs a, BucketArgs b)
{
    // per bucket: the stretch's count, then the next free place less the
    // bucket's start
    extern __shared__ int s_n[];  // nb
    // a bucket beyond what the sort holds: the rows are built the general way
    if (*a.maxlen > kBucketCap) return;  // uniform
    for (int x = threadIdx.x; x < b.nb; x += kGroupBlock) s_n[x] = 0;
    __syncthreads();
    const int64_t e0 = blockIdx.x * b.stretch, e1 = min(e0 + b.stretch, b.e);
    for (int64_t i0 = e0 + threadIdx.x; i0 < e1; i0 += kGroupBlock * kGroupU) {
        int s[kGroupU], d[kGroupU];
#pragma unroll
        for (int u = 0; u < kGroupU; ++u) {
            const int64_t i = min(i0 + u * kGroupBlock, e1 - 1);
            s[u] = b.src[i];
            d[u] = b.dst[i];
        }
#pragma unroll
        for (int u = 0; u < kGroupU; ++u)
            if (i0 + u * kGroupBlock < e1 && edge_ok(a, s[u], d[u]))
                atomicAdd(&s_n[s[u] >> b.shift], 1);
    }
    __syncthreads();
    for (int x = threadIdx.x; x < b.nb; x += kGroupBlock)
        if (s_n[x])
            s_n[x] = (int)(atomicAdd((unsigned long long *)(b.cursor + x),
                                     (unsigned long long)s_n[x]) -
                           (unsigned long long)b.start[x]);
    __syncthreads();
    for (int64_t i0 = e0 + threadIdx.x; i0 < e1; i0 += kGroupBlock * kGroupU) {
        int s[kGroupU], d[kGroupU];
        float w[kGroupU];
        int64_t at[kGroupU];
#pragma unroll
        for (int u = 0; u < kGroupU; ++u) {
            const int64_t i = min(i0 + u * kGroupBlock, e1 - 1);
            s[u] = b.src[i];
            d[u] = b.dst[i];
            w[u] = b.w[i];
        }
#pragma unroll
        for (int u = 0; u < kGroupU; ++u) {
            const bool ok = edge_ok(a, s[u], d[u]);
            at[u] = b.start[ok ? s[u] >> b.shift : 0];
        }
#pragma unroll
        for (int u = 0; u < kGroupU; ++u) {
            if (i0 + u * kGroupBlock >= e1 || !edge_ok(a, s[u], d[u])) continue;
            const int k = s[u] >> b.shift;
            const int64_t pos = at[u] + atomicAdd(&s_n[k], 1);
            a.col[pos] = (int32_t)(((uint32_t)(s[u] - (k << b.shift)) << 24) | (uint32_t)d[u]);
            a.w[pos] = w[u];
        }
    }
}

__global__ __launch_bounds__(kBlock) void k_row_maxlen(GraphArgs a)
{
    const int k = blockIdx.x * kBlock + threadIdx.x;
    int len = 0;
    if (k < a.n) {
        const int64_t l = a.row_ptr[k + 1] - a.row_ptr[k];
        len = (int)(l > 0x7fffffff ? 0x7fffffff : l);
    }
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) len = max(len, __shfl_xor(len, off, kWave));
    if (threadIdx.x % kWave == 0 && len > 0) atomicMax(a.maxlen, len);  // one per wave
}

// Order-preserving map of fp32 bits to uint32 (negative floats reversed).
__device__ __forceinline__ uint32_t f2ord(float f)
{
    const uint32_t b = __float_as_uint(f);
    return (b & 0x80000000u) ? ~b : (b | 0x80000000u);
}
__device__ __forceinline__ float ord2f(uint32_t o)
{
    return __uint_as_float((o & 0x80000000u) ? (o & 0x7fffffffu) : ~o);
}

// Sorts each row by (target, weight) with a bitonic network in LDS. Strides are
// powers of two: comparators are found by masks, not by integer division (10M
// edges, one row in a hundred of 14,000: the build 4010 -> 3370 us).
constexpr int kSortBlock = 1024;
__global__ __launch_bounds__(kSortBlock) void k_row_sort(GraphArgs a)
{
    extern __shared__ unsigned long long keys[];
    const int k = blockIdx.x, tid = threadIdx.x;
    const int64_t rs = a.row_ptr[k];
    const int len = (int)(a.row_ptr[k + 1] - rs);
    if (len <= 1) return;
    if (len > kMaxSortRow) {
        if (tid == 0) atomicOr(a.err, kErrRowTooLong);
        return;
    }
    int p2 = 2;
    while (p2 < len) p2 <<= 1;
    for (int x = tid; x < p2; x += kSortBlock)
        keys[x] = x < len ? (((unsigned long long)(uint32_t)a.col[rs + x] << 32) |
                             f2ord(a.w[rs + x]))
                          : ~0ull;
    __syncthreads();
    for (int size = 2; size <= p2; size <<= 1) {
        for (int stride = size >> 1; stride > 0; stride >>= 1) {
            for (int x = tid; x < (p2 >> 1); x += kSortBlock) {
                const int lo = x + (x & -stride);  // 2 stride (x / stride) + x % stride
                const int hi = lo + stride;
                const bool up = (lo & size) == 0;
                const unsigned long long u = keys[lo], v = keys[hi];
                if ((u > v) == up) {
                    keys[lo] = v;
                    keys[hi] = u;
                }
            }
            __syncthreads();
        }
    }
    for (int x = tid; x < len; x += kSortBlock) {
        const unsigned long long key = keys[x];
        a.col[rs + x] = (int32_t)(key >> 32);
        a.w[rs + x] = ord2f((uint32_t)key);
    }
}

// Sorts the entries of one bucket of rows by (row, target, weight) in LDS,
// writes them back (targets alone, and the compressed ones) and its rows'
// pointers. Every row is cut into `sub` ranges of targets; an entry's place is
// its range's start (one scan over all ranges of the bucket) plus the order
// in which it arrived there, and the few entries of a range (about one: ranges
// are as many as LDS holds counters) are then put in order by one thread. A
// bucket with a range of more than kSubMax entries (targets far from evenly
// spread) is sorted row by row with a bitonic network instead.
constexpr int kSortU = kBucketCap / kSortBlock;  // entries per thread
constexpr int kSubU = kBucketSubs / kSortBlock;  // ranges per thread
constexpr int kSubMax = 48;
static_assert(kBucketCap % kSortBlock == 0 && kBucketSubs % kSortBlock == 0, "whole rounds");

__global__ __launch_bounds__(kSortBlock) void k_bucket_sort(GraphArgs a, BucketArgs b)
{
    extern __shared__ unsigned long long s_e[];  // kBucketCap entries, then the ranges' starts
    int *s_off = reinterpret_cast<int *>(s_e + kBucketCap);  // kBucketSubs + 1
    __shared__ long long sh[kSortBlock / kWave];
    __shared__ int s_max;
    const int tid = threadIdx.x, k = blockIdx.x;
    const int r0 = k << b.shift, nr = min(1 << b.shift, a.n - r0);
    const int64_t e0 = b.fanout ? (int64_t)r0 * b.fanout : b.start[k];
    const int cnt = b.fanout ? nr * b.fanout : (int)(b.start[k + 1] - e0);  // <= kBucketCap
    if (cnt > kBucketCap) {  // (the host checks it)
        if (tid == 0) atomicOr(a.err, kErrRowTooLong);
        return;
    }
    const int sub = kBucketSubs >> b.shift;  // ranges per row
    const uint32_t f = b.scale;
    for (int x = tid; x <= kBucketSubs; x += kSortBlock) s_off[x] = 0;
    if (tid == 0) s_max = 0;
    __syncthreads();
    uint32_t key[kSortU], wk[kSortU];
    int at[kSortU];  // range (bits 0-15), order of arrival (16-31)
#pragma unroll
    for (int u = 0; u < kSortU; ++u) {
        const int x = u * kSortBlock + tid;
        const int64_t e = e0 + min(x, max(cnt - 1, 0));
        key[u] = cnt > 0 ? (uint32_t)a.col[e] : 0u;
        wk[u] = cnt > 0 ? f2ord(a.w[e]) : 0u;
        if (b.fanout) key[u] |= (uint32_t)(min(x, max(cnt - 1, 0)) / b.fanout) << 24;
    }
#pragma unroll
    for (int u = 0; u < kSortU; ++u) {
        at[u] = 0;
        if (u * kSortBlock + tid >= cnt) continue;
        const int q = (int)(key[u] >> 24) * sub + (int)__umulhi(key[u] & 0xffffffu, f);
        at[u] = q | (atomicAdd(&s_off[q], 1) << 16);
    }
    __syncthreads();
    {  // counts to starts
        int n[kSubU], sum = 0, top = 0;
#pragma unroll
        for (int v = 0; v < kSubU; ++v) {
            n[v] = s_off[kSubU * tid + v];
            sum += n[v];
            top = max(top, n[v]);
        }
        int at0 = (int)block_incl_scan_i64_n<kSortBlock>(sum, sh) - sum;
#pragma unroll
        for (int v = 0; v < kSubU; ++v) {
            s_off[kSubU * tid + v] = at0;
            at0 += n[v];
        }
        if (tid == kSortBlock - 1) s_off[kBucketSubs] = at0;
        if (top > kSubMax) atomicMax(&s_max, top);
    }
    __syncthreads();
#pragma unroll
    for (int u = 0; u < kSortU; ++u)
        if (u * kSortBlock + tid < cnt)
            s_e[s_off[at[u] & 0xffff] + (at[u] >> 16)] =
                ((unsigned long long)key[u] << 32) | wk[u];
    for (int r = tid; r < nr; r += kSortBlock) a.row_ptr[r0 + r] = e0 + s_off[r * sub];
    if (tid == 0 && r0 + nr == a.n) a.row_ptr[a.n] = e0 + cnt;
    __syncthreads();
    if (s_max == 0) {  // workgroup-uniform
        for (int q = tid; q < kBucketSubs; q += kSortBlock) {
            const int lo = s_off[q], hi = s_off[q + 1];
            for (int i = lo + 1; i < hi; ++i) {
                const unsigned long long v = s_e[i];
                int j = i;
                for (; j > lo && s_e[j - 1] > v; --j) s_e[j] = s_e[j - 1];
                s_e[j] = v;
            }
        }
    } else {
        // a bitonic network per row, with every comparator ascending (the
        // first round of a merge pairs mirrored entries), so that the entries
        // beyond the row stand for the largest key and are left out
        for (int r = 0; r < nr; ++r) {
            const int lo = s_off[r * sub], len = s_off[(r + 1) * sub] - lo;
            int p2 = 1;
            while (p2 < len) p2 <<= 1;
            for (int size = 2; size <= p2; size <<= 1) {
                for (int stride = size >> 1; stride > 0; stride >>= 1) {
                    const bool mirror = stride == size >> 1;
                    for (int x = tid; x < (p2 >> 1); x += kSortBlock) {
                        const int in = x & (stride - 1), at2 = 2 * (x - in);
                        const int i = at2 + in;
                        const int j = mirror ? at2 + 2 * stride - 1 - in : i + stride;
                        if (j < len) {
                            const unsigned long long u = s_e[lo + i], v = s_e[lo + j];
                            if (u > v) {
                                s_e[lo + i] = v;
                                s_e[lo + j] = u;
                            }
                        }
                    }
                    __syncthreads();
                }
            }
        }
    }
    __syncthreads();
    for (int x = tid; x < cnt; x += kSortBlock) {
        const unsigned long long v = s_e[x];
        const int32_t d = (int32_t)((v >> 32) & 0xffffffu);
        a.col[e0 + x] = d;
        a.w[e0 + x] = ord2f((uint32_t)v);
        if (a.col16) a.col16[e0 + x] = (uint16_t)(d % a.width);
    }
}

// First index in the row [p, p+len) (sorted by target) whose target is >= v.
__device__ __forceinline__ int lower_bound_col(const int32_t *p, int len, int64_t v)
{
    int lo = 0, hi = len;
    while (lo < hi) {
        const int mid = (lo + hi) >> 1;
        if ((int64_t)p[mid] < v) lo = mid + 1;
        else hi = mid;
    }
    return lo;
}

// Pivots (Fig. 1): piv[k][s] = lower_bound(row k, s*W), s = 0..S, so that
// row entries piv[k][s] .. piv[k][s+1]-1 target slice s. One wave per row,
// lanes over slices. Also the plastic prefix end of each row.
__global__ __launch_bounds__(kBlock) void k_pivots(GraphArgs a)
{
    const int lane = threadIdx.x % kWave;
    const int64_t waves = (int64_t)gridDim.x * (kBlock / kWave);
    for (int64_t k = ((int64_t)blockIdx.x * kBlock + threadIdx.x) / kWave; k < a.n;
         k += waves) {  // wave-uniform
        const int64_t rs = a.row_ptr[k];
        const int len = (int)(a.row_ptr[k + 1] - rs);
        const int32_t *row = a.col + rs;
        int32_t *out = a.piv + k * (int64_t)(a.n_slices + 1);
        for (int s = lane; s <= a.n_slices; s += kWave)
            out[s] = s == a.n_slices ? len : lower_bound_col(row, len, (int64_t)s * a.width);
        if (lane == 0) {
            int pe = 0;
            if (a.plastic == 2) pe = len;
            else if (a.plastic == 1 && k < a.n_exc) pe = lower_bound_col(row, len, a.n_exc);
            a.pend[k] = pe;
        }
    }
}

// Compressed targets: each entry's slice-local index, target - sW for the
// slice s = target / W that holds it (16 bits for W <= 65536).
__global__ __launch_bounds__(kBlock) void k_encode_targets(GraphArgs a, int64_t n_edges)
{
    const int64_t stride = (int64_t)gridDim.x * kBlock;
    for (int64_t e = (int64_t)blockIdx.x * kBlock + threadIdx.x; e < n_edges; e += stride)
        a.col16[e] = (uint16_t)(a.col[e] % a.width);
}

}  // namespace

hipError_t launch_scan_i64(hipStream_t s, int64_t *data, int64_t count, int64_t *bsum)
{
    if (count <= 0) return hipSuccess;
    const int64_t nb = (count + kScanChunk - 1) / kScanChunk;
    hipLaunchKernelGGL(k_scan_local, dim3((unsigned)nb), dim3(kBlock), 0, s, data, count, bsum);
    hipLaunchKernelGGL(k_scan_bsum, dim3(1), dim3(kBlock), 0, s, bsum, nb);
    hipLaunchKernelGGL(k_scan_add, dim3((unsigned)nb), dim3(kBlock), 0, s, data, count, bsum);
    return hipGetLastError();
}

hipError_t launch_graph_count_bernoulli(hipStream_t s, const GraphArgs &a)
{
    hipLaunchKernelGGL(k_count_bernoulli, dim3(a.n), dim3(kBlock), 0, s, a);
    return hipGetLastError();
}

hipError_t launch_graph_fill_bernoulli(hipStream_t s, const GraphArgs &a)
{
    hipLaunchKernelGGL(k_fill_bernoulli, dim3(a.n), dim3(kBlock), 0, s, a);
    return hipGetLastError();
}

hipError_t launch_graph_fill_fanout(hipStream_t s, const GraphArgs &a)
{
    hipLaunchKernelGGL(k_rowptr_fanout, dim3(blocks_for((int64_t)a.n + 1)), dim3(kBlock), 0, s,
                       a);
    if (a.col != nullptr) {
        hipLaunchKernelGGL(k_fill_fanout, dim3(blocks_for((int64_t)a.n * a.fanout, kBlock,
                                                          1 << 16)),
                           dim3(kBlock), 0, s, a);
    }
    return hipGetLastError();
}

hipError_t launch_edges_count(hipStream_t s, const GraphArgs &a, const int32_t *src,
                              const int32_t *dst, int64_t e)
{
    if (e <= 0) return hipSuccess;
    hipLaunchKernelGGL(k_edges_count, dim3(blocks_for(e, kBlock, 1 << 16)), dim3(kBlock), 0, s,
                       a, src, dst, e);
    return hipGetLastError();
}

hipError_t launch_edges_scatter(hipStream_t s, const GraphArgs &a, const int32_t *src,
                                const int32_t *dst, const float *w, int64_t e,
                                int64_t *cursor)
{
    if (e <= 0) return hipSuccess;
    hipLaunchKernelGGL(k_edges_scatter, dim3(blocks_for(e, kBlock, 1 << 16)), dim3(kBlock), 0,
                       s, a, src, dst, w, e, cursor);
    return hipGetLastError();
}

bool choose_buckets(BucketArgs &b, int32_t n, int64_t e, int64_t max_row)
{
    // rows per bucket: about kBucketAim edges, but no fewer than kBucketFew
    // buckets where there are rows for them, and as many as LDS can count
    int shift = 0;
    while (shift < kBucketShift && ((int64_t)n >> (shift + 1)) >= kBucketFew &&
           e * (2ll << shift) / n <= kBucketAim)
        ++shift;
    while (shift < kBucketShift && (((int64_t)n - 1) >> shift) + 1 > kBucketMax) ++shift;
    b.shift = shift;
    b.nb = (int32_t)((((int64_t)n - 1) >> shift) + 1);
    const int sub = kBucketSubs >> shift;
    b.scale = (uint32_t)std::min<uint64_t>(((uint64_t)sub << 32) / (uint64_t)n, 0xFFFFFFFFull);
    b.e = e;
    const int64_t stretches =
        std::max<int64_t>(1, std::min<int64_t>(256, (e + kGroupU * kGroupBlock - 1) / (kGroupU * kGroupBlock)));
    b.stretch = (e + stretches - 1) / stretches;
    b.grid = (int32_t)stretches;
    return b.nb <= kBucketMax && max_row <= kBucketCap &&
           (double)e / n * (double)(1 << shift) <= kBucketCap;
}

hipError_t launch_bucket_count(hipStream_t s, const GraphArgs &a, const BucketArgs &b)
{
    static std::mutex mu;
    static int granted = 48 * 1024;
    const int lds = b.nb * (int)sizeof(int);
    const hipError_t e = allow_dynamic_lds((const void *)k_bucket_count, lds, mu, granted);
    if (e != hipSuccess) return e;
    if (b.e > 0)
        hipLaunchKernelGGL(k_bucket_count, dim3(b.grid), dim3(kGroupBlock), lds, s, a, b);
    return hipGetLastError();
}

hipError_t launch_bucket_place(hipStream_t s, const GraphArgs &a, const BucketArgs &b)
{
    static std::mutex mu;
    static int granted = 48 * 1024;
    const int lds = b.nb * (int)sizeof(int);
    const hipError_t e = allow_dynamic_lds((const void *)k_bucket_place, lds, mu, granted);
    if (e != hipSuccess) return e;
    if (b.e > 0)
        hipLaunchKernelGGL(k_bucket_place, dim3(b.grid), dim3(kGroupBlock), lds, s, a, b);
    return hipGetLastError();
}

hipError_t launch_bucket_sort(hipStream_t s, const GraphArgs &a, const BucketArgs &b)
{
    static std::mutex mu;
    static int granted = 48 * 1024;
    const int lds = kBucketCap * (int)sizeof(unsigned long long) + (kBucketSubs + 1) * (int)sizeof(int);
    const hipError_t e = allow_dynamic_lds((const void *)k_bucket_sort, lds, mu, granted);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(k_bucket_sort, dim3(b.nb), dim3(kSortBlock), lds, s, a, b);
    return hipGetLastError();
}

hipError_t launch_row_maxlen(hipStream_t s, const GraphArgs &a)
{
    hipLaunchKernelGGL(k_row_maxlen, dim3(blocks_for(a.n)), dim3(kBlock), 0, s, a);
    return hipGetLastError();
}

hipError_t launch_row_sort(hipStream_t s, const GraphArgs &a, int pow2len)
{
    static std::mutex mu;
    static int granted = 64 * 1024;
    const size_t lds = (size_t)pow2len * sizeof(unsigned long long);
    const hipError_t e = allow_dynamic_lds((const void *)k_row_sort, (int)lds, mu, granted);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(k_row_sort, dim3(a.n), dim3(kSortBlock), lds, s, a);
    return hipGetLastError();
}

hipError_t launch_pivots(hipStream_t s, const GraphArgs &a)
{
    hipLaunchKernelGGL(k_pivots, dim3(blocks_for((int64_t)a.n * kWave)), dim3(kBlock), 0, s,
                       a);
    return hipGetLastError();
}

hipError_t launch_encode_targets(hipStream_t s, const GraphArgs &a, int64_t n_edges)
{
    if (n_edges <= 0) return hipSuccess;
    hipLaunchKernelGGL(k_encode_targets, dim3(blocks_for(n_edges, kBlock, 1 << 16)), dim3(kBlock),
                       0, s, a, n_edges);
    return hipGetLastError();
}

}  // namespace snn
