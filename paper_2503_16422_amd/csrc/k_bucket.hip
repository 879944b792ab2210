// Depth order of the visible Gaussians by bucketing (Eq. 2 blends "sorted by
// depth"; the order is (view, float64 depth, processing position)).
//
// A frame of a few hundred thousand Gaussians is far too small for a
// multi-pass radix sort to be bound by anything but its launches (three per
// digit pass).  Here three kernels produce the same order, and with it the
// exclusive sums of the tile counts that the emission needs:
//   1. count: each visible key (float32 depth bits, a monotone image of the
//      float64 depth) falls into one of NB buckets of its view, shared out over
//      the key range by a sample of the keys (KeyMap); per-block LDS
//      counts and tile sums (one 64-bit word), one global add per non-empty bucket.  The adds
//      return the block's place in each bucket, so every entry leaves with its
//      bucket and its slot there.  The order inside a bucket depends on the scheduling
//      and is repaired by 3.
//   2. scatter: every block scans its view's NB counts itself (no separate scan
//      launch) and writes its positions to their slots.  The first block of a
//      view publishes the buckets' starts.
//   3. sort: one block per bucket sorts its positions by (float64 depth bits,
//      position) -- a strict total order, so the result is unique and no tie
//      repair is needed -- by ranking them in LDS, and sums their tile counts
//      in that order.  A bucket larger than the LDS tile (many Gaussians at one
//      depth) is sorted in LDS-sized chunks that the block then merges pairwise
//      through a second buffer (each thread places a run of the output, found
//      by a binary search of its start's co-rank).
// The bucket map is monotone in the key, so buckets in index order hold
// increasing depths and the concatenation of the sorted buckets is the
// sorted sequence.
//
// The input is either a compacted list of one view's visible entries (SrcList)
// or what the preprocess left, culled entries included (SrcViews: one view or
// several, each padded to whole chunks so that a block has one view).  Reading
// flags and depths of all processed entries costs less than the two launches of
// a compaction in front.
#include <hip/hip_runtime.h>

#include "dev_util.h"
#include "fdgs_internal.h"

namespace fdgs {
namespace {

constexpr int kNT = 256;
// Entries per thread (KPT) of a counting / scattering workgroup: 4 up to 2^18
// entries, so that a frame's ~140k still fill the chip (masked frame of 200k:
// count and scatter 24 us, 27 with 16), 16 above (whole view chunks), where what
// counts is each workgroup's own setting up and the global adds, one per
// workgroup and non-empty bucket (a view of 500k: count and scatter 35 -> 30 us;
// 16 views of 225k: 134 -> 67 us).
constexpr int64_t kSmallUpTo = int64_t(1) << 18;
static_assert(kViewChunk == 16 * kNT, "a workgroup's entries belong to one view");
// A sorting workgroup is a chain of loads (start, position, depth) and a short
// ranking: what counts is that all of them (one per bucket, 4096 for a frame) are
// resident at once, 16 on a CU: 128 threads and under 10 KB of LDS.  (256 threads
// and 1024 positions: depth order of 200k 50 us against 45, 1M 152 against 156,
// four views of 300k 136 against 104, of 800k 348 against 325.)
constexpr int kSortNT = 128, kCap = 384;

__device__ __forceinline__ int64_t count_of(const int64_t *n_dev, int64_t n_max) {
    return n_dev ? min(*n_dev, n_max) : n_max;
}

// How the nb buckets divide a view's key range [kmin, kmax].  Evenly, a dense
// slab of the scene (a wall seen from the front, a far background) or a few far
// outliers leave most buckets empty while the rest crowd, and ranking a bucket
// costs its square.  So the range is cut into even bins, and each gets buckets by
// its share of a sample of the keys (three quarters of them) and by its width (a
// quarter).  A heavy bin (an eighth of the sample or more, and four times its
// even share) is cut once more, the same way; what is not cut further divides its
// buckets evenly.  The sample is one visible entry of each wavefront of up to
// kSampleBlocks preprocess workgroups, lanes and workgroups taken by a hash: how
// the entries are ordered in memory does not matter.  Every workgroup computes the same division.
// Depth order of 200k entries, even depths: 45 us, stored by depth 35 us; 90% of
// them in a slab of 1% of the depth 53 us, of 0.01% 120 us; all equal 30 ms.
// (Dividing the mean range of the workgroups instead: 46 us, 30 ms stored by
// depth, the slabs 6 and 54 ms; dividing the whole range evenly: the slabs 5 and
// 42 ms.)
constexpr int kBins = 128, kSub = 64, kHeavy = 8;
static_assert(kSampleBlocks == 2 * kNT, "two of them a thread");
struct MapTables {
    uint32_t base[kBins + 1];             // buckets before a bin
    uint32_t heavy[kBins];                // a heavy bin's place in sub, or ~0
    uint32_t sub[kHeavy][kSub + 1];       // buckets before a part of the bin, from its first
    uint32_t n_heavy, which[kHeavy];      // the heavy bins, in any order
    uint32_t hist[kBins];
    uint32_t sub_hist[kHeavy][kSub];
};
struct KeyMap {
    uint32_t kmin, kmax, nb;
    uint32_t bins;              // at most kBins
    double scale;               // bins per key
    const MapTables *t;
    // Position of a key in units of bins, and its bin.
    __device__ __forceinline__ double at(uint32_t key, uint32_t *c) const {
        const double x = (double)(max(key, kmin) - kmin) * scale;
        *c = min((uint32_t)x, bins - 1u);
        return x;
    }
    // Monotone map of a key to [0, nb).
    __device__ __forceinline__ uint32_t bucket(uint32_t key) const {
        uint32_t c;
        double x = at(key, &c) - (double)c;
        uint32_t first = t->base[c], n = t->base[c + 1] - first;
        const uint32_t h = t->heavy[c];
        if (h != ~0u) {
            x *= (double)kSub;
            const uint32_t q = min((uint32_t)x, (uint32_t)kSub - 1u);
            x -= (double)q;
            n = t->sub[h][q + 1] - t->sub[h][q];
            first += t->sub[h][q];
        }
        return min(first + min((uint32_t)(x * (double)n), max(n, 1u) - 1u), nb - 1u);
    }
    // Lowest key of bucket b, to within two.
    __device__ __forceinline__ uint32_t edge(uint32_t b) const {
        if (b == 0u) return kmin;
        if (b >= nb) return kmax;
        uint32_t lo = 0, hi = bins - 1u;                     // the last bin with base[c] < b
        while (lo < hi) {
            const uint32_t mid = (lo + hi + 1) >> 1;
            if (t->base[mid] < b) lo = mid; else hi = mid - 1;
        }
        const uint32_t h = t->heavy[lo];
        double x = (double)lo;
        uint32_t first = t->base[lo], n = t->base[lo + 1] - first;
        if (h != ~0u) {
            b -= first;
            uint32_t l = 0, u = kSub - 1;
            while (l < u) {
                const uint32_t mid = (l + u + 1) >> 1;
                if (t->sub[h][mid] < b) l = mid; else u = mid - 1;
            }
            first = t->sub[h][l];
            n = t->sub[h][l + 1] - first;
            x += ((double)l + (double)(b - first) / (double)n) / (double)kSub;
        } else {
            x += (double)(b - first) / (double)n;
        }
        return kmin + (uint32_t)fmin(x / scale, (double)(kmax - kmin));
    }
};

// Entries [lo, hi) of the view v that chunk c holds (none: hi <= lo), and
// whether it is the view's first chunk.
struct Chunk {
    int v;
    bool first;
    int64_t lo, hi;
    uint32_t chunk, n_chunks;    // its number among the view's chunks that hold entries
};

struct SrcList {
    const uint32_t *keys32, *vals;
    const int64_t *n_dev;
    int64_t n_max;
    const uint32_t *zrange;   // [min, max] of the keys
    __device__ __forceinline__ Chunk chunk(int64_t c, int64_t size) const {
        const int64_t n = count_of(n_dev, n_max);
        return Chunk{0, c == 0, c * size, min((c + 1) * size, n), (uint32_t)c, (uint32_t)((n + size - 1) / size)};
    }
    __device__ __forceinline__ bool load(int64_t j, uint32_t *key) const {
        *key = keys32[j];
        return true;
    }
    __device__ __forceinline__ uint32_t pos(int64_t j) const { return vals[j]; }
    // The key range, the thread's eight sampled keys (~0: none) and about how many all threads have.
    __device__ __forceinline__ void range(const Chunk &, uint64_t *, uint32_t *kmin, uint32_t *kmax,
                                          uint32_t (&sample)[8], uint32_t *sampled) const {
        *sampled = 0;
        *kmin = zrange[0];
        *kmax = zrange[1];
        for (uint32_t &k : sample) k = ~0u;
    }
};

struct SrcViews {
    const uint8_t *visible;
    const uint64_t *depth_key;
    const uint32_t *block_range;   // [min, max] key of each preprocess workgroup's visible entries
    const uint32_t *samples;       // of each view, or null: the ends of the sampled workgroups' ranges
    const int64_t *n_dev;          // one view (table null): device count
    int64_t n_max;
    const ViewDesc *table;
    const uint32_t *chunk_view;
    __device__ __forceinline__ Chunk chunk(int64_t c, int64_t size) const {
        int64_t base = 0, n;
        int v = 0;
        if (table) {
            v = (int)chunk_view[c * size / kViewChunk];
            base = table[v].p_off;
            n = table[v].n_proc;
        } else {
            n = count_of(n_dev, n_max);
        }
        return Chunk{v, c * size == base, c * size, min((c + 1) * size, base + n), (uint32_t)(c - base / size),
                     (uint32_t)((n + size - 1) / size)};
    }
    __device__ __forceinline__ bool load(int64_t j, uint32_t *key) const {
        const uint64_t d = depth_key[j];
        *key = __float_as_uint((float)__longlong_as_double((long long)d));   // z > 0: bit order = value order
        return visible[j] != 0;
    }
    __device__ __forceinline__ uint32_t pos(int64_t j) const { return (uint32_t)j; }
    // From the preprocess workgroups' ranges and samples (contains a barrier).
    __device__ __forceinline__ void range(const Chunk &w, uint64_t *s_red, uint32_t *kmin, uint32_t *kmax,
                                          uint32_t (&sample)[8], uint32_t *sampled) const {
        const int64_t base = table ? table[w.v].p_off : 0;
        const int64_t n = table ? table[w.v].n_proc : count_of(n_dev, n_max);
        const int64_t b0 = base / kPreprocessBlock, b1 = (base + n + kPreprocessBlock - 1) / kPreprocessBlock;
        *sampled = 4u * (uint32_t)min(b1 - b0, (int64_t)kSampleBlocks);
#pragma unroll
        for (int q = 0; q < kSampleBlocks / kNT; ++q) {
            const uint32_t s = threadIdx.x + (uint32_t)q * kNT;
            const int64_t b = b0 + sample_block(s, (uint32_t)(b1 - b0));
            uint4 k = make_uint4(~0u, ~0u, ~0u, ~0u);
            if (b < b1) {
                if (samples) {
                    k = reinterpret_cast<const uint4 *>(samples)[(size_t)w.v * kSampleBlocks + s];
                } else if (block_range[2 * b] <= block_range[2 * b + 1]) {
                    k.x = block_range[2 * b];
                    k.y = block_range[2 * b + 1];
                }
            }
            sample[4 * q] = k.x;
            sample[4 * q + 1] = k.y;
            sample[4 * q + 2] = k.z;
            sample[4 * q + 3] = k.w;
        }
        uint32_t lo = ~0u, hi = 0u;
        for (int64_t b = b0 + threadIdx.x; b < b1; b += kNT) {
            lo = min(lo, block_range[2 * b]);                // nothing visible: [~0, 0]
            hi = max(hi, block_range[2 * b + 1]);
        }
        uint64_t both = (uint64_t)lo << 32 | (uint32_t)~hi;  // both halves want their minimum
#pragma unroll
        for (int off = 32; off > 0; off >>= 1) {
            const uint64_t o = __shfl_xor(both, off, 64);
            both = (uint64_t)min((uint32_t)(both >> 32), (uint32_t)(o >> 32)) << 32 | min((uint32_t)both, (uint32_t)o);
        }
        if (lane_id() == 0) s_red[wave_id()] = both;
        __syncthreads();
        lo = ~0u;
        hi = 0u;
#pragma unroll
        for (int q = 0; q < kNT / 64; ++q) {
            lo = min(lo, (uint32_t)(s_red[q] >> 32));
            hi = max(hi, ~(uint32_t)s_red[q]);
        }
        *kmin = lo;
        *kmax = hi;
    }
};

// The view's map, its tables in *t (s_red: scratch; contains barriers).  Of n
// buckets, before the k-th of `parts` parts that `before` of `all` samples precede:
__device__ __forceinline__ uint32_t share_of(uint32_t n, uint32_t before, uint32_t all, uint32_t k, uint32_t parts) {
    const double by_width = (double)k / (double)parts;       // parts: a power of two
    return (uint32_t)((double)n * (all ? 0.75 * ((double)before / (double)all) + 0.25 * by_width : by_width));
}
template <typename Src>
__device__ __forceinline__ KeyMap key_map(const Src &src, const Chunk &w, uint32_t nb, MapTables *t, uint64_t *s_red) {
    const uint32_t i = threadIdx.x;
    for (uint32_t k = i; k < kHeavy * kSub; k += kNT) t->sub_hist[k / kSub][k % kSub] = 0u;
    if (i < kBins) t->hist[i] = 0u;
    if (i == 0) t->n_heavy = 0u;
    KeyMap m;
    uint32_t sample[8], sampled;
    src.range(w, s_red, &m.kmin, &m.kmax, sample, &sampled);
    // sixteen samples a bin (fewer say little), eight bins at least
    m.bins = kBins;
    while (m.bins > 8u && m.bins * 16u > sampled) m.bins >>= 1;
    m.nb = nb;
    m.t = t;
    m.scale = m.kmax >= m.kmin ? (double)m.bins / ((double)(m.kmax - m.kmin) + 1.0) : 0.0;
    __syncthreads();
    uint32_t c[8];
    double x[8];
#pragma unroll
    for (int q = 0; q < 8; ++q) {
        c[q] = ~0u;
        if (sample[q] == ~0u) continue;
        x[q] = m.at(sample[q], &c[q]);
        atomicAdd(&t->hist[c[q]], 1u);
    }
    __syncthreads();
    const uint32_t mine = i < m.bins ? t->hist[i] : 0u;
    uint32_t all;
    const uint32_t before = block_exclusive_sum<kNT>(mine, reinterpret_cast<uint32_t *>(s_red), &all);
    if (i <= m.bins) t->base[i] = i == m.bins ? nb : share_of(nb, before, all, i, m.bins);
    if (i < m.bins) {
        const bool heavy = mine * min(m.bins / 4u, (uint32_t)kHeavy) >= all && all;   // at most kHeavy of them
        const uint32_t h = heavy ? atomicAdd(&t->n_heavy, 1u) : ~0u;
        t->heavy[i] = h;
        if (heavy) t->which[h] = i;
    }
    __syncthreads();
    if (t->n_heavy) {                                        // uniform
#pragma unroll
        for (int q = 0; q < 8; ++q)
            if (c[q] != ~0u && t->heavy[c[q]] != ~0u)
                atomicAdd(&t->sub_hist[t->heavy[c[q]]][min((uint32_t)((x[q] - (double)c[q]) * (double)kSub),
                                                           (uint32_t)kSub - 1u)], 1u);
        __syncthreads();
        for (uint32_t h = (uint32_t)wave_id(); h < t->n_heavy; h += kNT / 64) {
            const uint32_t b = t->which[h];
            const uint32_t n = t->base[b + 1] - t->base[b], v = t->sub_hist[h][lane_id()];
            t->sub[h][lane_id()] = share_of(n, wave_inclusive_sum(v) - v, t->hist[b], (uint32_t)lane_id(), kSub);
            if (lane_id() == 0) t->sub[h][kSub] = n;
        }
        __syncthreads();
    }
    return m;
}

constexpr int kRedWords = kNT / 64 + 1;          // 64-bit words of LDS that key_map() needs

// Monotone 32-bit image of the depth bits of a bucket's entries (its keys lie in
// [lo - 2, hi + 2]): the offset from below the lowest key, without the lowest
// bits where the bucket is too wide (a float32 step is 2^29 float64 steps;
// beyond the expected span it saturates).
struct Image {
    uint64_t base;
    int shift;
    __device__ __forceinline__ uint32_t of(uint64_t depth) const {
        const uint64_t d = depth > base ? (depth - base) >> shift : 0ull;
        return (uint32_t)min(d, (uint64_t)0xfffffffeull);
    }
};
__device__ __forceinline__ Image image_of(uint32_t lo, uint32_t hi) {
    const uint32_t from = lo - min(lo, 2u);
    const uint64_t width = (uint64_t)(max(hi, lo) - from) + 5u;
    Image im;
    const double z = (double)__uint_as_float(from);
    const uint64_t bits = (uint64_t)__double_as_longlong(z);
    im.base = bits > (1ull << 29) ? bits - (1ull << 29) : 0ull;
    im.shift = 0;
    while (((width << 29) >> im.shift) >> 32) ++im.shift;
    return im;
}

constexpr int kMaxPer = 4096 / kNT;      // buckets per thread at the largest nb
// A bucket's (block's, view's) word: entries above, their tiles in the low
// kBucketTileBits bits.
constexpr int kTileBits = kBucketTileBits;
__device__ __forceinline__ uint32_t entries_of(uint64_t w) { return (uint32_t)(w >> kTileBits); }
__device__ __forceinline__ uint64_t tiles_of(uint64_t w) { return w & ((uint64_t(1) << kTileBits) - 1); }
__device__ __forceinline__ uint64_t add64(uint64_t *p, uint64_t v) {
    return atomicAdd(reinterpret_cast<unsigned long long *>(p), (unsigned long long)v);
}

// Leaves each entry's bucket + 1 (0: not visible) in `bucket` and its place there in `slot`.
template <int KPT, typename Src>
__global__ void __launch_bounds__(kNT) bucket_count_kernel(Src src, uint32_t nb, BucketWork w, const uint32_t *tiles,
                                                           uint16_t *bucket, uint32_t *slot) {
    extern __shared__ uint64_t s_cnt[];                      // [nb]
    __shared__ uint64_t s_red[kRedWords];
    __shared__ MapTables s_map;
    const Chunk c = src.chunk(blockIdx.x, KPT * kNT);
    if (c.lo >= c.hi) return;                                // uniform
    // the entries' loads first: the range and the cleared counts come while they are on their way
    uint32_t key[KPT], nt[KPT];
    bool in[KPT];
#pragma unroll
    for (int r = 0; r < KPT; ++r) {
        const int64_t j = min(c.lo + (int64_t)r * kNT + threadIdx.x, c.hi - 1);
        in[r] = src.load(j, &key[r]) && c.lo + (int64_t)r * kNT + threadIdx.x < c.hi;
        nt[r] = tiles ? tiles[src.pos(j)] : 0u;
    }
    for (uint32_t b = threadIdx.x; b < nb; b += kNT) s_cnt[b] = 0;
    const KeyMap map = key_map(src, c, nb, &s_map, s_red);
    uint32_t bk[KPT], rank[KPT];
    uint64_t mine = 0;
#pragma unroll
    for (int r = 0; r < KPT; ++r) {
        bk[r] = rank[r] = 0;
        if (!in[r]) continue;
        bk[r] = map.bucket(key[r]);
        const uint64_t one = (uint64_t(1) << kTileBits) + nt[r];
        rank[r] = entries_of(add64(&s_cnt[bk[r]], one));
        mine += one;
    }
    __syncthreads();
    // the block's place in buckets t, t + kNT, ...: all adds on their way before the first result is used
    uint64_t *count = w.count + (size_t)c.v * nb;
    uint64_t lc[kMaxPer], lb[kMaxPer];
#pragma unroll
    for (int k = 0; k < kMaxPer; ++k) {
        const uint32_t b = threadIdx.x + (uint32_t)k * kNT;
        lc[k] = b < nb ? s_cnt[b] : 0u;
    }
#pragma unroll
    for (int k = 0; k < kMaxPer; ++k) {
        const uint32_t b = threadIdx.x + (uint32_t)k * kNT;
        lb[k] = lc[k] ? add64(&count[b], lc[k]) : 0u;
    }
#pragma unroll
    for (int k = 0; k < kMaxPer; ++k) {
        const uint32_t b = threadIdx.x + (uint32_t)k * kNT;
        if (lc[k]) s_cnt[b] = entries_of(lb[k]);
    }
    __syncthreads();
#pragma unroll
    for (int r = 0; r < KPT; ++r) {
        const int64_t j = c.lo + (int64_t)r * kNT + threadIdx.x;
        if (j >= c.hi) continue;
        bucket[j] = in[r] ? (uint16_t)(bk[r] + 1u) : (uint16_t)0;
        if (in[r]) slot[j] = (uint32_t)s_cnt[bk[r]] + rank[r];
    }
    if (w.view) {                                            // uniform: the views' totals
        uint64_t total;
        block_exclusive_sum<kNT>(mine, s_red, &total);
        if (threadIdx.x == 0 && total) add64(&w.view[c.v], total);
    }
    // the buckets' bounds, for the sort: each of the view's blocks has its part
    uint32_t *edge = w.edge + (size_t)c.v * (nb + 1u);
    const uint32_t per = nb / c.n_chunks + 1u;
    for (uint32_t k = threadIdx.x; k < per; k += kNT)
        if (c.chunk * per + k <= nb) edge[c.chunk * per + k] = map.edge(c.chunk * per + k);
}

// Every block scans its view's bucket counts into s_start (exclusive, from the
// views before); the view's first block also publishes them (start[V nb] =
// total) and the tile sums' scan for the sort.
template <int KPT, typename Src>
__global__ void __launch_bounds__(kNT) bucket_scatter_kernel(Src src, uint32_t nb, int V, BucketWork w,
                                                             const uint16_t *bucket, const uint32_t *slot,
                                                             uint32_t *out, int64_t n_out, bool tiles, int64_t *counts) {
    extern __shared__ uint32_t s_start[];                    // [nb]
    __shared__ uint32_t s_tmp[kNT / 64 + 1];
    __shared__ uint64_t s_tmp64[kNT / 64 + 1];
    const Chunk c = src.chunk(blockIdx.x, KPT * kNT);
    if (c.lo >= c.hi && !c.first) return;                    // uniform; a view's first block always publishes
    const uint64_t *count = w.count + (size_t)c.v * nb;
    // exclusive scan of the counts: thread t owns the contiguous slice [t * per, (t + 1) * per)
    const uint32_t per = nb >= (uint32_t)kNT ? nb / kNT : 1u;
    const uint32_t b0 = threadIdx.x * per;
    uint64_t cn[kMaxPer];
    uint32_t bk[KPT], sl[KPT], pos[KPT];
#pragma unroll
    for (int k = 0; k < kMaxPer; ++k) cn[k] = count[min(b0 + (uint32_t)k, nb - 1u)];
#pragma unroll
    for (int r = 0; r < KPT; ++r) {
        const int64_t j = c.lo + (int64_t)r * kNT + threadIdx.x;
        bk[r] = j < c.hi ? bucket[j] : 0u;
        sl[r] = j < c.hi ? slot[j] : 0u;
        pos[r] = j < c.hi ? src.pos(j) : 0u;
    }
    // entries and tiles of the views before
    uint64_t vis_before = 0, tiles_before = 0;
    if (c.v > 0) {                                           // uniform
        uint64_t a = 0, t = 0;
        for (int u = threadIdx.x; u < c.v; u += kNT) {
            a += entries_of(w.view[u]);
            t += tiles_of(w.view[u]);
        }
        block_exclusive_sum<kNT>(a, s_tmp64, &vis_before);
        if (c.first) block_exclusive_sum<kNT>(t, s_tmp64, &tiles_before);
    }
    uint32_t sum = 0;
#pragma unroll
    for (int k = 0; k < kMaxPer; ++k)
        if ((uint32_t)k < per && b0 + k < nb) sum += entries_of(cn[k]);
    uint32_t total;
    uint32_t run = block_exclusive_sum<kNT>(sum, s_tmp, &total) + (uint32_t)vis_before;
#pragma unroll
    for (int k = 0; k < kMaxPer; ++k)
        if ((uint32_t)k < per && b0 + k < nb) {
            s_start[b0 + k] = run;
            run += entries_of(cn[k]);
        }
    __syncthreads();
#pragma unroll
    for (int r = 0; r < KPT; ++r) {
        if (bk[r] == 0u) continue;
        const uint64_t to = (uint64_t)s_start[min(bk[r], nb) - 1u] + sl[r];
        if (to < (uint64_t)n_out) out[to] = pos[r];
    }
    if (!c.first) return;                                    // uniform
    uint32_t *start = w.start + (size_t)c.v * nb;
    for (uint32_t b = threadIdx.x; b < nb; b += kNT) start[b] = s_start[b];
    const bool last = c.v == V - 1;
    if (last && threadIdx.x == 0) start[nb] = (uint32_t)vis_before + total;
    uint64_t all = 0;
    if (tiles) {
        uint64_t *tstart = w.tstart + (size_t)c.v * nb;
        uint64_t ts = 0;
#pragma unroll
        for (int k = 0; k < kMaxPer; ++k)
            if ((uint32_t)k < per && b0 + k < nb) ts += tiles_of(cn[k]);
        uint64_t trun = block_exclusive_sum<kNT>(ts, s_tmp64, &all) + tiles_before;
#pragma unroll
        for (int k = 0; k < kMaxPer; ++k)
            if ((uint32_t)k < per && b0 + k < nb) {
                tstart[b0 + k] = trun;
                trun += tiles_of(cn[k]);
            }
    }
    if (last && counts && threadIdx.x == 0) {
        counts[0] = (int64_t)(vis_before + total);
        counts[1] = (int64_t)(tiles_before + all);
    }
}

// (depth bits, position) order; positions are distinct, so it is strict.
__device__ __forceinline__ bool before(uint64_t da, uint32_t pa, uint64_t db, uint32_t pb) {
    return da < db || (da == db && pa < pb);
}

// One block sorts m <= CAP (key, position) pairs held in LDS by rank:
// element e goes to the number of elements that precede it.  Every thread
// compares its own elements (e = t + NT r) against all m from LDS
// broadcasts; wavefronts without elements skip the loop.  The ranks come from
// 32-bit images of the keys first (Image): two vector instructions per compare
// and four keys per LDS read, where the 64-bit key with the position takes
// about six and two reads.  Two elements with one image would have one rank:
// then s_owner[rank] misses one of them, and the order by the whole (key,
// position), which is strict, decides.  s_owner receives each rank's element.
// Entries [m, m rounded up to 16) of the images and to 8 of the keys are set to
// all ones, which precede nothing.
template <int R, int NT>
__device__ __forceinline__ void ranks_by_image(const uint32_t *s_img, int m, uint32_t (&rk)[R]) {
    uint32_t ke[R];
#pragma unroll
    for (int r = 0; r < R; ++r) {
        const int e = (int)threadIdx.x + NT * r;
        ke[r] = e < m ? s_img[e] : 0u;
        rk[r] = 0;
    }
    if ((int)(threadIdx.x & ~63u) >= m) return;           // uniform over the wavefront
    for (int f0 = 0; f0 < m; f0 += 16) {
        uint32_t kf[16];
#pragma unroll
        for (int u = 0; u < 16; ++u) kf[u] = s_img[f0 + u];
#pragma unroll
        for (int u = 0; u < 16; ++u)
#pragma unroll
            for (int r = 0; r < R; ++r) rk[r] += kf[u] < ke[r] ? 1u : 0u;
    }
}
template <int R, int NT>
__device__ __forceinline__ void ranks_by_key(const uint64_t *s_key, const uint32_t *s_pos, int m, uint32_t (&rk)[R]) {
    uint64_t ke[R];
    uint32_t pe[R];
#pragma unroll
    for (int r = 0; r < R; ++r) {
        const int e = (int)threadIdx.x + NT * r;
        ke[r] = e < m ? s_key[e] : ~0ull;
        pe[r] = e < m ? s_pos[e] : ~0u;
        rk[r] = 0;
    }
    const int m8 = (m + 7) & ~7;
    for (int f0 = 0; f0 < m8; f0 += 8) {
        uint64_t kf[8];
        uint32_t pf[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) {
            kf[u] = s_key[f0 + u];
            pf[u] = s_pos[f0 + u];
        }
#pragma unroll
        for (int u = 0; u < 8; ++u)
#pragma unroll
            for (int r = 0; r < R; ++r) rk[r] += before(kf[u], pf[u], ke[r], pe[r]) ? 1u : 0u;
    }
}
template <int R, int NT>
__device__ __forceinline__ void rank_sort_r(const uint64_t *s_key, const uint32_t *s_pos, const uint32_t *s_img, int m,
                                            uint32_t *s_owner, uint32_t *s_twice) {
    uint32_t rk[R];
    auto own = [&]() {
#pragma unroll
        for (int r = 0; r < R; ++r)
            if ((int)threadIdx.x + NT * r < m) s_owner[rk[r]] = threadIdx.x + NT * r;
        __syncthreads();
    };
    ranks_by_image<R, NT>(s_img, m, rk);
    own();
#pragma unroll
    for (int r = 0; r < R; ++r) {
        const uint32_t e = threadIdx.x + NT * r;
        if ((int)e < m && s_owner[rk[r]] != e) *s_twice = 1u;
    }
    __syncthreads();
    if (*s_twice == 0u) return;                            // uniform
    ranks_by_key<R, NT>(s_key, s_pos, m, rk);
    own();
}

// s_owner[rank] = element for the m pairs (contains barriers, the first before any read).
template <int NT, int CAP>
__device__ void rank_sort(uint64_t *s_key, uint32_t *s_pos, uint32_t *s_img, int m, uint32_t *s_owner,
                          uint32_t *s_twice) {
    for (int i = m + (int)threadIdx.x; i < ((m + 15) & ~15); i += NT) s_img[i] = ~0u;
    for (int i = m + (int)threadIdx.x; i < ((m + 7) & ~7); i += NT) {
        s_key[i] = ~0ull;
        s_pos[i] = ~0u;
    }
    if (threadIdx.x == 0) *s_twice = 0u;
    __syncthreads();
    if (m <= NT) rank_sort_r<1, NT>(s_key, s_pos, s_img, m, s_owner, s_twice);
    else if (m <= 2 * NT) rank_sort_r<2, NT>(s_key, s_pos, s_img, m, s_owner, s_twice);
    else rank_sort_r<CAP / NT, NT>(s_key, s_pos, s_img, m, s_owner, s_twice);
}

// Block b sorts bucket b; with tiles, offsets[j] = the tiles of the entries
// before the j-th of the order (from the bucket's tstart).
template <int NT, int CAP>
__global__ void __launch_bounds__(NT) bucket_sort_kernel(const uint32_t *start, const uint32_t *edge, uint32_t nb,
                                                              const uint32_t *bucketed, const uint64_t *depth_key,
                                                              int64_t n_max, uint32_t *alt, uint32_t *out,
                                                              const uint32_t *tiles, const uint64_t *tstart,
                                                              uint64_t *offsets) {
    __shared__ uint64_t s_key[CAP + 8];
    __shared__ __attribute__((aligned(16))) uint32_t s_img[CAP];
    __shared__ uint32_t s_pos[CAP + 8], s_tiles[CAP], s_owner[CAP];
    __shared__ uint32_t s_twice;
    __shared__ uint32_t s_wave[NT / 64];
    __shared__ uint64_t s_tmp[NT / 64 + 1];
    const uint32_t lo = start[blockIdx.x], hi = (uint32_t)min((int64_t)start[blockIdx.x + 1], n_max);
    const uint32_t *e = edge + blockIdx.x + blockIdx.x / nb;   // nb + 1 per view
    const uint32_t key_lo = e[0], key_hi = e[1];
    const uint64_t tiles_before = tiles ? tstart[blockIdx.x] : 0;
    const int64_t m = (int64_t)hi - lo;
    if (m <= 0) return;
    const Image im = image_of(key_lo, key_hi);
    const uint32_t last = (uint32_t)(n_max - 1);    // positions index depth_key[0, n_max)
    // sorted runs of CAP (all of the bucket when it fits)
    for (int64_t c0 = 0; c0 < m; c0 += CAP) {
        const int len = (int)min((int64_t)CAP, m - c0);
        for (int i = threadIdx.x; i < len; i += NT) {
            const uint32_t pos = min(bucketed[lo + c0 + i], last);
            const uint64_t key = depth_key[pos];
            s_pos[i] = pos;
            s_key[i] = key;
            s_img[i] = im.of(key);
            if (tiles) s_tiles[i] = tiles[pos];
        }
        rank_sort<NT, CAP>(s_key, s_pos, s_img, len, s_owner, &s_twice);
        for (int j = threadIdx.x; j < len; j += NT) out[lo + c0 + j] = s_pos[s_owner[j]];
        if (m <= CAP) break;
        __syncthreads();
    }
    if (m <= CAP) {
        if (!tiles) return;
        // exclusive sums of the tile counts in the new order: each thread's
        // consecutive elements, the wavefront, the wavefronts before (at most
        // CAP counts of 2^22 tiles: 32 bits hold the sums)
        const int per = ((int)m + NT - 1) / NT, j0 = (int)threadIdx.x * per;
        uint32_t t[CAP / NT], sum = 0;
#pragma unroll
        for (int q = 0; q < CAP / NT; ++q) {
            t[q] = q < per && j0 + q < (int)m ? s_tiles[s_owner[j0 + q]] : 0u;
            sum += t[q];
        }
        const uint32_t inc = wave_inclusive_sum(sum);
        if (lane_id() == 63) s_wave[wave_id()] = inc;
        __syncthreads();
        uint64_t run = tiles_before + (inc - sum);
        for (int w = 0; w < wave_id(); ++w) run += s_wave[w];
#pragma unroll
        for (int q = 0; q < CAP / NT; ++q)
            if (q < per && j0 + q < (int)m) {
                offsets[lo + j0 + q] = run;
                run += t[q];
            }
        return;
    }
    // pairwise merges of runs of width w: a thread places kRun consecutive
    // elements of a pair's output (a pair has a multiple of kRun places): how many
    // of the elements before them come from the first run by a binary search,
    // then one comparison each.  (An element per search took 10 to 20 dependent
    // loads each: 200k equal depths 59 ms, 30 ms now.)
    constexpr int kRun = 16;
    static_assert(CAP % kRun == 0, "a thread's run lies in one pair");
    uint32_t *src = out + lo, *dst = alt + lo;
    for (int64_t w = CAP; w < m; w <<= 1) {
        for (int64_t i0 = (int64_t)threadIdx.x * kRun; i0 < m; i0 += (int64_t)NT * kRun) {
            const int64_t a0 = i0 / (2 * w) * (2 * w), i = i0 - a0;
            const int64_t la = min(w, m - a0);
            const int64_t lb = max((int64_t)0, min(w, m - a0 - w));
            const uint32_t *A = src + a0, *B = src + a0 + la;
            int64_t s = max((int64_t)0, i - lb), e = min(i, la);
            while (s < e) {
                const int64_t mid = (s + e) >> 1;
                const uint32_t pa = A[mid], pb = B[i - 1 - mid];
                if (before(depth_key[pa], pa, depth_key[pb], pb)) s = mid + 1; else e = mid;
            }
            int64_t ia = s, ib = i - s;
            uint32_t pa = ia < la ? A[ia] : 0u, pb = ib < lb ? B[ib] : 0u;
            uint64_t ka = ia < la ? depth_key[pa] : 0ull, kb = ib < lb ? depth_key[pb] : 0ull;
            const int64_t end = min(i + kRun, la + lb);
            for (int64_t j = i; j < end; ++j) {
                if (ib >= lb || (ia < la && before(ka, pa, kb, pb))) {
                    dst[a0 + j] = pa;
                    if (++ia < la) {
                        pa = A[ia];
                        ka = depth_key[pa];
                    }
                } else {
                    dst[a0 + j] = pb;
                    if (++ib < lb) {
                        pb = B[ib];
                        kb = depth_key[pb];
                    }
                }
            }
        }
        __syncthreads();
        uint32_t *t = src; src = dst; dst = t;
    }
    if (src != out + lo)
        for (int64_t i = threadIdx.x; i < m; i += NT) out[lo + i] = src[i];
    if (!tiles) return;
    uint64_t run = tiles_before;
    for (int64_t j0 = 0; j0 < m; j0 += NT) {
        const int64_t j = j0 + threadIdx.x;
        uint64_t total;
        const uint64_t ex =
            block_exclusive_sum<NT>(j < m ? (uint64_t)tiles[min(src[j], last)] : uint64_t(0), s_tmp, &total);
        if (j < m) offsets[lo + j] = run + ex;
        run += total;
    }
}

}  // namespace

// About 64 positions per bucket, between 64 and 4096 buckets.
int bucket_log2_for(int64_t n_max) {
    int l = 6;
    while (l < 12 && (int64_t(1) << l) * 64 < n_max) ++l;
    return l;
}

size_t bucket_scratch_words(int64_t n_max) {
    const int64_t nb = int64_t(1) << bucket_log2_for(n_max);
    return (size_t)(3 * nb + 1 + 2 + nb + 1);
}

BucketWork bucket_work(uint32_t *words, int64_t n_view_max, int32_t V, size_t *n_words, size_t *n_clear) {
    const size_t nb = (size_t(1) << bucket_log2_for(n_view_max)) * (size_t)V;
    BucketWork w;
    size_t at = 0;
    auto take = [&](size_t n) {   // whole 64-bit words
        uint32_t *p = words + at;
        at += (n + 1) / 2 * 2;
        return p;
    };
    w.count = reinterpret_cast<uint64_t *>(take(2 * nb));
    w.view = reinterpret_cast<uint64_t *>(take(2 * (size_t)V));
    *n_clear = at;
    w.tstart = reinterpret_cast<uint64_t *>(take(2 * nb));
    w.start = take(nb + 1);
    w.edge = take(nb + (size_t)V);
    *n_words = at;
    return w;
}

namespace {

template <int KPT, typename Src>
hipError_t order_buckets(const Src &src, int64_t n_view_max, int32_t V, const BucketWork &w,
                         const uint64_t *depth_key, int64_t n_max, uint32_t *alt, uint32_t *bucketed, uint32_t *out,
                         const uint32_t *tiles, uint64_t *offsets, int64_t *counts, hipStream_t s) {
    // until the sort writes them, `out` holds the entries' buckets and `alt` their slots
    const uint32_t nb = 1u << bucket_log2_for(n_view_max);
    const int64_t chunks = (n_max + KPT * kNT - 1) / (KPT * kNT);
    hipLaunchKernelGGL((bucket_count_kernel<KPT, Src>), dim3((unsigned)chunks), dim3(kNT),
                       sizeof(uint64_t) * nb, s, src, nb, w, tiles, reinterpret_cast<uint16_t *>(out), alt);
    hipLaunchKernelGGL((bucket_scatter_kernel<KPT, Src>), dim3((unsigned)chunks), dim3(kNT), sizeof(uint32_t) * nb, s, src, nb,
                       (int)V, w, reinterpret_cast<const uint16_t *>(out), (const uint32_t *)alt, bucketed, n_max,
                       tiles != nullptr, counts);
    hipLaunchKernelGGL((bucket_sort_kernel<kSortNT, kCap>), dim3(nb * (unsigned)V), dim3(kSortNT), 0, s, (const uint32_t *)w.start,
                       (const uint32_t *)w.edge, nb, (const uint32_t *)bucketed, depth_key, n_max, alt, out, tiles,
                       (const uint64_t *)w.tstart, offsets);
    return hipGetLastError();
}

}  // namespace

hipError_t depth_order_buckets(const uint32_t *keys32, const uint32_t *vals, const int64_t *n_vis_dev, int64_t n_max,
                               const uint64_t *depth_key, uint32_t *work, uint32_t *alt, uint32_t *bucketed,
                               uint32_t *out, hipStream_t s) {
    if (n_max == 0) return hipSuccess;
    const uint32_t nb = 1u << bucket_log2_for(n_max);
    BucketWork w{};
    w.count = reinterpret_cast<uint64_t *>(work);
    w.start = work + 2 * nb;
    w.edge = work + 3 * nb + 3;
    return order_buckets<4>(SrcList{keys32, vals, n_vis_dev, n_max, work + 3 * nb + 1}, n_max, 1, w,
                         depth_key, n_max, alt, bucketed, out, nullptr, nullptr, nullptr, s);
}

hipError_t depth_order_views(const uint8_t *visible, const uint64_t *depth_key, const uint32_t *tiles,
                             const uint32_t *block_range, const int64_t *n_dev, int64_t n_total, const ViewDesc *table,
                             const uint32_t *chunk_view, int32_t V, int64_t n_view_max, uint32_t *work, uint32_t *alt,
                             uint32_t *bucketed, uint32_t *out, uint64_t *offsets, int64_t *counts, hipStream_t s,
                             const uint32_t *samples) {
    size_t words = 0, clear = 0;
    const BucketWork w = bucket_work(work, n_view_max, V, &words, &clear);
    const SrcViews src{visible, depth_key, block_range, samples, n_dev, n_total, table, chunk_view};
    return n_total <= kSmallUpTo ? order_buckets<4>(src, n_view_max, V, w, depth_key, n_total, alt, bucketed, out, tiles,
                                                    offsets, counts, s)
                                 : order_buckets<16>(src, n_view_max, V, w, depth_key, n_total, alt, bucketed, out, tiles,
                                                     offsets, counts, s);
}

}  // namespace fdgs
