// Vector quantisation of the SH coefficients (the post-processing of Sec. 5:
// each Gaussian's 16 x 3 SH coefficients are replaced by a codebook entry).
// Lloyd's k-means over the 48-vectors (basis-major, then channel):
//   assign: a(i) = argmin_j ||x_i - c_j||^2, equal distances to the lower j;
//   update: c_j = mean of the x_i with a(i) = j; an empty cluster keeps c_j.
//
// The distance that decides is float32: t_d = x_d - c_d, acc = fma(t_d, t_d,
// acc) in component order (dist_exact).  Evaluating it for every (Gaussian,
// entry) pair is bound by the vector ALU (96 operations a pair: 2.57 ms for
// 200k x 4096).  It is a contraction but for |x|^2 and |c|^2, so the matrix
// cores screen it (vq_screen_kernel) with a bound on how far the screened
// score can lie from the exact distance, and only the Gaussians whose best
// entry the bound leaves open (about 2% there) are given to the exact kernel.
// The result is the exact kernel's for every input.  Screening 233 us (1.0
// PFLOP/s of bfloat16 products; a large product of the library reaches 1.2 on
// this card) and exact 63 us, for 2570 us before.
//
// The update sorts (cluster, index) pairs with the stable radix sort, so each
// cluster's members are contiguous and in index order, and sums them in
// float64 in that order: deterministic, and the float32 mean is within one
// rounding of the exact one.
#include <hip/hip_runtime.h>
#include <math.h>

#include <algorithm>

#include "dev_util.h"
#include "fdgs_internal.h"

namespace fdgs {
namespace {

constexpr int kD = 48;        // coefficients per vector
constexpr int kNT = 256;

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));

// Screening in bfloat16 pairs: x = x_hi + x_lo + r with |x_lo| <= 2^-8 |x| and
// |r| <= 2^-16 |x|, and three matrix products lo hi + hi lo + hi hi.  With
// Q = |x|^2 + |c|^2 (so S = sum |x_d c_d| <= Q / 2) the score
// D = x.c - |c|^2 / 2 is off by at most
//   3.03 2^-16 S      what the split and the missing lo lo product leave
// + 49 2^-23 S        the 48 additions of hi hi to sums of at most 1.01 S, an ulp
//                     each, and the 96 before them to sums below 2^-6 S
// + 2^-23 Q           adding -|c|^2 / 2, and its rounding
// + 2^-19 Q           the four low bits that give way to the row
//   <= 2.82e-5 Q,
// and the exact float32 distance by at most 50 2^-24 d^2 <= 0.6e-5 Q.  In
// distance units |(|x|^2 - 2 D) - acc| <= 6.3e-5 Q, taken as kKappa Q.
constexpr float kKappa = 6.4e-5f;
constexpr float kHalfKappa = 0.5f * kKappa;
// Flushed denormals: an absolute error far below this.
constexpr float kTiny = 0x1p-100f;
// Entries of this squared norm and above, or without a finite one, are left out of the
// screening (no product of the rest with a vector below kSure overflows).
constexpr float kHuge = 0x1p100f;
// The screening decides only for vectors and nearest entries of squared norms below
// this: an entry left out is then more than (2^50 - 2^45)^2 away, the nearest at most (2^46)^2.
constexpr float kSure = 0x1p90f;

constexpr int kEnt = 32;                       // entries per matrix tile (rows)
constexpr int kSteps = kD / 16;                // products of depth 16 per tile
constexpr int kFragVecs = kSteps * 2 * 64;     // 16-byte vectors per entry tile: step, hi / lo, lane
constexpr int kScreenWaves = 4;
constexpr int kColTiles = 2;                   // 32-Gaussian tiles per wavefront
constexpr int kScreenRows = kScreenWaves * kColTiles * 32;   // Gaussians per workgroup
constexpr int kStage = 2;                      // entry tiles per LDS stage
constexpr int kScreenPerCu = 3;                // workgroups a CU holds (168 registers)
constexpr int kScreenGroups = 256 * kScreenPerCu;
constexpr float kLowest = -3e38f;              // below every score, and finite with any low bits
constexpr float kFloor = -0x1p110f;            // scores of entries that take part lie above it

// code[j][d] = sh plane d at Gaussian init[j] (indices clamped into the model)
__global__ void __launch_bounds__(kNT) vq_gather_kernel(const float *sh, int64_t n, const uint32_t *init,
                                                        int64_t k, float *code) {
    const int64_t i = (int64_t)blockIdx.x * kNT + threadIdx.x;
    if (i >= k * kD) return;
    const int64_t j = i / kD;
    const int d = (int)(i % kD);
    const int64_t g = min((int64_t)init[j], n - 1);
    code[i] = sh[(int64_t)d * n + g];
}

// rows[i][d] = sh plane d at Gaussian i, through LDS (a workgroup per 64
// Gaussians): the update and the exact kernel read whole vectors of scattered
// Gaussians, 192 contiguous bytes here against 48 cache lines in the planes.
constexpr int kRowTile = 64;
__global__ void __launch_bounds__(kNT) vq_rows_kernel(const float *sh, int64_t n, float *rows) {
    __shared__ float s[kD][kRowTile + 1];
    const int64_t i0 = (int64_t)blockIdx.x * kRowTile;
    const int cnt = (int)min((int64_t)kRowTile, n - i0);
    for (int e = threadIdx.x; e < kD * kRowTile; e += kNT) {
        const int d = e / kRowTile, c = e % kRowTile;
        if (c < cnt) s[d][c] = sh[(int64_t)d * n + i0 + c];
    }
    __syncthreads();
    for (int e = threadIdx.x; e < cnt * kD; e += kNT) rows[i0 * kD + e] = s[e % kD][e / kD];
}

// Component d of Gaussian i: from the rows, or from the planes of a model too
// large for a copy.
template <bool ROWS>
__device__ __forceinline__ float component(const float *x, int64_t n, int64_t i, int d) {
    return ROWS ? x[i * kD + d] : x[(int64_t)d * n + i];
}

__device__ __forceinline__ void split_bf16(const float (&v)[8], bf16x8 *hi, bf16x8 *lo) {
#pragma unroll
    for (int q = 0; q < 8; ++q) {
        const __bf16 h = (__bf16)v[q];
        (*hi)[q] = h;
        (*lo)[q] = (__bf16)(v[q] - (float)h);
    }
}

// One wavefront per tile of 32 entries: their fragments in the order the
// matrix instruction takes them (lane l: entry l % 32, components
// 16 s + 8 (l / 32) + 0..7), their squared norms, and what is added to a row's
// products, -(1/2 - kappa/2) |c|^2 (kLowest for the rows past k).  An entry whose
// squared norm is kHuge or more, infinite or NaN counts as such a row (zeros and
// kLowest): a score of its own could be infinite or NaN and would displace the
// running best.  Block 0 clears the counter of open Gaussians.
__global__ void __launch_bounds__(64) vq_frag_kernel(const float *code, int64_t k, bf16x8 *frag, float *start,
                                                     float *norm2, uint32_t *n_open) {
    const int lane = threadIdx.x;
    if (blockIdx.x == 0 && lane == 0) *n_open = 0u;
    const int64_t j = (int64_t)blockIdx.x * kEnt + lane % 32;
    double sum = 0.0;
    float v[kSteps][8];
#pragma unroll
    for (int s = 0; s < kSteps; ++s)
#pragma unroll
        for (int q = 0; q < 8; ++q) {
            v[s][q] = j < k ? code[j * kD + 16 * s + 8 * (lane / 32) + q] : 0.0f;
            sum += (double)v[s][q] * (double)v[s][q];
        }
    sum += __shfl_xor(sum, 32, 64);
    const float n2 = (float)sum;
    const bool in = j < k && n2 < kHuge;
#pragma unroll
    for (int s = 0; s < kSteps; ++s) {
        if (!in)
#pragma unroll
            for (int q = 0; q < 8; ++q) v[s][q] = 0.0f;
        bf16x8 hi, lo;
        split_bf16(v[s], &hi, &lo);
        bf16x8 *dst = frag + ((int64_t)blockIdx.x * kSteps + s) * 2 * 64;
        dst[lane] = hi;
        dst[64 + lane] = lo;
    }
    if (lane < 32) {
        norm2[j] = n2;                                  // padded to whole tiles
        start[j] = in ? -(0.5f - kHalfKappa) * n2 : kLowest;
    }
}

// Top two of two disjoint sets' (largest, second, position of the largest).
__device__ __forceinline__ void merge_top(float &m1, float &m2, uint32_t &j, float o1, float o2, uint32_t oj) {
    m2 = fmaxf(fmaxf(m2, o2), fminf(m1, o1));
    if (o1 > m1) {
        m1 = o1;
        j = oj;
    }
}

// Largest of two non-NaN floats without the operand canonicalisation fmaxf needs.
__device__ __forceinline__ float max_plain(float a, float b) {
    float r;
    asm("v_max_f32 %0, %1, %2" : "=v"(r) : "v"(a), "v"(b));
    return r;
}

// The sweep is (blocks of 256 Gaussians) x (tiles of 32 entries), cut into one
// contiguous piece of `per` tiles per workgroup, whatever block a tile belongs
// to: every workgroup is resident and gets the same work.  (A workgroup per
// block of Gaussians leaves a second, almost empty round behind: 782
// workgroups on 768 places took 278 us, 768 equal pieces 233 us at 200k x 4096.)  A
// workgroup writes the result of its part of each block it meets to that
// block's place number (workgroup - first workgroup of the block).
struct Sweep {
    int64_t n_blocks;     // blocks of kScreenRows Gaussians
    int32_t n_tiles;      // entry tiles
    int64_t per;          // tiles per workgroup, a multiple of kStage
    __host__ __device__ int64_t total() const { return n_blocks * n_tiles; }
    __host__ __device__ int64_t first_of(int64_t block) const { return block * n_tiles / per; }
    __host__ __device__ int64_t last_of(int64_t block) const { return ((block + 1) * n_tiles - 1) / per; }
};

// Screening: for each Gaussian the largest and second largest of
// a_j = D_j + kappa/2 |c_j|^2 over a workgroup's entries, and the largest's
// entry.  Entries are the rows of the 32x32 result, Gaussians its columns, so
// a lane keeps its column's best in registers; 64 Gaussians per wavefront hold
// their split vectors in registers for the whole sweep, and the four
// wavefronts of a workgroup share the entry tiles through LDS (two tiles a
// stage, the next stage on its way while one is used).  The four low bits of a
// score give way to its result register (the row), so a score costs four
// vector instructions; per 64 x 32 pairs they run beside 18 matrix
// instructions of 8 passes.
__global__ void __launch_bounds__(kScreenWaves * 64, kScreenPerCu) vq_screen_kernel(
    const float *sh, int64_t n, const u32x4 *frag, const float *start, Sweep sw, float *out1, float *out2,
    uint32_t *outj, float *out_norm2) {
    constexpr int kNThr = kScreenWaves * 64;
    constexpr int kVecs = kStage * kFragVecs;              // 16-byte vectors per stage
    constexpr int kPer = kVecs / kNThr;                    // per thread
    static_assert(kVecs % kNThr == 0, "whole loads per thread");
    __shared__ u32x4 s_frag[2][kVecs];
    __shared__ float s_start[2][kStage * kEnt];
    const int lane = lane_id(), half = lane / 32, t = threadIdx.x;
    const int n_tiles = sw.n_tiles;
    const int64_t vec_end = (int64_t)n_tiles * kFragVecs - 1;
    const int start_end = n_tiles * kEnt - 1;
    u32x4 rf[kPer];
    float rs = 0.0f;
    // a stage's tiles, which follow each other; past the last one the loads repeat its end, which is not used
    auto fetch = [&](int tile) {
#pragma unroll
        for (int p = 0; p < kPer; ++p) rf[p] = frag[min((int64_t)tile * kFragVecs + p * kNThr + t, vec_end)];
        if (t < kStage * kEnt) rs = start[min(tile * kEnt + t, start_end)];
    };
    auto put = [&](int b) {
#pragma unroll
        for (int p = 0; p < kPer; ++p) s_frag[b][p * kNThr + t] = rf[p];
        if (t < kStage * kEnt) s_start[b][t] = rs;
    };
    const int64_t w0 = (int64_t)blockIdx.x * sw.per, w1 = min(w0 + sw.per, sw.total());
    int b = 0;
    for (int64_t w = w0; w < w1;) {                        // each block of Gaussians the piece meets
        const int64_t block = w / n_tiles;
        const int t0 = (int)(w - block * n_tiles), t1 = (int)min((int64_t)n_tiles, t0 + (w1 - w));
        w += t1 - t0;
        fetch(t0);
        const int64_t row0 = block * kScreenRows + wave_id() * (kColTiles * 32) + lane % 32;
        bf16x8 xh[kColTiles][kSteps], xl[kColTiles][kSteps];
        float norm2[kColTiles];
#pragma unroll
        for (int c = 0; c < kColTiles; ++c) {
            const int64_t i = min(row0 + 32 * c, n - 1);
            float sum = 0.0f;
#pragma unroll
            for (int s = 0; s < kSteps; ++s) {
                float v[8];
#pragma unroll
                for (int q = 0; q < 8; ++q) v[q] = sh[(int64_t)(16 * s + 8 * half + q) * n + i];
#pragma unroll
                for (int q = 0; q < 8; ++q) sum = fmaf(v[q], v[q], sum);
                split_bf16(v, &xh[c][s], &xl[c][s]);
            }
            norm2[c] = sum + __shfl_xor(sum, 32, 64);
        }
        float m1[kColTiles], m2[kColTiles];
        int mt[kColTiles];                                 // tile of the largest
#pragma unroll
        for (int c = 0; c < kColTiles; ++c) {
            m1[c] = m2[c] = kLowest;
            mt[c] = 0;
        }
        put(b);
        __syncthreads();
        for (int tile = t0; tile < t1; tile += kStage, b ^= 1) {
            const bool more = tile + kStage < t1;
            if (more) fetch(tile + kStage);
#pragma unroll
            for (int u = 0; u < kStage; ++u) {
                if (tile + u >= t1) break;                 // uniform
                const bf16x8 *f = reinterpret_cast<const bf16x8 *>(s_frag[b] + u * kFragVecs) + lane;
                bf16x8 ah[kSteps], al[kSteps];
#pragma unroll
                for (int s = 0; s < kSteps; ++s) {
                    ah[s] = f[s * 128];
                    al[s] = f[s * 128 + 64];
                }
                // the small products first, while the sums are small; then hi hi
                f32x16 acc[kColTiles];
#pragma unroll
                for (int c = 0; c < kColTiles; ++c) acc[c] = f32x16{};
#pragma unroll
                for (int s = 0; s < kSteps; ++s) {
#pragma unroll
                    for (int c = 0; c < kColTiles; ++c)
                        acc[c] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(al[s], xh[c][s], acc[c], 0, 0, 0);
#pragma unroll
                    for (int c = 0; c < kColTiles; ++c)
                        acc[c] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(ah[s], xl[c][s], acc[c], 0, 0, 0);
                }
#pragma unroll
                for (int s = 0; s < kSteps; ++s)
#pragma unroll
                    for (int c = 0; c < kColTiles; ++c)
                        acc[c] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(ah[s], xh[c][s], acc[c], 0, 0, 0);
                float from[16];                            // result register r: row 8 (r / 4) + 4 half + r % 4
#pragma unroll
                for (int g = 0; g < 4; ++g) {
                    const float4 v = *reinterpret_cast<const float4 *>(s_start[b] + u * kEnt + 8 * g + 4 * half);
                    from[4 * g] = v.x;
                    from[4 * g + 1] = v.y;
                    from[4 * g + 2] = v.z;
                    from[4 * g + 3] = v.w;
                }
#pragma unroll
                for (int c = 0; c < kColTiles; ++c) {
                    const float was = m1[c];
#pragma unroll
                    for (int r = 0; r < 16; ++r) {
                        const float v = __uint_as_float((__float_as_uint(acc[c][r] + from[r]) & ~15u) | (uint32_t)r);
                        m2[c] = __builtin_amdgcn_fmed3f(v, m1[c], m2[c]);   // m2 <= m1: the second largest of the three
                        m1[c] = max_plain(v, m1[c]);
                    }
                    mt[c] = m1[c] != was ? tile + u : mt[c];
                }
            }
            if (more) put(b ^ 1);
            __syncthreads();
        }
        const int64_t place = (int64_t)blockIdx.x - sw.first_of(block);
#pragma unroll
        for (int c = 0; c < kColTiles; ++c) {
            const uint32_t r = __float_as_uint(m1[c]) & 15u;
            uint32_t j = (uint32_t)mt[c] * kEnt + 8u * (r >> 2) + 4u * (uint32_t)half + (r & 3u);
            const float o1 = __shfl_xor(m1[c], 32, 64), o2 = __shfl_xor(m2[c], 32, 64);
            const uint32_t oj = __shfl_xor(j, 32, 64);
            merge_top(m1[c], m2[c], j, o1, o2, oj);
            const int64_t i = row0 + 32 * c;
            if (half == 0 && i < n) {
                const int64_t o = place * n + i;
                out1[o] = m1[c];
                out2[o] = m2[c];
                outj[o] = j;
                if (place == 0) out_norm2[i] = norm2[c];
            }
        }
    }
}

// Per Gaussian, over its block's places: the entry j* of the largest a is the nearest
// one for certain when a_j* - a_j > kappa (|x|^2 + |c_j*|^2) for the second
// largest a_j (then |x|^2 - 2 D_j - kappa/2 ... exceeds j*'s bound for every
// other entry).  Otherwise -- also for any NaN, for norms so large that a product
// could have overflowed, and where no entry took part (the largest a is then a
// padding row's, below kFloor) -- the Gaussian joins the open list; its
// assignment holds the top bit and its place there, and its best starts as
// (inf, entry 0), what the exact search returns when no distance is finite.
constexpr uint32_t kOpen = 0x80000000u;

__global__ void __launch_bounds__(kNT) vq_resolve_kernel(const float *in1, const float *in2, const uint32_t *inj,
                                                         const float *x_norm2, const float *c_norm2, int64_t n,
                                                         Sweep sw, uint32_t *assign, uint32_t *open_list,
                                                         unsigned long long *best, uint32_t *n_open) {
    static_assert(kNT == kScreenRows, "a workgroup per block of Gaussians");
    __shared__ uint32_t s_tmp[kNT / 64 + 1];
    __shared__ uint32_t s_at;
    const int64_t i = (int64_t)blockIdx.x * kNT + threadIdx.x;
    bool open = false;
    if (i < n) {
        float m1 = in1[i], m2 = in2[i];
        uint32_t j = inj[i];
        const int places = (int)(sw.last_of(blockIdx.x) - sw.first_of(blockIdx.x)) + 1;
        for (int s = 1; s < places; ++s) {
            const int64_t o = (int64_t)s * n + i;
            merge_top(m1, m2, j, in1[o], in2[o], inj[o]);
        }
        const float xn = x_norm2[i], cn = c_norm2[j];
        const bool sure = m1 - m2 > kKappa * (xn + cn) * 1.001f + kTiny && m1 > kFloor && xn < kSure && cn < kSure;
        open = !sure;
        if (sure) assign[i] = j;
    }
    uint32_t total;
    const uint32_t rank = block_exclusive_sum<kNT>(open ? 1u : 0u, s_tmp, &total);
    if (threadIdx.x == 0 && total) s_at = atomicAdd(n_open, total);
    __syncthreads();
    if (open) {
        const uint32_t slot = s_at + rank;
        open_list[slot] = (uint32_t)i;
        best[slot] = (unsigned long long)__float_as_uint(INFINITY) << 32;
        assign[i] = kOpen | slot;
    }
}

// The exact search of the open Gaussians: a lane per Gaussian and a split of
// the entries per workgroup (one wavefront; the entry is the same for every
// lane, so its components come through the scalar cache), 96 operations per
// pair.  (distance bits, entry) packed in 64 bits order as distance, then
// entry; a NaN or an infinity never beats the start value.  Without a list every
// Gaussian is open, at the place of its number.
constexpr int kExactEntries = 64;    // entries per workgroup
constexpr int kExactGroups = 128;    // workgroups along the list (each strides over it)
constexpr int kLeanGroups = 4096;    // the same without a list
template <bool ROWS>
__global__ void __launch_bounds__(64) vq_exact_kernel(const float *__restrict__ x, int64_t n,
                                                      const float *__restrict__ code, int64_t k,
                                                      const uint32_t *__restrict__ open_list,
                                                      const uint32_t *__restrict__ n_open, unsigned long long *best) {
    const int64_t cnt = open_list ? (int64_t)*n_open : n;
    const int64_t j0 = (int64_t)blockIdx.x * kExactEntries, j1 = min(j0 + kExactEntries, k);
    for (int64_t g = blockIdx.y; g * 64 < cnt; g += gridDim.y) {
        const int64_t slot = g * 64 + threadIdx.x;
        const int64_t i = open_list ? (int64_t)open_list[min(slot, cnt - 1)] : min(slot, n - 1);
        float v[kD];
#pragma unroll
        for (int d = 0; d < kD; ++d) v[d] = component<ROWS>(x, n, i, d);
        float low = INFINITY;
        uint32_t lj = 0;
        for (int64_t j = j0; j < j1; ++j) {
            const float *c = code + j * kD;
            float acc = 0.0f;
#pragma unroll
            for (int d = 0; d < kD; ++d) {
                const float dif = v[d] - c[d];
                acc = fmaf(dif, dif, acc);
            }
            if (acc < low) {
                low = acc;
                lj = (uint32_t)j;
            }
        }
        if (slot < cnt && low < INFINITY)
            atomicMin(&best[slot], ((unsigned long long)__float_as_uint(low) << 32) | lj);
    }
}

// Every Gaussian open, without a screening.
__global__ void __launch_bounds__(kNT) vq_open_all_kernel(int64_t n, uint32_t *assign, unsigned long long *best) {
    const int64_t i = (int64_t)blockIdx.x * kNT + threadIdx.x;
    if (i >= n) return;
    best[i] = (unsigned long long)__float_as_uint(INFINITY) << 32;
    assign[i] = kOpen | (uint32_t)i;
}

// The open Gaussians' assignments filled in; with keys, also the (cluster,
// index) pairs of the update's sort.
__global__ void __launch_bounds__(kNT) vq_keys_kernel(uint32_t *assign, const unsigned long long *best, int64_t n,
                                                      uint32_t *keys, uint32_t *vals) {
    const int64_t i = (int64_t)blockIdx.x * kNT + threadIdx.x;
    if (i >= n) return;
    uint32_t a = assign[i];
    if (a & kOpen) {
        a = (uint32_t)best[a & ~kOpen];
        assign[i] = a;
    }
    if (keys) {
        keys[i] = a;
        vals[i] = (uint32_t)i;
    }
}

// Block j (kD lanes, one per component): float64 sum of cluster j's members
// in index order; an empty cluster keeps its vector.  The sum is a serial
// chain by definition, so what counts is that its loads don't wait for each
// other: 64 member indices come in one load, and kAhead vectors are in flight
// at a time (164 -> 15 us an iteration at 200k x 4096, with the vectors as
// rows).
constexpr int kAhead = 16;
template <bool ROWS>
__global__ void __launch_bounds__(64) vq_update_kernel(const float *x, int64_t n, const uint32_t *members, const uint32_t *ranges, float *code) {
    const int lane = threadIdx.x, d = min(lane, kD - 1);
    const uint32_t s = ranges[2 * blockIdx.x], e = ranges[2 * blockIdx.x + 1];
    if (e <= s) return;
    double acc = 0.0;
    for (uint32_t m0 = s; m0 < e; m0 += 64) {
        const int cnt = (int)min(64u, e - m0);
        const int mine = (int)min((int64_t)members[m0 + (uint32_t)min(lane, cnt - 1)], n - 1);
        for (int q0 = 0; q0 < cnt; q0 += kAhead) {
            float v[kAhead];
#pragma unroll
            for (int q = 0; q < kAhead; ++q)
                v[q] = component<ROWS>(x, n, __builtin_amdgcn_readlane(mine, min(q0 + q, cnt - 1)), d);
#pragma unroll
            for (int q = 0; q < kAhead; ++q)
                if (q0 + q < cnt) acc += (double)v[q];
        }
    }
    if (lane < kD) code[(int64_t)blockIdx.x * kD + lane] = (float)(acc / (double)(e - s));
}

inline unsigned blocks(int64_t n, int nt) { return (unsigned)((n + nt - 1) / nt); }

}  // namespace

namespace {

// Models of up to this many Gaussians get a copy of their vectors as rows
// (192 B each, at most 3 GiB); larger ones are read in place.
constexpr int64_t kRowsUpTo = int64_t(1) << 24;

// One piece per workgroup that the device holds (fewer where there is less than
// a stage of tiles for each).
inline Sweep sweep_of(int64_t n, int64_t k) {
    Sweep sw;
    sw.n_blocks = (n + kScreenRows - 1) / kScreenRows;
    sw.n_tiles = (int32_t)((k + kEnt - 1) / kEnt);
    sw.per = ((sw.total() + kScreenGroups - 1) / kScreenGroups + kStage - 1) / kStage * kStage;
    return sw;
}

// lean: only what the update's sort needs (16 bytes per Gaussian); the search's
// 64-bit results then lie in its second buffers.
struct VqScratch {
    bool lean;
    uint32_t *keys, *vals, *keys2, *vals2, *ranges, *open_list, *n_open, *pick;
    unsigned long long *best;
    float *rows, *top1, *top2, *x_norm2, *c_norm2, *start;
    bf16x8 *frag;
    void *sort;
    size_t bytes;
};

VqScratch vq_layout(void *scratch, int64_t n, int64_t k, bool lean) {
    VqScratch v{};
    v.lean = lean;
    uintptr_t at = reinterpret_cast<uintptr_t>(scratch);
    const uintptr_t base = at;
    auto take = [&](size_t bytes) {
        at = (at + 255) & ~uintptr_t(255);
        void *p = reinterpret_cast<void *>(at);
        at += bytes;
        return p;
    };
    const Sweep sw = sweep_of(n, k);
    const int64_t n_tiles = sw.n_tiles;
    const int64_t sn = n * ((n_tiles + sw.per - 1) / sw.per + 1);    // places a block can have
    for (uint32_t **p : {&v.keys, &v.vals})
        *p = static_cast<uint32_t *>(take(sizeof(uint32_t) * n));
    v.ranges = static_cast<uint32_t *>(take(sizeof(uint32_t) * 2 * k));
    if (lean) {
        const int64_t whole = (n + 63) / 64 * 64;
        v.best = static_cast<unsigned long long *>(take(sizeof(unsigned long long) * whole));
        v.keys2 = reinterpret_cast<uint32_t *>(v.best);
        v.vals2 = v.keys2 + whole;
        v.sort = take(sort_scratch_bytes(n));
        v.bytes = at - base + 256;
        return v;
    }
    for (uint32_t **p : {&v.keys2, &v.vals2, &v.open_list}) *p = static_cast<uint32_t *>(take(sizeof(uint32_t) * n));
    v.n_open = static_cast<uint32_t *>(take(sizeof(uint32_t)));
    v.best = static_cast<unsigned long long *>(take(sizeof(unsigned long long) * n));
    v.rows = n <= kRowsUpTo ? static_cast<float *>(take(sizeof(float) * kD * n)) : nullptr;
    v.top1 = static_cast<float *>(take(sizeof(float) * sn));
    v.top2 = static_cast<float *>(take(sizeof(float) * sn));
    v.pick = static_cast<uint32_t *>(take(sizeof(uint32_t) * sn));
    v.x_norm2 = static_cast<float *>(take(sizeof(float) * n));
    v.c_norm2 = static_cast<float *>(take(sizeof(float) * n_tiles * kEnt));
    v.start = static_cast<float *>(take(sizeof(float) * n_tiles * kEnt));
    v.frag = static_cast<bf16x8 *>(take(sizeof(bf16x8) * kFragVecs * n_tiles));
    v.sort = take(sort_scratch_bytes(n));
    v.bytes = at - base + 256;
    return v;
}

}  // namespace

size_t vq_scratch_bytes(int64_t n, int64_t k, bool lean) { return vq_layout(nullptr, n, k, lean).bytes; }

hipError_t vq_kmeans(const float *sh, int64_t n, const uint32_t *init, int64_t k, int32_t iterations, float *code,
                     uint32_t *assign, void *scratch, bool lean, hipStream_t s) {
    if (n <= 0 || k <= 0) return hipSuccess;
    const VqScratch v = vq_layout(scratch, n, k, lean);
    const Sweep sw = sweep_of(n, k);
    const int n_tiles = sw.n_tiles;
    const float *x = v.rows ? v.rows : sh;
    auto assign_all = [&](uint32_t *keys, uint32_t *vals) {
        if (v.lean) {
            hipLaunchKernelGGL(vq_open_all_kernel, dim3(blocks(n, kNT)), dim3(kNT), 0, s, n, assign, v.best);
            hipLaunchKernelGGL(vq_exact_kernel<false>,
                               dim3(blocks(k, kExactEntries), std::min(blocks(n, 64), (unsigned)kLeanGroups)), dim3(64), 0,
                               s, x, n, (const float *)code, k, (const uint32_t *)nullptr, (const uint32_t *)nullptr,
                               v.best);
            hipLaunchKernelGGL(vq_keys_kernel, dim3(blocks(n, kNT)), dim3(kNT), 0, s, assign,
                               (const unsigned long long *)v.best, n, keys, vals);
            return;
        }
        hipLaunchKernelGGL(vq_frag_kernel, dim3((unsigned)n_tiles), dim3(64), 0, s, (const float *)code, k, v.frag,
                           v.start, v.c_norm2, v.n_open);
        hipLaunchKernelGGL(vq_screen_kernel, dim3((unsigned)((sw.total() + sw.per - 1) / sw.per)),
                           dim3(kScreenWaves * 64), 0, s, sh, n, reinterpret_cast<const u32x4 *>(v.frag),
                           (const float *)v.start, sw, v.top1, v.top2, v.pick, v.x_norm2);
        hipLaunchKernelGGL(vq_resolve_kernel, dim3(blocks(n, kNT)), dim3(kNT), 0, s, (const float *)v.top1,
                           (const float *)v.top2, (const uint32_t *)v.pick, (const float *)v.x_norm2,
                           (const float *)v.c_norm2, n, sw, assign, v.open_list, v.best, v.n_open);
        hipLaunchKernelGGL(v.rows ? vq_exact_kernel<true> : vq_exact_kernel<false>,
                           dim3(blocks(k, kExactEntries), std::min(blocks(n, 64), (unsigned)kExactGroups)), dim3(64), 0,
                           s, x, n, (const float *)code, k, (const uint32_t *)v.open_list, (const uint32_t *)v.n_open,
                           v.best);
        hipLaunchKernelGGL(vq_keys_kernel, dim3(blocks(n, kNT)), dim3(kNT), 0, s, assign,
                           (const unsigned long long *)v.best, n, keys, vals);
    };
    if (v.rows)
        hipLaunchKernelGGL(vq_rows_kernel, dim3(blocks(n, kRowTile)), dim3(kNT), 0, s, sh, n, v.rows);
    hipLaunchKernelGGL(vq_gather_kernel, dim3(blocks(k * kD, kNT)), dim3(kNT), 0, s, sh, n, init, k, code);
    for (int32_t it = 0; it < iterations; ++it) {
        assign_all(v.keys, v.vals);
        int alt = 0;
        int bits = 1;
        while (bits < 32 && (int64_t(1) << bits) < k) ++bits;
        hipError_t e = radix_sort_u32(v.keys, v.vals, v.keys2, v.vals2, nullptr, n, 0, bits, v.sort, &alt, s);
        if (e != hipSuccess) return e;
        const uint32_t *sk = alt ? v.keys2 : v.keys, *sv = alt ? v.vals2 : v.vals;
        e = launch_tile_ranges(sk, nullptr, n, (int32_t)k, v.ranges, s);
        if (e != hipSuccess) return e;
        hipLaunchKernelGGL(v.rows ? vq_update_kernel<true> : vq_update_kernel<false>, dim3((unsigned)k), dim3(64), 0, s,
                           x, n, sv, (const uint32_t *)v.ranges, code);
    }
    assign_all(nullptr, nullptr);
    return hipGetLastError();
}

}  // namespace fdgs
