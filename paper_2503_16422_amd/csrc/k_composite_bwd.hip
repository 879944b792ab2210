// Adjoint of the per-tile compositing (Eq. 2 and Eq. 3 differentiated with
// respect to each record's centre, conic, opacity and colour).
#include <hip/hip_runtime.h>

#include <algorithm>

#include "dev_composite.h"
#include "dev_util.h"
#include "fdgs_internal.h"

namespace fdgs {
namespace {

using namespace comp;

struct BwdArgs {
    RenderParams rp;
    int32_t W, H;
    const uint32_t *ranges;
    const uint32_t *ids;
    const Rec2D *rec;
    const float *T_final;
    const uint32_t *n_contrib;
    const float *dL;
    G2d g2d;           // per entry: du, dv, d conic a, b, c, d opacity, d rgb
    const uint32_t *order;   // tiles longest list first (workgroup b takes tile order[b]), or NULL: raster order
};

// Adjoint, walking each pixel's list back to front from its last contributor.
// The transmittance in front of Gaussian i is recovered as T_{i+1} / (1 - a_i)
// from the stored final T, so no per-pixel list is kept.  With g = dL/dC, the
// colour behind i seen from just behind it, R_i = (colour behind i + T_final
// bg) . g / T_{i+1}, obeys R_{i-1} = R_i + a_i (c_i . g - R_i) from R = bg . g
// at the last contributor, and
//   dL/dc_i = a_i T_i g,    dL/da_i = T_i (c_i . g - R_i),
// then a_i = min(a_max, o_i G_i) -> (o_i, conic, centre).  With d_i = a_i
// dL/da_i at the pixels where the clamp is inactive (the derivative of alpha
// with respect to the exponent), every conic and centre gradient is a linear
// combination of per-Gaussian sums over the pixels, (dx, dy) = pixel centre -
// Gaussian centre and v = q (dy + s dx) the exponent's scaled distance to the
// footprint's centre line (log2 G = lo + kx dx^2 - v^2):
//   dL/du = -2 ln2 (kx sum d dx - q s sum d v),   dL/dv = 2 ln2 q sum d v,
//   dL/d(a, b, c) = -1/2 sum d dx^2, -sum d dx dy, -1/2 sum d dy^2,
//   dL/do = sum d / o
// (the centre terms in the exponent's own form, which does not cancel for
// needle-shaped footprints).  A pixel adds four of these sums (its column's
// dx gives the rest) and the conversion happens once per Gaussian and tile.
// A thread owns PPT pixels of a column of its wavefront's cell (the forward's
// layout).  The nine sums of two records at a time are reduced over the
// wavefront together (wave_sums18), leaving one sum in each of 18 lanes, which
// add them into the tile's LDS accumulators with one instruction.  After each
// batch the sums leave the tile as gradients, nine consecutive lanes to the
// nine values of a Gaussian, which share one 128-byte line of g2d: an atomic
// instruction then touches eight or nine lines, where a thread per Gaussian
// touched 64 lines nine times.  Over the tiles the gradients add up in float64: a
// large footprint's terms cancel over hundreds of tiles, and the parameter adjoint
// amplifies what float32 sums in arbitrary order leave.  (Fine-tuning frame, 200k
// Gaussians, 16x16 tiles: adjoint 500 -> 238 us, of which the global adds took 190
// and the LDS adds 68; training view, 500k, 32x32: 311 -> 227 us.)  A wavefront
// walks only the records whose footprint ellipse reaches its cell: the others have
// alpha below alpha_min at every one of its pixels and contribute nothing.
template <int CTRL>
__device__ __forceinline__ float dpp_of(float v) {
    return __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, v), CTRL, 0xf, 0xf, true));
}
constexpr int kVals = 9;   // sums of d, d dx, d v, d dx^2, d dx dy, d dy^2; colour r, g, b

// fold_halves over each pair of rows of 16 lanes: a in the even rows, b in the odd ones.
__device__ __forceinline__ float fold16(float a, float b) {
    const auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(a), __float_as_uint(b), false, false);
    return __uint_as_float(r[0]) + __uint_as_float(r[1]);
}
// Sums over the wavefront of nine values of two records, one in each of 18
// lanes.  Every step folds two quantities into one register whose lane halves
// hold one each, so the work halves from step to step: 44 vector instructions
// for 18 sums.  The first lane of each group of four holds value
// 0 to 7 as lane_value says, lanes 1 and 33 value 8.
__device__ __forceinline__ float wave_sums18(const float (&v1)[kVals], const float (&v2)[kVals], int lane) {
    float x[kVals];
#pragma unroll
    for (int j = 0; j < kVals; ++j) x[j] = fold_halves(v1[j], v2[j]);          // record = lane / 32
    float y[5];
#pragma unroll
    for (int j = 0; j < 4; ++j) y[j] = fold16(x[2 * j], x[2 * j + 1]);    // value's bit 0 = lane / 16 % 2
    y[4] = fold16(x[8], x[8]);
#pragma unroll
    for (int j = 0; j < 5; ++j) y[j] += dpp_of<0x128>(y[j]);              // row_ror:8
    const float z0 = (lane & 8) ? y[1] : y[0];                            // bit 1 = lane / 8 % 2
    const float z1 = (lane & 8) ? y[3] : y[2];
    const float w0 = z0 + dpp_of<0x141>(z0), w1 = z1 + dpp_of<0x141>(z1); // row_half_mirror
    float s = (lane & 4) ? w1 : w0;                                       // bit 2 = lane / 4 % 2
    float e = y[4] + dpp_of<0x141>(y[4]);
    s += dpp_of<0x4E>(s);                                                 // quad_perm(2,3,0,1)
    e += dpp_of<0x4E>(e);
    s += dpp_of<0xB1>(s);                                                 // quad_perm(1,0,3,2)
    e += dpp_of<0xB1>(e);
    return (lane & 3) == 0 ? s : e;
}
// The value whose sum lane holds for record lane / 32, or -1 where another lane has it.
__device__ __forceinline__ int lane_value(int lane) {
    if ((lane & 3) == 0) return ((lane >> 4) & 1) | ((lane >> 3) & 1) << 1 | ((lane >> 2) & 1) << 2;
    return (lane & 31) == 1 ? 8 : -1;
}

template <int TW, int TH, int BATCH, int PPT>
__global__ void __launch_bounds__(TW *TH / PPT) composite_bwd_kernel(BwdArgs a) {
    constexpr int NT = TW * TH / PPT;
    using C = Cells<TW, TH, PPT>;
    // per-wavefront bitmaps of the batch's records that reach its cell (as in the forward)
    constexpr bool kBits = C::NW > 1;
    constexpr int kWords = BATCH / 64;
    __shared__ uint64_t s_bits[kBits ? C::NW * kWords : 1];
    // per staged record three float4: gx, q s, c0, kx | log2 opacity, q, r, g | b, gy, opacity, id
    __shared__ float4 s_rec[3 * BATCH];
    __shared__ float s_acc[BATCH * kVals];   // per-Gaussian sums of the tile
    // the longest lists first, as in the forward's longest-first schedule: they
    // run beside the rest of the launch instead of alone at its end
    const int tile = a.order ? (int)a.order[blockIdx.x] : (int)blockIdx.x;
    const int tx = tile % a.rp.tiles_x, ty = tile / a.rp.tiles_x;
    const int wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x / 64), lane = lane_id();
    const int lx = (wave % C::CX) * C::CW + lane % C::CW, ly0 = (wave / C::CX) * C::CH + (lane / C::CW) * PPT;
    const int px = tx * TW + lx, py0 = ty * TH + ly0;
    const int bx0 = ((tx * TW) & ~(kBlockSize - 1)) + kBlockHalf;   // as in the forward
    const int by0 = ((ty * TH) & ~(kBlockSize - 1)) + kBlockHalf;
    const float fx = (float)(px - bx0) + 0.5f;
    const float ox = (float)bx0, oy = (float)by0;
    const uint32_t start = a.ranges[2 * tile];
    const float amin = a.rp.alpha_min, amax = a.rp.alpha_max;
    const uint32_t amax_bits = __float_as_uint(amax);
    const int64_t plane = (int64_t)a.W * a.H;
    float fy[PPT], g0[PPT], g1[PPT], g2[PPT], T[PPT], R[PPT];
    uint32_t last[PPT];
    uint32_t my_max = 0;
#pragma unroll
    for (int p = 0; p < PPT; ++p) {
        const int py = py0 + p;
        fy[p] = (float)(py - by0) + 0.5f;
        g0[p] = g1[p] = g2[p] = 0.f;
        T[p] = 1.f;
        last[p] = 0;
        if (px < a.W && py < a.H) {
            const int64_t pix = (int64_t)py * a.W + px;
            g0[p] = a.dL[pix];
            g1[p] = a.dL[plane + pix];
            g2[p] = a.dL[2 * plane + pix];
            T[p] = a.T_final[pix];
            last[p] = a.n_contrib[pix];
        }
        R[p] = a.rp.bg[0] * g0[p] + a.rp.bg[1] * g1[p] + a.rp.bg[2] * g2[p];   // bg . g
        my_max = max(my_max, last[p]);
    }
    // block-wide maximum of `last` bounds the walk
    __shared__ uint32_t s_max;
    if (threadIdx.x == 0) s_max = 0;
    __syncthreads();
    atomicMax(&s_max, my_max);
    __syncthreads();
    const uint32_t walk_end = start + s_max;
    for (int j = threadIdx.x; j < BATCH * kVals; j += NT) s_acc[j] = 0.0f;
    const int my_value = lane_value(lane);
    for (int64_t top = (int64_t)walk_end; top > (int64_t)start; top -= BATCH) {
        const uint32_t lo = (uint32_t)max((int64_t)start, top - BATCH);
        const int cnt = (int)(top - lo);
        __syncthreads();
        for (int k0 = 0; k0 < cnt; k0 += NT) {
            const int k = k0 + (int)threadIdx.x;
            uint32_t cells = 0u;
            if (k < cnt) {
                const uint32_t id = a.ids[lo + k];
                const Rec2D r = a.rec[id];
                const ExpRec q = stage_exp(r, ox, oy);
                s_rec[3 * k] = make_float4(q.gx, q.s, q.c0, q.kx);
                s_rec[3 * k + 1] = make_float4(q.lo, q.q, r.c.x, r.c.y);
                s_rec[3 * k + 2] = make_float4(r.c.z, q.gy, r.b.w, __uint_as_float(id));
                if constexpr (kBits) cells = reached_cells<TW, TH, PPT>(r, a.rp, tx * TW, ty * TH);
            }
            if constexpr (kBits) {
                const int word = k0 / 64 + wave;
#pragma unroll
                for (int w = 0; w < C::NW; ++w) {
                    const uint64_t m = __ballot((cells >> w) & 1u);
                    if (lane == 0 && word < kWords) s_bits[w * kWords + word] = m;
                }
            }
        }
        __syncthreads();
        // alpha of record k at the thread's pixels: raw = opacity x G, and the
        // clamped alpha where the forward blended it (its position before the
        // pixel's last contributor and alpha >= alpha_min), else 0; also the
        // column offset dx and each pixel's centre-line distance v
        auto alphas = [&](int k, bool real, float &dx, float (&vl)[PPT], float (&raw)[PPT], float (&al)[PPT]) {
            const uint32_t pos = lo + k - start;   // position in the tile list
            const float4 g = s_rec[3 * k];
            const float4 h = s_rec[3 * k + 1];
            dx = fx - g.x;
            const float A = exp2_col_a(g.w, h.x, dx), B = exp2_col_t(g.y, g.z, fx);
#pragma unroll
            for (int p = 0; p < PPT; ++p) {
                vl[p] = exp2_line(h.y, B, fy[p]);   // the forward's exponent, term by term
                raw[p] = __builtin_amdgcn_exp2f(fmaf(-vl[p], vl[p], A));
                const float alpha = clamp_alpha(raw[p], amax_bits);
                al[p] = (real && pos < last[p] && alpha >= amin) ? alpha : 0.0f;
            }
        };
        // record k's terms at the thread's pixels, back to front (an alpha of 0
        // leaves T and R unchanged and adds nothing)
        auto grad = [&](int k, float dx, const float (&vl)[PPT], const float (&raw)[PPT], const float (&al)[PPT],
                        float (&v)[kVals]) {
            const float4 h = s_rec[3 * k + 1];
            const float4 e = s_rec[3 * k + 2];   // b, gy, -, id
            // the moments in y from each pixel's own dy: expanded about one pixel of the
            // column they cancel for footprints thin in y that lie beside another (of four
            // pixels a thread: 20 times the error of log_scale's gradient)
            float D = 0.f, Dv = 0.f, Dy = 0.f, Dyy = 0.f;
            v[6] = v[7] = v[8] = 0.f;
#pragma unroll
            for (int p = 0; p < PPT; ++p) {
                T[p] *= __builtin_amdgcn_rcpf(1.0f - al[p]);   // transmittance in front of i
                const float w = al[p] * T[p];
                v[6] = fmaf(w, g0[p], v[6]);
                v[7] = fmaf(w, g1[p], v[7]);
                v[8] = fmaf(w, g2[p], v[8]);
                const float d = fmaf(h.z, g0[p], fmaf(h.w, g1[p], e.x * g2[p])) - R[p];   // c.g - R
                R[p] = fmaf(al[p], d, R[p]);
                const float dpow = raw[p] < amax ? al[p] * (T[p] * d) : 0.0f;
                D += dpow;
                Dv = fmaf(vl[p], dpow, Dv);
                const float dy = fy[p] - e.y;
                Dy = fmaf(dy, dpow, Dy);
                Dyy = fmaf(dy * dy, dpow, Dyy);
            }
            v[0] = D;
            v[1] = dx * D;
            v[2] = Dv;
            v[3] = (dx * dx) * D;
            v[4] = dx * Dy;
            v[5] = Dyy;
        };
        // records k1 (behind) then k2 (in front); with real2 false only k1
        auto pair = [&](int k1, int k2, bool real2) {
            float x1, x2, l1[PPT], l2[PPT], r1[PPT], a1[PPT], r2[PPT], a2[PPT];
            alphas(k1, true, x1, l1, r1, a1);
            alphas(k2, real2, x2, l2, r2, a2);
            bool any = false;
#pragma unroll
            for (int p = 0; p < PPT; ++p) any = any || a1[p] > 0.0f || a2[p] > 0.0f;
            if (__ballot(any) == 0ull) return;
            float v1[kVals], v2[kVals];
            grad(k1, x1, l1, r1, a1, v1);
            grad(k2, x2, l2, r2, a2, v2);
            const float sum = wave_sums18(v1, v2, lane);
            if (my_value >= 0 && (lane < 32 || real2)) atomicAdd(s_acc + (lane < 32 ? k1 : k2) * kVals + my_value, sum);
        };
        if constexpr (kBits) {
            // only the records whose ellipse reaches this wavefront's cell, back to front
            for (int c = (cnt - 1) / 64; c >= 0; --c) {
                const uint64_t word = s_bits[wave * kWords + c];
                uint64_t bits = ((uint64_t)(uint32_t)__builtin_amdgcn_readfirstlane((int)(word >> 32)) << 32) |
                                (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)word);
                while (bits != 0ull) {
                    const int b1 = 63 - __builtin_clzll(bits);
                    const uint64_t rest = bits & ~(1ull << b1);
                    const bool two = rest != 0ull;
                    const int b2 = two ? 63 - __builtin_clzll(rest) : b1;
                    bits = two ? rest & ~(1ull << b2) : 0ull;
                    pair(c * 64 + b1, c * 64 + b2, two);
                }
            }
        } else {
            for (int k = cnt - 1; k >= 0; k -= 2) pair(k, k > 0 ? k - 1 : k, k > 0);
        }
        __syncthreads();
        // sums to gradients, one global add per (Gaussian, value) for the whole tile
        for (int i = threadIdx.x; i < cnt * kVals; i += NT) {
            const int k = i / kVals, j = i - k * kVals;
            float out = s_acc[i];                                // d r, g, b
            if (j < 6) {
                // value j from the sums m (j = 0: m and m2); a record no pixel blended
                // leaves its zeros alone (its opacity can be 0, its kx infinite)
                const float m = s_acc[k * kVals + (j < 5 ? j + 1 : 0)], m2 = j == 0 ? s_acc[k * kVals + 2] : 0.0f;
                const float4 g = s_rec[3 * k];                   // gx, q s, c0, kx
                if (m == 0.0f && m2 == 0.0f) out = 0.0f;
                else if (j == 0) out = -2.0f * kLn2 * (g.w * m - g.y * m2);       // d u
                else if (j == 1) out = 2.0f * kLn2 * s_rec[3 * k + 1].y * m;      // d v
                else if (j == 5) out = m / s_rec[3 * k + 2].z;                    // d opacity
                else out = (j == 3 ? -1.0f : -0.5f) * m;                          // d conic a, b, c
            }
            if (out == 0.0f) continue;
            const int64_t id = (int64_t)__float_as_uint(s_rec[3 * k + 2].w);
            if (a.g2d.wide) atomicAdd(a.g2d.line(id) + j, (double)out);   // uniform
            else atomicAdd(a.g2d.narrow(id) + j, out);
        }
        __syncthreads();
        for (int i = threadIdx.x; i < cnt * kVals; i += NT) s_acc[i] = 0.0f;
    }
}

// Zeroes the visible Gaussians' values of g2d, the only ones the adjoint adds to and reads: PER
// pieces of type T per Gaussian.
template <typename T, int PER>
__global__ void __launch_bounds__(256) clear_g2d_kernel(const uint32_t *vis_list, const int64_t *n_vis_dev, int64_t n_max,
                                                        T *g2d) {
    const int64_t n = min(*n_vis_dev, n_max) * PER;
    for (int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x; i < n; i += (int64_t)gridDim.x * 256)
        g2d[(int64_t)vis_list[i / PER] * PER + i % PER] = T{};
}

// Pixels per thread in the adjoint: 1 for 8x8 tiles, else 4 when the forward
// took 4 and 2 otherwise.
struct BwdLaunch {
    BwdArgs a;
    int32_t ppt;
};
template <int TW, int TH, int BATCH>
void launch_bwd(const BwdLaunch &l, int n_tiles, hipStream_t s) {
    if constexpr (TW * TH == 64) {
        hipLaunchKernelGGL((composite_bwd_kernel<TW, TH, BATCH, 1>), dim3(n_tiles), dim3(64), 0, s, l.a);
    } else if (l.ppt == 4) {
        hipLaunchKernelGGL((composite_bwd_kernel<TW, TH, BATCH, 4>), dim3(n_tiles), dim3(TW * TH / 4), 0, s, l.a);
    } else {
        hipLaunchKernelGGL((composite_bwd_kernel<TW, TH, BATCH, 2>), dim3(n_tiles), dim3(TW * TH / 2), 0, s, l.a);
    }
}

}  // namespace

hipError_t launch_composite_backward(const RenderParams &rp, int32_t W, int32_t H, int32_t batch, int32_t ppt,
                                     const uint32_t *ranges, const uint32_t *ids, const Rec2D *rec,
                                     const float *T_final, const uint32_t *n_contrib,
                                     const float *dL_drgb, G2d g2d, int64_t /*n_proc_max*/,
                                     const uint32_t *order, hipStream_t s) {
    BwdLaunch l{BwdArgs{rp, W, H, ranges, ids, rec, T_final, n_contrib, dL_drgb, g2d, order}, ppt};
    const int n_tiles = rp.tiles_x * rp.tiles_y;
    FDGS_DISPATCH(launch_bwd, l);
    return hipGetLastError();
}

hipError_t launch_clear_g2d(const uint32_t *vis_list, const int64_t *n_vis_dev, int64_t n_max, G2d g2d, hipStream_t s) {
    if (n_max == 0) return hipSuccess;
    const dim3 grid((unsigned)std::min<int64_t>((n_max * (kG2dStride / 2) + 255) / 256, 2048));
    if (g2d.wide)
        hipLaunchKernelGGL((clear_g2d_kernel<double2, kG2dStride / 2>), grid, dim3(256), 0, s, vis_list, n_vis_dev, n_max,
                           static_cast<double2 *>(g2d.p));
    else
        hipLaunchKernelGGL((clear_g2d_kernel<float, kG2dVals>), grid, dim3(256), 0, s, vis_list, n_vis_dev, n_max,
                           static_cast<float *>(g2d.p));
    return hipGetLastError();
}

}  // namespace fdgs
