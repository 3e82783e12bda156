// gfx950 kernels of the ray march (arXiv 2604.11856, Sec. 2.2.3): per (ray,
// spectral chunk) the RTE march far -> target with the spectral trapezoid
// fused in, in the cell-constant or the linear-j segment scheme, and the
// deterministic sums of per-block partials and of ray fluxes.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <cstdint>
#include <type_traits>

#include "lrt_device.h"
#include "lrt_internal.h"
#include "lrt_math.h"

namespace lrt {

namespace {

// One row (the PPT consecutive points k0.. of a lane) of eta and kappa, from the
// wave's first point in the rows of the segment's cell (the same for the whole
// wave, so the loads take a 64-bit scalar base, which bands of any length need,
// and the lane's 32-bit offset from it); left: points of the band from there.
template <int PPT, typename T>
__device__ __forceinline__ void load_row(const T *erow, const T *krow, uint32_t k0, int32_t left, bool vec,
                                         T (&ev)[PPT], T (&kv)[PPT])
{
    if (vec) {   // vector loads of up to 16 bytes
        constexpr int V = sizeof(T) == 4 ? PPT : 2;
        // (aligned to the element only: global loads take any such address)
        typedef T Vec __attribute__((ext_vector_type(V), aligned(sizeof(T))));
#pragma unroll
        for (int j = 0; j < PPT; j += V) {
            const Vec a = *(const Vec *)((const char *)erow + k0 * (uint32_t)sizeof(T) + j * sizeof(T));
            const Vec b = *(const Vec *)((const char *)krow + k0 * (uint32_t)sizeof(T) + j * sizeof(T));
#pragma unroll
            for (int i = 0; i < V; ++i) {
                ev[j + i] = a[i];
                kv[j + i] = b[i];
            }
        }
        return;
    }
#pragma unroll
    for (int j = 0; j < PPT; ++j) {
        const bool ok = (int32_t)k0 + j < left;
        ev[j] = ok ? erow[k0 + j] : (T)0;
        kv[j] = ok ? krow[k0 + j] : (T)0;
    }
}

// March of one (ray, chunk of 64 x PPT points), far -> target.
//   LINEAR = false: cell-constant segments, I <- I e^-tau + eta ds F(tau).
//   LINEAR = true: linear-j segments between LOS nodes at the far end of the
//     ray, the midpoint of every cell segment and the target; a node takes its
//     cell's state, so the node spacings are ds_0/2, (ds_m-1 + ds_m)/2, ...,
//     ds_M-1/2, and each segment uses the far node's kappa.
// T_far (NULL: all free) gives per ray the temperature of a solid far
// boundary (0: free), whose blackbody intensity starts the march.
// The (ray, chunk) of wave `wave` of workgroup b (b: index in the whole grid,
// launch offset b0 + blockIdx.x): the workgroup owns RAYS rays x (4 / RAYS)
// consecutive chunks, one (ray, chunk) per wave.  Workgroups go round-robin to
// the 8 XCDs (b % 8), each with its own L2.  Without `shared`, XCD x takes a
// contiguous range of the chunk-major items, so every ray of a spectral chunk
// runs on one XCD and the rows the rays share come from that XCD's L2; with it
// the items are taken in their own chunk-major order, so all XCDs work on the
// same chunk, whose rows stay in the chip-wide last-level cache.  When every
// wall point has the same rays (per_wall > 0) a chunk's rays are taken
// direction-major: the rays an XCD runs together are then nearly parallel lines
// from neighbouring wall points, which cross nearly the same cells.  A bijection
// onto [0, n_rays) x [0, n_chunks) for any sizes (ray = -1 for the waves past
// the last ray or chunk).  (A contiguous range of each chunk's rays per XCD was
// 60 % slower: the directions' paths differ in length.)
template <int RAYS>
__device__ __forceinline__ void march_item(uint32_t b, int32_t wave, const DevRays &rays, int32_t n_chunks,
                                           int32_t shared, int &ray, int &chunk)
{
    constexpr int CHUNKS = kMarchThreads / 64 / RAYS;
    const uint32_t n_groups = ((uint32_t)rays.n_rays + RAYS - 1) / RAYS;
    const uint32_t n_cgroups = ((uint32_t)n_chunks + CHUNKS - 1) / CHUNKS;
    const uint32_t n = n_groups * n_cgroups, x = b % kXCDs, i = b / kXCDs;
    const uint32_t per = n / kXCDs, rem = n % kXCDs;
    const uint32_t gi = shared ? b : x * per + min(x, rem) + i;
    chunk = (int)(gi / n_groups) * CHUNKS + wave / RAYS;
    const int32_t q = (int32_t)(gi % n_groups) * RAYS + wave % RAYS;
    if (q >= rays.n_rays || chunk >= n_chunks) {
        ray = -1;   // past the last ray or chunk: this wave has nothing to do
    } else if (rays.per_wall > 0) {
        const int32_t n_wall = rays.n_rays / rays.per_wall;
        ray = (q % n_wall) * rays.per_wall + q / n_wall;   // direction-major
    } else {
        ray = q;
    }
}

//
// The rays' segments come 64 at a time, one per lane: its cell, its length and
// the factors of the segment law from the length and the cell's scales.  The
// wave then walks them, the segment's values broadcast from its lane, its rows
// (one vector load per array) requested kAhead segments before they are used,
// so that few rays, too few waves to hide a load behind each other, do not wait
// for every row in turn.
template <typename T>
__device__ __forceinline__ T lane_value(T v, int l)
{
    if constexpr (sizeof(T) == 8) {
        const uint64_t b = __builtin_bit_cast(uint64_t, v);
        const uint32_t lo = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)b, l);
        const uint32_t hi = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)(b >> 32), l);
        return __builtin_bit_cast(T, ((uint64_t)hi << 32) | lo);
    } else {
        return __builtin_bit_cast(T, __builtin_amdgcn_readlane(__builtin_bit_cast(int, v), l));
    }
}

template <bool FP32, bool LINEAR, int PPT, int RAYS>
__global__ __launch_bounds__(kMarchThreads) void march_kernel(
    DevRays rays, DevGrid g, int32_t k_first, int32_t n_band, const void *eta_v,
    const void *kappa_v, const int32_t *escale, const double *T_far, double *I_out,
    double *partials, int32_t n_chunks, int32_t shared, uint32_t b0)
{
    const int lane = threadIdx.x & 63, wave = uniform_i(threadIdx.x >> 6);
    int ray, chunk;
    march_item<RAYS>(b0 + blockIdx.x, wave, rays, n_chunks, shared, ray, chunk);
    if (ray < 0) return;
    // The wave's first point, band-relative.  The last chunk of a band that ends
    // inside one is moved back to end with the band, so that its rows come by
    // vector loads too; the points before its own are the chunk before's (skip).
    // With guarded loads, point by point, one wave of it took as long as three
    // others and held its XCD up (2,048 cells, 6,144 rays: 284 us on 1,000 points,
    // 184 on 1,024).
    const int32_t start = min(chunk * (64 * PPT), max(n_band - 64 * PPT, 0));
    const int32_t skip = chunk * (64 * PPT) - start;
    const int32_t left = n_band - start;        // points of the band from there on
    const int32_t k0 = lane * PPT;              // the lane's first point, from there
    const int64_t m0 = rays.off[ray], m1 = rays.off[ray + 1];
    double I[PPT];
    const double Tw = T_far ? T_far[ray] : 0.0;
#pragma unroll
    for (int j = 0; j < PPT; ++j) {
        I[j] = 0.0;
        if (Tw > 0.0 && k0 + j < left) I[j] = planck_f64(g.nu_min + (double)(k_first + start + k0 + j) * g.h, Tw);
    }
    // vector loads unless the band is shorter than a chunk
    const bool vec = left >= 64 * PPT;
    using T = std::conditional_t<FP32, float, double>;
    const T *eta = (const T *)eta_v;
    const T *kap = (const T *)kappa_v;
    constexpr int kAhead = FP32 ? 4 : 2;
    T ev[kAhead][PPT], kv[kAhead][PPT];

    // linear-j: the far node of the next segment (its coefficients, scales and length)
    [[maybe_unused]] T pe[PPT], pk[PPT];
    [[maybe_unused]] int32_t pee = 0, pek = 0;
    [[maybe_unused]] double pds = 0.0;
    // one linear-j segment from node (fe, fk) to node ne, lengths scaled by the
    // nodes' powers of two (Lf = Ln = L and Lk = L in double precision).  Where many
    // waves keep the vector units busy (256-point chunks) a point at which the whole
    // wave is thin takes the series alone, and the points one after the other need
    // fewer registers; few waves would wait for the vote instead.
    constexpr bool kThinVote = FP32 && PPT == 4;
    [[maybe_unused]] auto linear_segment = [&](const T (&fe)[PPT], const T (&fk)[PPT], const T (&ne)[PPT], double Lf,
                                               double Ln, T Lk) {
#pragma unroll
        for (int j = 0; j < PPT; ++j) {
            if constexpr (FP32) {
                const float t = fk[j] * Lk;
                float wf, wn;
                if constexpr (kThinVote) {
                    linear_j_series_f32(t, wf, wn);
                    if (__all(fabsf(t) < kLinearThin)) {
                        // 1 - e^-t = t f with f = wf + wn
                        const double x = (double)(t * (wf + wn));
                        I[j] = fma(-x, I[j], fma((double)(wf * fe[j]), Lf, fma((double)(wn * ne[j]), Ln, I[j])));
                        continue;
                    }
                }
                const float e = __builtin_amdgcn_exp2f(t * (float)(-kLog2e));
                linear_j_weights_f32(t, e, wf, wn);
                I[j] = fma(I[j], (double)e, (double)(wf * fe[j]) * Lf + (double)(wn * ne[j]) * Ln);
            } else {
                const LinearLaw w = linear_law(fk[j] * Lk);
                I[j] = I[j] * w.e + Lf * (w.far * fe[j] + w.near * ne[j]);
            }
        }
    };

    // the segment loop, with vector or guarded row loads chosen once outside it
    const int32_t n_seg = (int32_t)(m1 - m0);
    auto march = [&](auto vec_c) {
        auto load = [&](int slot, int32_t c) {
            const int64_t row = (int64_t)c * n_band + start;
            load_row<PPT, T>(eta + row, kap + row, (uint32_t)k0, left, decltype(vec_c)::value, ev[slot], kv[slot]);
        };
        for (int32_t i0 = 0; i0 < n_seg; i0 += 64) {
            const int32_t n = min(64, n_seg - i0);
            int32_t c = 0, ee = 0, ek = 0;
            double ds = 0.0;
            if (lane < n) {
                c = rays.cell[m0 + i0 + lane];
                ds = rays.ds[m0 + i0 + lane];
                if constexpr (FP32) {
                    ee = escale[2 * c + 0];
                    ek = escale[2 * c + 1];
                }
            }
            // the segment's factors, per lane: cell-constant dsu, dsl; linear-j
            // (far node: the previous lane's, or the last of the previous 64,
            // or at the far end the segment's own with half its length) Lf, Ln, Lk
            [[maybe_unused]] float dsu = 0.0f;
            [[maybe_unused]] double dsl = 0.0, Lf = 0.0, Ln = 0.0;
            [[maybe_unused]] T Lk = 0;
            if constexpr (!LINEAR) {
                if constexpr (FP32) segment_scales(ds, ee, ek, dsu, dsl);
            } else {
                double fds = __shfl_up(ds, 1);
                int32_t fee = __shfl_up(ee, 1), fek = __shfl_up(ek, 1);
                if (lane == 0) {
                    fds = i0 > 0 ? pds : 0.0;
                    fee = i0 > 0 ? pee : ee;
                    fek = i0 > 0 ? pek : ek;
                }
                const double L = 0.5 * (fds + ds);
                Lf = ldexp(L, fee);
                Ln = ldexp(L, ee);
                Lk = FP32 ? (T)fmin(ldexp(L, fek), 3.0e38) : (T)L;
                pds = lane_value(ds, n - 1);
                pee = lane_value(ee, n - 1);
                pek = lane_value(ek, n - 1);
            }
#pragma unroll
            for (int j = 0; j < kAhead; ++j)
                if (j < n) load(j, lane_value(c, j));
            for (int32_t s0 = 0; s0 < n; s0 += kAhead) {
#pragma unroll
                for (int q = 0; q < kAhead; ++q) {
                    const int32_t s = s0 + q;
                    if (s >= n) break;
                    if constexpr (LINEAR) {
                        const double lf = lane_value(Lf, s), ln = FP32 ? lane_value(Ln, s) : lf;
                        const T lk = FP32 ? lane_value(Lk, s) : (T)lf;
                        if (i0 + s == 0)
                            linear_segment(ev[q], kv[q], ev[q], lf, ln, lk);   // far end -> first midpoint
                        else
                            linear_segment(pe, pk, ev[q], lf, ln, lk);         // midpoint -> midpoint
#pragma unroll
                        for (int j = 0; j < PPT; ++j) {
                            pe[j] = ev[q][j];
                            pk[j] = kv[q][j];
                        }
                    } else if constexpr (FP32) {
                        segment_points_f32<PPT>(ev[q], kv[q], lane_value(dsu, s), lane_value(dsl, s), I);
                    } else {
                        const double d = lane_value(ds, s);
#pragma unroll
                        for (int j = 0; j < PPT; ++j) {
                            const CellLaw w = cell_law(kv[q][j] * d);
                            // (three operations; with fma(I, 1 + em, source), four,
                            // 1.57 -> 1.61 ms, and after 150 cells an error of 3.9e-16
                            // against 3.4, a library's functions and divisions 4.3)
                            I[j] = fma(I[j], w.em, I[j]) + ev[q][j] * d * w.f;
                        }
                    }
                    if (s + kAhead < n) load(q, lane_value(c, s + kAhead));
                }
            }
        }
    };
    if (vec)
        march(std::true_type{});
    else
        march(std::false_type{});
    if constexpr (LINEAR) {
        if (n_seg > 0) {   // last midpoint -> target
            const double L = 0.5 * pds;
            linear_segment(pe, pk, pe, ldexp(L, pee), ldexp(L, pee),
                           FP32 ? (T)fmin(ldexp(L, pek), 3.0e38) : (T)L);
        }
    }
    // outputs: I and the trapezoid partial with global-index weights
    double part = 0.0;
#pragma unroll
    for (int j = 0; j < PPT; ++j) {
        if (k0 + j >= skip && k0 + j < left) {
            const int32_t kl = start + k0 + j, kg = k_first + kl;
            const double w = (kg == 0 || kg == g.n_points - 1) ? 0.5 * g.h : g.h;
            part += w * I[j];
            if (I_out) I_out[(int64_t)ray * n_band + kl] = I[j];
        }
    }
    // the wave's sum in a fixed order (xor-shuffles)
    for (int o = 32; o > 0; o >>= 1) part += __shfl_xor(part, o);
    if (lane == 0) partials[(int64_t)ray * n_chunks + chunk] = part;
}

// Row sums of the march's per-chunk partials, 2^lg lanes to a row: each lane
// takes every 2^lg-th column, then the lanes are summed by xor-shuffles, a fixed
// order for a given row length.  acc (NULL: none) receives the running sum over
// calls (set by the first, added to by the others), acc_host (NULL: none) a copy of it
// in pinned host memory.  (One thread per row, its loads one after the other,
// took 813 us on the stagnation line's 17 rows of 8,192 and 16 us on 8 rows of
// 118.)
__global__ void reduce_rows_kernel(const double *p, int32_t n_rows, int32_t n_cols, int32_t lg, double *out,
                                   double *acc, int32_t first, double *acc_host)
{
    const int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    const int64_t r = t >> lg;
    const int lane = (int)(t & ((1 << lg) - 1));
    double s = 0.0;
    if (r < n_rows) {
        const double *row = p + r * n_cols;
#pragma unroll 8
        for (int j = lane; j < n_cols; j += 1 << lg) s += row[j];
    }
    for (int o = (1 << lg) >> 1; o > 0; o >>= 1) s += __shfl_xor(s, o);
    if (lane == 0 && r < n_rows) {
        out[r] = s;
        if (acc) {
            const double v = first ? s : acc[r] + s;
            acc[r] = v;
            if (acc_host) acc_host[r] = v;
        }
    }
}

// Flux of each wall point, one wave per wall point: its rays over the lanes,
// then the lanes by xor-shuffles.
__global__ __launch_bounds__(64) void wall_sum_kernel(const double *I_int, const double *weight,
                                                      const int64_t *wall_off, double *q)
{
    const int w = blockIdx.x;
    const int64_t r1 = wall_off[w + 1];
    double s = 0.0;
    for (int64_t r = wall_off[w] + threadIdx.x; r < r1; r += 64) s += weight[r] * I_int[r];
    for (int o = 32; o > 0; o >>= 1) s += __shfl_xor(s, o);
    if (threadIdx.x == 0) q[w] = s;
}

}  // namespace

hipError_t launch_march(bool fp32, bool linear, const MarchPlan &plan, const DevRays &rays, const DevGrid &g,
                        int32_t k_first, int32_t n_band, const void *eta, const void *kappa,
                        const int32_t *escale, const double *T_far, double *I_out,
                        double *partials, hipStream_t st)
{
    if (rays.n_rays == 0) return hipSuccess;
    const int64_t n_rays = rays.n_rays, cg = kMarchThreads / 64 / plan.rays;
    const int64_t n_blocks = (n_rays + plan.rays - 1) / plan.rays * ((plan.n_chunks + cg - 1) / cg);
    if (n_blocks > (int64_t)UINT32_MAX) return hipErrorInvalidConfiguration;
    for (int64_t b0 = 0; b0 < n_blocks; b0 += kMaxLaunchBlocks) {
        const dim3 grid((unsigned)std::min(kMaxLaunchBlocks, n_blocks - b0));
#define LRT_MARCH(F, LIN, P, R)                                                                            \
    hipLaunchKernelGGL((march_kernel<F, LIN, P, R>), grid, dim3(kMarchThreads), plan.lds, st, rays, g, k_first, \
                       n_band, eta, kappa, escale, T_far, I_out, partials, plan.n_chunks,                  \
                       plan.shared ? 1 : 0, (uint32_t)b0)
#define LRT_MARCH_P(F, LIN)                                                       \
    if (plan.ppt == 2 && plan.rays == 1) LRT_MARCH(F, LIN, 2, 1);                 \
    else if (plan.ppt == 2) LRT_MARCH(F, LIN, 2, 4);                              \
    else if (plan.rays == 1) LRT_MARCH(F, LIN, 4, 1); else LRT_MARCH(F, LIN, 4, 4)
        if (fp32) {
            if (linear) LRT_MARCH_P(true, true); else LRT_MARCH_P(true, false);
        } else {
            if (linear) LRT_MARCH_P(false, true); else LRT_MARCH_P(false, false);
        }
#undef LRT_MARCH_P
#undef LRT_MARCH
        const hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}

hipError_t launch_reduce_rows(const double *partials, int32_t n_rows, int32_t n_cols, double *out, double *acc,
                              bool first, double *acc_host, hipStream_t st)
{
    if (n_rows == 0) return hipSuccess;
    int32_t lg = 0;   // a wave per row, or as many lanes as a short row has columns
    while (lg < 6 && (1 << lg) < n_cols && ((int64_t)n_rows << lg) < (int64_t(1) << 30)) ++lg;
    hipLaunchKernelGGL(reduce_rows_kernel, dim3(blocks_for((int64_t)n_rows << lg, 256)), dim3(256), 0, st, partials,
                       n_rows, n_cols, lg, out, acc, first ? 1 : 0, acc_host);
    return hipGetLastError();
}

hipError_t launch_wall_sum(const double *I_int, const double *weight, const int64_t *wall_off,
                           int32_t n_wall, double *q, hipStream_t st)
{
    if (n_wall == 0) return hipSuccess;
    hipLaunchKernelGGL(wall_sum_kernel, dim3((unsigned)n_wall), dim3(64), 0, st, I_int, weight, wall_off, q);
    return hipGetLastError();
}

}  // namespace lrt
