// Auxiliary gfx950 kernels of the radiation library: the fixed-order FP64 folds of the
// accumulate kernels' FP32 partials, read-out (intensity and Cartesian spectrum), fills,
// the tracked-particle (post-processing) kernels and a transcendental probe.

#include <hip/hip_ext.h>
#include <hip/hip_runtime.h>
#include <math.h>
#include <stdint.h>

#include <algorithm>

#include "rad_device.h"
#include "rad_internal.h"

namespace rad {

namespace {

// ---------------------------------------------------------------------------------------
// Post-processing variant: tracked particles keep their own time integral
// T_m(n, omega) = sum_j A_{j,m}(n) exp(i omega tau_{j,m}) (no form factor) in FP64,
// layout [m][omega][dir][4]; the form factor is applied only when the spectrum is read.
//
// One workgroup of NT threads per (particle, tile of TD directions x OB blocks of
// W = kTrackW frequencies), OB = min(NT / W, smallest power of two >= the number of
// frequency blocks), TD = NT / OB.  The steps of a push are taken S = OB at a
// time: the S x TD (step, direction) geometries (FP64, as in the main path) are computed
// once, one per thread, into LDS, then every thread walks its W frequencies for each of the
// S steps with the main path's three-term walk from the block's middle frequency (or,
// for explicit frequency lists, the per-term FP64 phase).  The per-(step, direction) set-up is thus shared by OB * W
// frequencies.  Up to kStepGroup steps of one push are summed in FP32 registers before one
// read-modify-write of the FP64 integrals, so a multi-step push moves 64 B per particle and
// grid point per group instead of per step (the main path likewise sums hundreds of
// particles in FP32 per partial).  W = 8 (rather than 16) lets the kernel fit four
// waves per SIMD.
// ---------------------------------------------------------------------------------------
constexpr int kStepGroup = 128;
constexpr int kTrackW = 8;
// Workgroup sizes: 256 threads for multi-step pushes, 512 for one-step pushes (measured:
// 512 is 7 % faster on one-step pushes, whose workgroups mostly wait for their integrals,
// and 42 % slower on a 100-step push).
constexpr int kTrackThreads = 256;
constexpr int kTrackThreadsOneStep = 512;

struct TrackedTiling {
    int ob;     // frequency blocks per workgroup (also the steps per sub-chunk)
    int td;     // directions per workgroup
    int n_dt;   // direction tiles
    int n_ot;   // frequency tiles
};

__host__ __device__ inline TrackedTiling tracked_tiling(int n_dir, int n_omega, int nt)
{
    const int max_ob = nt / kTrackW;
    const int n_blocks = (n_omega + kTrackW - 1) / kTrackW;
    int ob = 1;
    while (ob < n_blocks && ob < max_ob) ob *= 2;
    TrackedTiling t;
    t.ob = ob;
    t.td = nt / ob;
    t.n_dt = (n_dir + t.td - 1) / t.td;
    t.n_ot = (n_blocks + ob - 1) / ob;
    return t;
}

// Waves per SIMD the tracked kernel is compiled for: four (at most 128 VGPRs).  It fits
// without spills because the read-modify-write of the integrals keeps only two 32-byte
// loads in flight per thread (eight needed 166 VGPRs, i.e. three waves per SIMD; the
// four-wave build is 6 % faster on 100-step pushes and 8 % on one-step pushes).  More
// waves let one workgroup's read-modify-write overlap another's arithmetic.
#ifndef RAD_TRACK_WAVES
#define RAD_TRACK_WAVES 4
#endif

template <typename InT, bool DIRECT, int NT>
__global__ void __launch_bounds__(NT, RAD_TRACK_WAVES) k_tracked_accumulate(TrackedArgs a)
{
    constexpr int W = kTrackW;
    constexpr int SMAX = NT / kTrackW;
    __shared__ double raw[11 * SMAX];            // [field][step] of the sub-chunk
    __shared__ float4 geo[NT];                   // [step][direction]: A1, A2, w
    __shared__ double tau[NT];                   // [step][direction]: tau / (2 pi)
    const TrackedTiling tl = tracked_tiling(a.n_dir, a.n_omega, NT);
    const int S = tl.ob, TD = tl.td;
    const int tid = threadIdx.x;
    int64_t b = blockIdx.x;
    const int dt = (int)(b % tl.n_dt);
    b /= tl.n_dt;
    const int ot = (int)(b % tl.n_ot);
    const int64_t m = b / tl.n_ot;               // grid: n_particles x n_ot x n_dt workgroups
    const int dl = tid % TD;
    const int d = dt * TD + dl;
    const int dg = d < a.n_dir ? d : a.n_dir - 1;
    const int n_blocks = (a.n_omega + W - 1) / W;
    const int ob = ot * tl.ob + tid / TD;         // this thread's frequency block
    const bool live = d < a.n_dir && ob < n_blocks;
    const int o0 = (ob < n_blocks ? ob : n_blocks - 1) * W;
    const int kmax = a.n_omega - o0 < W ? a.n_omega - o0 : W;
    constexpr int KS = W / 2;                     // seeded frequency of the block
    const double om_seed = a.omega[o0] + (double)KS * a.domega;
    double om[DIRECT ? W : 1];
    if constexpr (DIRECT) {
#pragma unroll
        for (int k = 0; k < W; ++k) om[k] = a.omega[o0 + (k < kmax ? k : kmax - 1)];
    }
    const int ss = tid / TD;                      // set-up role: step ss of the sub-chunk
    constexpr int G = 2;
    double4* T = reinterpret_cast<double4*>(a.T) + (m * a.n_omega + o0) * a.n_dir + d;
    for (int j0 = 0; j0 < a.n_steps; j0 += kStepGroup) {
        const int j1 = a.n_steps - j0 < kStepGroup ? a.n_steps : j0 + kStepGroup;
        float4 acc[W];
#pragma unroll
        for (int k = 0; k < W; ++k) acc[k] = make_float4(0.f, 0.f, 0.f, 0.f);
        for (int js = j0; js < j1; js += S) {
            const int ns = j1 - js < S ? j1 - js : S;
            // 1. the particle's states at the sub-chunk's steps (step-major SoA input)
            if (tid < ns) {
                const int64_t i = (int64_t)(js + tid) * a.n_particles + m;
#pragma unroll
                for (int f = 0; f < 9; ++f) raw[f * SMAX + tid] = load_wide<InT>(a.f[f], i);
                raw[9 * SMAX + tid] = 1.0;     // weights enter only at read-out
                raw[10 * SMAX + tid] = a.t + (double)(js + tid) * a.dt;
            }
            __syncthreads();
            // 2. one (step, direction) geometry per thread
            {
                float4 gv = make_float4(0.f, 0.f, 1.f, 0.f);
                double ph = 0.0;
                if (ss < ns)
                    particle_direction_setup<0, !DIRECT, SMAX>(raw, ss, a.dirs9 + 9 * dg, a.domega, gv, ph, a.err);
                geo[tid] = gv;
                tau[tid] = ph;
            }
            __syncthreads();
            // 3. W frequencies per step; raw is rewritten only after every thread has passed
            //    the barrier above, and geo/tau only after the next sub-chunk's first barrier
            for (int s = 0; s < ns; ++s) {
                const float4 gv = geo[s * TD + dl];
                const double ph = tau[s * TD + dl];
                // the three-term walk's sign factors sigma_k ride on A (nA = -A)
                float nA1 = 0.f, nA2 = 0.f;
                if constexpr (!DIRECT) {
                    nA1 = -gv.x;
                    nA2 = -gv.y;
                    asm volatile("" : "+v"(nA1), "+v"(nA2));
                }
                auto add = [&](int k, float xr, float xi) {
                    const float a1 = (!DIRECT && (k & 2)) ? nA1 : gv.x;
                    const float a2 = (!DIRECT && (k & 2)) ? nA2 : gv.y;
                    acc[k].x = fmaf(a1, xr, acc[k].x);
                    acc[k].y = fmaf(a1, xi, acc[k].y);
                    acc[k].z = fmaf(a2, xr, acc[k].z);
                    acc[k].w = fmaf(a2, xi, acc[k].w);
                };
                if constexpr (DIRECT) {
#pragma unroll
                    for (int k = 0; k < W; ++k) {
                        float zr, zi;
                        sincos_rev_fast(static_cast<float>(frac_rev(om[k] * ph)), zi, zr);
                        add(k, zr, zi);
                    }
                } else {
                    // the main path's three-term walk on y_k = sigma_k z_k, sigma = (+, +, -, -)
                    // by k mod 4, from the seed at frequency KS (a multiple of 4, so y_KS = z):
                    // forward from (y_KS, y_KS+1 = z w) by y_{k+1} = c_k y_k + y_{k-1}, backward
                    // from (y_KS, y_KS-1 = -c y_KS + y_KS+1) by y_{k-1} = c'_k y_k + y_{k+1};
                    // c = 2 Re(w), c_k = +c / -c and c'_k = -c / +c for even / odd k
                    static_assert(KS % 4 == 0, "the sign pattern assumes y_KS = y_KS+1 = +z");
                    float zr, zi;
                    sincos_rev_fast(static_cast<float>(frac_rev(om_seed * ph)), zi, zr);
                    const float wr = gv.z, wi = gv.w;
                    float pc = 2.f * wr, nc = -2.f * wr;
                    asm volatile("" : "+v"(pc), "+v"(nc));
                    float pr = zr, pi = zi;
                    float cr = fmaf(zr, wr, -(zi * wi)), ci = fmaf(zr, wi, zi * wr);
                    const float ybr = fmaf(nc, zr, cr), ybi = fmaf(nc, zi, ci);
                    add(KS, pr, pi);
                    add(KS + 1, cr, ci);
#pragma unroll
                    for (int k = KS + 1; k < W - 1; ++k) {
                        const float ck = (k & 1) ? nc : pc;
                        const float nr = fmaf(ck, cr, pr), ni = fmaf(ck, ci, pi);
                        pr = cr; pi = ci; cr = nr; ci = ni;
                        add(k + 1, cr, ci);
                    }
                    pr = zr; pi = zi;
                    cr = ybr; ci = ybi;
                    add(KS - 1, cr, ci);
#pragma unroll
                    for (int k = KS - 1; k > 0; --k) {
                        const float ck = (k & 1) ? pc : nc;
                        const float nr = fmaf(ck, cr, pr), ni = fmaf(ck, ci, pi);
                        pr = cr; pi = ci; cr = nr; ci = ni;
                        add(k - 1, cr, ci);
                    }
                }
            }
        }
        // 4. read-modify-write of the integrals, G loads in flight before their stores
        //    (consecutive threads hold consecutive directions: 32 B each, contiguous).  Known
        //    zeros are not read (the first push of 512 particles x 100 steps x 128 x 256 points 355
        //    -> 328 us, of one step of 256 particles x 64 x 256 43 -> 29).
        const bool zero = a.T_zero && j0 == 0;
        if (live) {
            // an opaque copy of the stride keeps the W addresses from being hoisted out of
            // the step-group loop (they would stay live through the hot loop)
            int64_t stride = a.n_dir;
            asm volatile("" : "+s"(stride));
#pragma unroll
            for (int q = 0; q < W; q += G) {
                double4 t[G];
#pragma unroll
                for (int u = 0; u < G; ++u) {
                    t[u] = make_double4(0.0, 0.0, 0.0, 0.0);
                    if (q + u < kmax && !zero) t[u] = T[(q + u) * stride];
                }
#pragma unroll
                for (int u = 0; u < G; ++u) {
                    const int k = q + u;
                    if (k < kmax) {
                        t[u].x += (double)acc[k].x;
                        t[u].y += (double)acc[k].y;
                        t[u].z += (double)acc[k].z;
                        t[u].w += (double)acc[k].w;
                        T[k * stride] = t[u];
                    }
                }
            }
        }
    }
}

// I[d][k] = C |sum_m F_m(d, k) T_m(k, d)|^2 with F_m = sqrt(N_m + (N_m^2 - N_m) g) in FP64;
// g from gk[k] (1-D shape) or g3[d][k] (3-D shape).
//
// Bound by the one read of T (32 B per particle and point).  A block of 256 threads is
// PT = 256 / G points x G groups of particles: one thread per point leaves most CUs idle
// (32768 points are 128 blocks) and walks all particles through one load at a time.  The
// groups' sums are added in group order through LDS, so the result is reproducible.
// 512 particles x 32768 points (537 MB): 268 us with one thread per point,
// 110 us (4.9 TB/s, the rate of a large copy) with 8 groups; 256 x 16384 points (134 MB):
// 72 us and 22 us with 32.
template <int G>
__global__ void __launch_bounds__(256) k_tracked_finalize(const double* __restrict__ T, const double* __restrict__ wts,
                                                          const double* __restrict__ gk, const double* __restrict__ g3,
                                                          int64_t n_particles, int n_dir, int n_omega, double C,
                                                          double* __restrict__ I, const int* err, int* flag_out)
{
    constexpr int PT = 256 / G;
    constexpr int U = 4;                          // particles in flight per thread
    __shared__ double red[G][4][PT];
    const int p = threadIdx.x % PT, q = threadIdx.x / PT;
    const int64_t points = (int64_t)n_dir * n_omega;
    // consecutive threads take consecutive directions, so the reads of T are contiguous
    const int64_t i = (int64_t)blockIdx.x * PT + p;
    const int64_t ic = i < points ? i : points - 1;
    const int k = (int)(ic / n_dir), d = (int)(ic % n_dir);
    const double g = g3 ? g3[(int64_t)d * n_omega + k] : gk[k];
    const int64_t per = (n_particles + G - 1) / G;
    const int64_t m0 = (int64_t)q * per;
    const int64_t m1 = m0 + per < n_particles ? m0 + per : n_particles;
    const double2* t = reinterpret_cast<const double2*>(T) + 2 * ic;
    double s0 = 0, s1 = 0, s2 = 0, s3 = 0;
    for (int64_t m = m0; m < m1; m += U) {
        double2 lo[U], hi[U];
        double N[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int64_t mu = m + u < m1 ? m + u : m1 - 1;
            lo[u] = t[2 * mu * points];
            hi[u] = t[2 * mu * points + 1];
            N[u] = wts[mu];
        }
#pragma unroll
        for (int u = 0; u < U; ++u) {
            if (m + u < m1) {
                const double F = sqrt(fmax(N[u] + (N[u] * N[u] - N[u]) * g, 0.0));
                s0 += F * lo[u].x; s1 += F * lo[u].y; s2 += F * hi[u].x; s3 += F * hi[u].y;
            }
        }
    }
    if constexpr (G > 1) {
        red[q][0][p] = s0; red[q][1][p] = s1; red[q][2][p] = s2; red[q][3][p] = s3;
        __syncthreads();
        if (q == 0) {
#pragma unroll
            for (int r = 1; r < G; ++r) {
                s0 += red[r][0][p]; s1 += red[r][1][p]; s2 += red[r][2][p]; s3 += red[r][3][p];
            }
        }
    }
    if (q == 0 && i < points) I[(int64_t)d * n_omega + k] = C * (s0 * s0 + s1 * s1 + s2 * s2 + s3 * s3);
    if (flag_out && blockIdx.x == 0 && threadIdx.x == 0) *flag_out = *err;
}

typedef float f32x4 __attribute__((ext_vector_type(4)));

// FP64 sum of the FP32 partials *at(k), k in [k0, k1), in order, with U 16-byte loads in
// flight; in the last round what is past the end is the last one again and not added.
template <int U, typename At>
__device__ __forceinline__ void fold_range(int k0, int k1, At at, double (&a)[4])
{
    auto add = [&](const f32x4& v) {
        a[0] += (double)v.x;
        a[1] += (double)v.y;
        a[2] += (double)v.z;
        a[3] += (double)v.w;
    };
    f32x4 v[U];
    int k = k0;
    for (; k + U <= k1; k += U) {
#pragma unroll
        for (int u = 0; u < U; ++u) v[u] = __builtin_nontemporal_load(at(k + u));
#pragma unroll
        for (int u = 0; u < U; ++u) add(v[u]);
    }
    if (k < k1) {
#pragma unroll
        for (int u = 0; u < U; ++u) v[u] = __builtin_nontemporal_load(at(k + u < k1 ? k + u : k1 - 1));
#pragma unroll
        for (int u = 0; u < U; ++u)
            if (k + u < k1) add(v[u]);
    }
}

// The G groups' sums of PT points, added in group order: thread t < 4 PT gets component
// t % 4 of point t / 4.
template <int G, int PT>
__device__ __forceinline__ double fold_groups(double (&red)[G][4 * PT], int p, int q, const double (&a)[4])
{
    static_assert(4 * PT <= 256, "one component per thread");
#pragma unroll
    for (int c = 0; c < 4; ++c) red[q][4 * p + c] = a[c];
    __syncthreads();
    double s = 0.0;
    const int t = threadIdx.x;
    if (t < 4 * PT) {
#pragma unroll
        for (int r = 0; r < G; ++r) s += red[r][t];
    }
    return s;
}

// S[p] += sum over splits of part[s][p] for every grid point p (four components: S1r,
// S1i, S2r, S2i) in FP64, in a fixed order; times `scale` from point `scale_from` on.  Bound by the one read of the partials (16 B
// per split and point, non-temporal), and on small grids by the latency of that read: a
// block of 256 threads is PT = 256 / G points x G groups of consecutive splits, with
// kFoldUnroll loads in flight per thread (twice that without groups), so that a grid of a
// few hundred points is not one serial chain of loads.  The groups' sums are added in group
// order through LDS.  157 splits x 3700 points (9.3 MB): 16.5 us with one thread per point,
// 6.0 us with 16 groups; 63 splits x 482 points: 10.9 and 4.3 us; 128 splits x 32768 points
// (67 MB): 12.7 us (5.3 TB/s) without groups.
constexpr int kFoldUnroll = 8;

template <int G>
__global__ void __launch_bounds__(256) k_fold(const f32x4* __restrict__ part, double* __restrict__ S,
                                              int splits, int64_t points, double scale, int64_t scale_from)
{
    constexpr int PT = 256 / G;
    const int p = threadIdx.x % PT, q = threadIdx.x / PT;
    const int64_t i0 = (int64_t)blockIdx.x * PT;
    const int64_t i = i0 + p < points ? i0 + p : points - 1;
    const int per = (splits + G - 1) / G;
    const int k0 = q * per, k1 = k0 + per < splits ? k0 + per : splits;
    double a[4] = {0.0, 0.0, 0.0, 0.0};
    fold_range<G == 1 ? 2 * kFoldUnroll : kFoldUnroll>(k0, k1, [&](int k) { return part + (int64_t)k * points + i; }, a);
    if constexpr (G == 1) {
        if (i0 + p < points) {
            double2* s2 = reinterpret_cast<double2*>(S) + 2 * i;
            double2 lo = s2[0], hi = s2[1];
            const double f = i < scale_from ? 1.0 : scale;
            lo.x += f * a[0]; lo.y += f * a[1]; hi.x += f * a[2]; hi.y += f * a[3];
            s2[0] = lo;
            s2[1] = hi;
        }
    } else {
        __shared__ double red[G][4 * PT];
        const double s = fold_groups<G, PT>(red, p, q, a);
        const int t = threadIdx.x;
        if (t < 4 * PT && 4 * i0 + t < 4 * points) S[4 * i0 + t] += (i0 + t / 4 < scale_from ? 1.0 : scale) * s;
    }
}

// Batched fold: for every (grid, tile) job and every in-grid point of the tile, add the
// listed segments' partial values (in list order within a group, then in group order, FP64)
// into the grid's S.  As k_fold: PT elements of a tile x G groups of the job's list; the
// lists are as uneven as the bunches (1 to several hundred segments), so the groups also
// shorten the longest one.  12 bunches, 64 x 256 points each, 1024 ranges (137 MB): 73 us
// with one thread per element and one load in flight, 26.5 us (5.2 TB/s) here.
constexpr int kBatchFoldGroups = 8;
constexpr int kBatchFoldPoints = 256 / kBatchFoldGroups;

__global__ void __launch_bounds__(256) k_fold_batch(const int32_t* __restrict__ n_jobs_dev,
                                                    const FoldJob* __restrict__ jobs,
                                                    const int32_t* __restrict__ seg_list,
                                                    const f32x4* __restrict__ seg_part, int TD, int TO)
{
    constexpr int G = kBatchFoldGroups, PT = kBatchFoldPoints;
    __shared__ double red[G][4 * PT];
    const int n_jobs = *n_jobs_dev;
    const int per_job = TD * TO;                  // a multiple of 64
    const int blocks_per_job = per_job / PT;
    const int64_t total = (int64_t)blocks_per_job * n_jobs;
    const int p = threadIdx.x % PT, q = threadIdx.x / PT;
    for (int64_t blk = blockIdx.x; blk < total; blk += gridDim.x) {
        const FoldJob fj = jobs[blk / blocks_per_job];
        const int e0 = (int)(blk % blocks_per_job) * PT;
        const int n = fj.list_end - fj.list_begin;
        const int per = (n + G - 1) / G;
        const int k0 = fj.list_begin + q * per;
        const int k1 = k0 + per < fj.list_end ? k0 + per : fj.list_end;
        double a[4] = {0.0, 0.0, 0.0, 0.0};
        fold_range<kFoldUnroll>(k0, k1, [&](int k) { return seg_part + (int64_t)seg_list[k] * per_job + e0 + p; }, a);
        const double s = fold_groups<G, PT>(red, p, q, a);
        const int t = threadIdx.x, e = e0 + t / 4;
        const int og = fj.tw * TO + e / TD, dg = fj.td * TD + e % TD;
        if (t < 4 * PT && og < fj.n_omega && dg < fj.n_dir) fj.S[((int64_t)og * fj.n_dir + dg) * 4 + t % 4] += s;
        __syncthreads();
    }
}

// Read-out kernels: a block of 256 threads takes td x tk (direction, frequency) points, one per
// thread.  S is [omega][dir] and the results are [dir][omega], so the points are read with
// consecutive threads on consecutive directions (512 B a row of 16) and written through LDS with
// consecutive threads on consecutive frequencies: full lines also where the result is
// page-locked host memory.  16 x 16 points, and on grids of fewer directions or frequencies the
// power of two that holds them (out_tile): in 16 x 16 a single direction would leave 15 of 16
// threads idle (1 x 1048576 points, device read-outs one after another: 26.6 us each, 6.8 here;
// 1048576 x 1: 30.5 and 7.0).
struct OutTile {
    int ld, lk;    // log2 of its directions and frequencies, 8 together
};

OutTile out_tile(int n_dir, int n_omega)
{
    auto log2_of = [](int n) {      // of the power of two that holds n, at most 16
        int l = 0;
        while (l < 4 && (1 << l) < n) ++l;
        return l;
    };
    const int ld = log2_of(n_dir), lk = log2_of(n_omega);
    return ld < 4 ? OutTile{ld, 8 - ld} : OutTile{8 - lk, lk};
}

struct OutPoint {
    int d, k;      // the thread's point when reading S: consecutive directions
    bool in;
    int d0, k0;    // the block's first point
};

__device__ __forceinline__ OutPoint out_point(OutTile tl, int n_dir, int n_omega)
{
    const int tiles_k = (int)((n_omega + (1u << tl.lk) - 1) >> tl.lk);
    OutPoint o;
    o.d0 = (int)(blockIdx.x / tiles_k) << tl.ld;
    o.k0 = (int)(blockIdx.x % tiles_k) << tl.lk;
    o.d = o.d0 + (threadIdx.x & ((1 << tl.ld) - 1));
    o.k = o.k0 + (threadIdx.x >> tl.ld);
    o.in = o.d < n_dir && o.k < n_omega;
    return o;
}

// I[d][k] = C * (|S1|^2 + |S2|^2), S layout [omega][dir][4].
__global__ void __launch_bounds__(256) k_finalize(const double* __restrict__ S, double* __restrict__ I, OutTile tl,
                                                  int n_dir, int n_omega, double C, const int* err, int* flag_out)
{
    __shared__ double tile[2 * 256];              // [frequency][td + 1]
    const OutPoint o = out_point(tl, n_dir, n_omega);
    const int row = (1 << tl.ld) + 1;
    if (o.in) {
        const double2* s = reinterpret_cast<const double2*>(S) + 2 * ((int64_t)o.k * n_dir + o.d);
        const double2 a = s[0], b = s[1];
        tile[(o.k - o.k0) * row + o.d - o.d0] = C * (a.x * a.x + a.y * a.y + b.x * b.x + b.y * b.y);
    }
    __syncthreads();
    const int kl = threadIdx.x & ((1 << tl.lk) - 1), dl = threadIdx.x >> tl.lk;
    const int k = o.k0 + kl, d = o.d0 + dl;
    if (d < n_dir && k < n_omega) I[(int64_t)d * n_omega + k] = tile[kl * row + dl];
    if (flag_out && blockIdx.x == 0 && threadIdx.x == 0) *flag_out = *err;
}

// Cartesian complex spectrum out[((d*n_omega + k)*3 + c)*2 + {re, im}] = e1_c S1 + e2_c S2.
__global__ void __launch_bounds__(256) k_cartesian(const double* __restrict__ S, const double* __restrict__ dirs9,
                                                   double* __restrict__ out, OutTile tl, int n_dir, int n_omega,
                                                   const int* err, int* flag_out)
{
    __shared__ double tile[(6 + 1) * 256];        // [direction][6 tk + 1]
    const OutPoint o = out_point(tl, n_dir, n_omega);
    const int row = (6 << tl.lk) + 1;
    if (o.in) {
        const double2* s = reinterpret_cast<const double2*>(S) + 2 * ((int64_t)o.k * n_dir + o.d);
        const double2 a = s[0], b = s[1];
        const double* e = dirs9 + 9 * o.d;
        double* v = tile + (o.d - o.d0) * row + 6 * (o.k - o.k0);
#pragma unroll
        for (int c = 0; c < 3; ++c) {
            v[2 * c + 0] = e[3 + c] * a.x + e[6 + c] * b.x;
            v[2 * c + 1] = e[3 + c] * a.y + e[6 + c] * b.y;
        }
    }
    __syncthreads();
    const int live = 6 * (n_omega - o.k0 < (1 << tl.lk) ? n_omega - o.k0 : 1 << tl.lk);
    for (int i = threadIdx.x; i < 6 * 256; i += 256) {
        const int dl = i / 6 >> tl.lk, r = i - dl * (row - 1), d = o.d0 + dl;
        if (d < n_dir && r < live) out[((int64_t)d * n_omega + o.k0) * 6 + r] = tile[dl * row + r];
    }
    if (flag_out && blockIdx.x == 0 && threadIdx.x == 0) *flag_out = *err;
}

// Zeroes n2 pairs of doubles and the error flag in one launch (the flag's own launch cost a
// reset another 2 to 5 us on the GPU).
__global__ void __launch_bounds__(256) k_reset(double2* p, int64_t n2, int* err)
{
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n2) p[i] = make_double2(0.0, 0.0);
    if (i == 0) *err = 0;
}

// out[4i..4i+3] = hardware sin/cos and library sin/cos of 2*pi*in[i].
__global__ void k_trig_probe(const float* in, float* out, int n)
{
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    float s, c, s2, c2;
    sincos_rev_fast(in[i], s, c);
    sincos_rev_accurate(in[i], s2, c2);
    out[4 * i + 0] = s;
    out[4 * i + 1] = c;
    out[4 * i + 2] = s2;
    out[4 * i + 3] = c2;
}

inline unsigned grid1d(int64_t n, int bs) { return (unsigned)((n + bs - 1) / bs); }

}  // namespace

hipError_t launch_fold_batch(const int32_t* n_jobs_dev, const FoldJob* jobs, int max_jobs,
                             const int32_t* seg_list, const float* seg_part, int td, int to, hipStream_t st)
{
    if (max_jobs <= 0) return hipSuccess;
    const int64_t total = (int64_t)max_jobs * td * to / kBatchFoldPoints;
    const int blocks = (int)std::min<int64_t>(total, 16384);
    hipLaunchKernelGGL(k_fold_batch, dim3(blocks), dim3(256), 0, st, n_jobs_dev, jobs, seg_list,
                       reinterpret_cast<const f32x4*>(seg_part), td, to);
    return hipGetLastError();
}

namespace {

template <int G>
hipError_t launch_fold_g(const f32x4* part, double* S, int splits, int64_t points, double scale, int64_t scale_from,
                         hipStream_t st, hipEvent_t ev_start, hipEvent_t ev_stop)
{
    const dim3 grid(grid1d(points, 256 / G));
    if (ev_start || ev_stop) {
        void* args[] = {&part, &S, &splits, &points, &scale, &scale_from};
        return hipExtLaunchKernel(reinterpret_cast<const void*>(k_fold<G>), grid, dim3(256), args, 0, st, ev_start,
                                  ev_stop, 0);
    }
    hipLaunchKernelGGL(k_fold<G>, grid, dim3(256), 0, st, part, S, splits, points, scale, scale_from);
    return hipGetLastError();
}

}  // namespace

hipError_t launch_fold(const float* part, double* S, int splits, int64_t count, double scale, int64_t scale_from,
                       hipStream_t st, hipEvent_t ev_start, hipEvent_t ev_stop)
{
    const int64_t points = count / 4;
    if (points <= 0) return hipSuccess;
    const f32x4* p4 = reinterpret_cast<const f32x4*>(part);
    auto go = [&](auto fold) { return fold(p4, S, splits, points, scale, scale_from, st, ev_start, ev_stop); };
    // Groups of splits per block.  From 32768 points on, one thread per point with 16 loads
    // in flight already reads at the rate HBM delivers (128 splits x 32768 points 12.7 us, 4
    // groups 12.8; 256 splits 20.9 against 21.7; 65536 points 12.2 against 13.0).  Below, its
    // blocks are too few: 3700 points 16.5 us against 6.0 with 16 groups.  Groups are of one
    // length, so the last of them may be empty (17 splits are 8 groups of two, one of one and
    // seven of none); an empty group adds zeros.
    if (points >= 32768 || splits < 4) return go(launch_fold_g<1>);
    if (points >= 8192 || splits < 16) return go(launch_fold_g<4>);
    return go(launch_fold_g<16>);
}

namespace {

unsigned out_blocks(OutTile tl, int n_dir, int n_omega)
{
    return grid1d(n_dir, 1 << tl.ld) * grid1d(n_omega, 1 << tl.lk);
}

}  // namespace

hipError_t launch_finalize(const double* S, double* I, int n_dir, int n_omega, double C, const int* err,
                           int* flag_out, hipStream_t st)
{
    const OutTile tl = out_tile(n_dir, n_omega);
    hipLaunchKernelGGL(k_finalize, dim3(out_blocks(tl, n_dir, n_omega)), dim3(256), 0, st, S, I, tl, n_dir, n_omega, C,
                       err, flag_out);
    return hipGetLastError();
}

hipError_t launch_cartesian(const double* S, const double* dirs9, double* out, int n_dir, int n_omega, const int* err,
                            int* flag_out, hipStream_t st)
{
    const OutTile tl = out_tile(n_dir, n_omega);
    hipLaunchKernelGGL(k_cartesian, dim3(out_blocks(tl, n_dir, n_omega)), dim3(256), 0, st, S, dirs9, out, tl, n_dir,
                       n_omega, err, flag_out);
    return hipGetLastError();
}

hipError_t launch_reset(double* p, int64_t n, int* err, hipStream_t st)
{
    hipLaunchKernelGGL(k_reset, dim3(std::max(1u, grid1d(n / 2, 256))), dim3(256), 0, st,
                       reinterpret_cast<double2*>(p), n / 2, err);
    return hipGetLastError();
}

int tracked_step_group() { return kStepGroup; }

template <int NT>
hipError_t launch_tracked_nt(const TrackedArgs& a, int dtype, bool direct, hipStream_t st)
{
    const TrackedTiling tl = tracked_tiling(a.n_dir, a.n_omega, NT);
    const int64_t blocks = a.n_particles * tl.n_dt * tl.n_ot;
    if (blocks > 0x7fffffff) return hipErrorInvalidConfiguration;
    const dim3 grid((unsigned)blocks);
    const dim3 block(NT);
    if (dtype == 0) {
        if (direct) hipLaunchKernelGGL((k_tracked_accumulate<float, true, NT>), grid, block, 0, st, a);
        else hipLaunchKernelGGL((k_tracked_accumulate<float, false, NT>), grid, block, 0, st, a);
    } else {
        if (direct) hipLaunchKernelGGL((k_tracked_accumulate<double, true, NT>), grid, block, 0, st, a);
        else hipLaunchKernelGGL((k_tracked_accumulate<double, false, NT>), grid, block, 0, st, a);
    }
    return hipGetLastError();
}

hipError_t launch_tracked_accumulate(const TrackedArgs& a, int dtype, bool direct, hipStream_t st)
{
    if (a.n_particles <= 0 || a.n_steps <= 0 || a.n_dir <= 0 || a.n_omega <= 0) return hipSuccess;
    return a.n_steps == 1 ? launch_tracked_nt<kTrackThreadsOneStep>(a, dtype, direct, st)
                          : launch_tracked_nt<kTrackThreads>(a, dtype, direct, st);
}

hipError_t launch_tracked_finalize(const double* T, const double* wts, const double* gk, const double* g3,
                                   int64_t n_particles, int n_dir, int n_omega, double C, double* I, const int* err,
                                   int* flag_out, hipStream_t st)
{
    const int64_t points = (int64_t)n_dir * n_omega;
    auto go = [&](auto kern, int groups) {
        hipLaunchKernelGGL(kern, dim3(grid1d(points, 256 / groups)), dim3(256), 0, st, T, wts, gk, g3, n_particles,
                           n_dir, n_omega, C, I, err, flag_out);
        return hipGetLastError();
    };
    // Groups of particles per block: as few as give the chip 4096 waves (16 per CU).
    if (points >= 262144 || n_particles < 8) return go(k_tracked_finalize<1>, 1);
    if (points >= 32768 || n_particles < 64) return go(k_tracked_finalize<8>, 8);
    return go(k_tracked_finalize<32>, 32);
}

hipError_t launch_trig_probe(const float* in, float* out, int n, hipStream_t st)
{
    if (n <= 0) return hipSuccess;
    hipLaunchKernelGGL(k_trig_probe, dim3(grid1d(n, 256)), dim3(256), 0, st, in, out, n);
    return hipGetLastError();
}

}  // namespace rad
