// Matrix-core accumulate kernel for the frequencies of a uniform grid over which the 1-D shape
// factor g is one constant (a point shape everywhere; a Gaussian wherever it has underflowed
// to zero, which is all but the first few frequencies of a wide grid).
//
// There the weight F_m of a macro-particle does not depend on the frequency, so with
// omega_k = Omega_q + j domega (k = 16 q + j) the sum over particles
//     S(n, k) = sum_m [F_m A_m(n) exp(i j domega tau_m)] exp(i Omega_q tau_m)
// is, for each direction, a matrix product over the particles: rows (q, re/im), columns
// (j, re/im) for each of the two polarizations.  The general kernel spends 8 VALU operations on
// each term; here a term's 8 multiply-adds are the matrix cores', and the VALU only forms the
// factors: 32 row and 64 column values per particle for 256 frequencies.
//
// * Factors.  Each is sin or cos of an FP64 phase, reduced to [0, 1) revolutions before it
//   leaves FP64 (cos as sin a quarter revolution on); nothing is walked.  The columns carry
//   F A in FP32.
// * FP32 product on f16 matrix cores.  Each FP32 factor is split into two f16 parts (11 + 11
//   bits and their signs), and the products of parts low high, high low and high high are
//   summed in FP32.  The columns are held to below 2^15 by a power of two for each 64 particles
//   and polarization, so that every magnitude fits f16 and the low parts of columns far below
//   the largest are not lost in its denormals (held to below 1, the error of a bunch's spectrum
//   was 1.2 times this).  The FP32 matrix instructions take 16 cycles for 64 terms and add to the
//   VALU's time; the f16 ones take 3.75 cycles of it and run beside the rest.
// * Sums.  A matrix instruction works in passes of 8 products, and within a pass it cuts every
//   product toward zero at 2^-24 of the largest term, the accumulator included: added to a
//   long sum, each product would lose a part of itself that grows with the sum (measured: 16
//   times the general kernel's error where the sums cancel, and a shrink of the order of 1e-5
//   where they are coherent).  So each 16 particles' products are summed from zero, the small
//   ones first, and the VALU adds the result to the FP32 sums, one rounding for 16
//   particles.  The accumulator itself is cut toward minus infinity; the columns change sign
//   from one 16 particles to the next, and the first ones from split to split, which turns
//   that into noise (with one sign for each 64 particles, splits of 32 to 64 had all the same,
//   and pushes of 3e4 particles twice the error).
// * The hardware sine is cut toward zero in its last bit: 3.2e-8 of it is missing on average,
//   twice in each term, and some 4e-9 more by the cuts of the products.  The fold scales this
//   kernel's sums back (kMxScale).  Its own error is then the rounding of two phases to 24 bits
//   and of two sines.
// * Error of S against FP64.  Root mean square per frequency, over 100 pushes drawn from point
//   and Gaussian grids of 1 to 128 directions and 100 to 1024 frequencies, three bunches each:
//   0.46 to 0.98 of the general kernel's, geometric mean 0.54; the largest of a frequency 0.46 in
//   the mean, 1.01 at most.  16384 particles x 256 steps whose sums cancel 1.4e-5 there and 2.9e-6
//   here; 60000 x 4 coherent terms 1.1e-7 and 8e-8; identical particles 3.6e-6 and 1.7e-7.
// * A wave owns one direction and RG x 256 frequencies, and shares nothing with other waves:
//   64 particles at a time, each lane computes one particle's geometry (FP64, as in the general
//   kernel) into the wave's own LDS, then four steps of 16 particles.  A row group's
//   matrix products run while the VALU forms the next one's rows.  Consecutive waves take
//   consecutive directions, so that their 16-byte partial sums fill lines.
// * Head.  A wide grid's Gaussian differs from its constant at the first frequency or two only.
//   Up to kMxHead of them are summed apart, each lane over its particles (weight, FP64 phase and
//   two complex multiply-adds per particle and frequency, kept in LDS), and replace the
//   matrix product's values there: a launch of the general kernel over a block of 16 for
//   the first of 1024 frequencies costs 570 us (16384 particles x 32 steps x 64 directions),
//   nearly a quarter of the 2430 for all of them this way.
// * Bound by the VALU: per 16 particles about 400 cycles for the columns and, for each 256
//   frequencies, 240 for the rows, 90 for the sums and 20 for each of the 6 matrix
//   instructions.  200000 particles x 64 directions: 512 frequencies 1.2e13 terms/s (550 us),
//   768 1.3e13, 1024 1.4e13; 128 x 256 8.8e12; the general kernel's walk 4.3e12 to 5.3e12.  Two
//   waves per SIMD are enough (with three, two row groups spill: 570 us).
#include <hip/hip_ext.h>
#include <hip/hip_runtime.h>
#include <math.h>
#include <stdint.h>

#include "rad_device.h"
#include "rad_internal.h"

namespace rad {

namespace {

typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef _Float16 f16x2 __attribute__((ext_vector_type(2)));
typedef _Float16 f16x8 __attribute__((ext_vector_type(8)));
typedef float f32x2 __attribute__((ext_vector_type(2)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));

constexpr int kMxThreads = 256;
// A particle as the matrix loop needs it: tau / (2 pi) and F A in the two polarizations.
struct __align__(16) MxParticle {
    double ph;
    float a1, a2;
};

// Two FP32 values as pairs of f16 parts (packed, first value in the low half), high + low.
__device__ __forceinline__ void split_pair(float v0, float v1, uint32_t& hi, uint32_t& lo)
{
    const f16x2 h = __builtin_convertvector((f32x2{v0, v1}), f16x2);
    const f32x2 r = {v0 - static_cast<float>(h.x), v1 - static_cast<float>(h.y)};
    hi = __builtin_bit_cast(uint32_t, h);
    lo = __builtin_bit_cast(uint32_t, __builtin_convertvector(r, f16x2));
}

// The largest of 64 lanes' values, in a scalar register.
template <int CTRL>
__device__ __forceinline__ uint32_t max_with(uint32_t v)
{
    const uint32_t o = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, CTRL, 0xf, 0xf, false);
    return o > v ? o : v;
}

__device__ __forceinline__ uint32_t wave_max(uint32_t v)
{
    v = max_with<0x111>(v);                                 // row_shr 1, 2, 4, 8: of each 16 lanes
    v = max_with<0x112>(v);
    v = max_with<0x114>(v);
    v = max_with<0x118>(v);
    v = max_with<0x142>(v);                                 // row_bcast 15 and 31: across rows
    v = max_with<0x143>(v);
    return (uint32_t)__builtin_amdgcn_readlane((int)v, 63);
}

// The largest column is scaled to just below 2^15, near the top of f16's range: its low part and
// smaller columns lie above f16's denormals then (scaled to 1, a column 2^-10 of the largest kept 14 bits).
constexpr int kColumnBits = 15;

// The exponent of the power of two just above |a| of all lanes, at least that of the smallest
// columns' scale (a scalar).
__device__ __forceinline__ int wave_exponent(float a)
{
    const int e = (int)(wave_max(__builtin_bit_cast(uint32_t, a) & 0x7fffffffu) >> 23) - 126;
    return e < kColumnBits - 126 ? kColumnBits - 126 : e;
}

// The FP32 bits of 2^e, e from -126.
__device__ __forceinline__ uint32_t power_bits(int e) { return (uint32_t)(e + 127) << 23; }

// sin of 2 pi (om ph + quarter), the phase reduced in FP64.
__device__ __forceinline__ float phase_sin(double om, double ph, double quarter)
{
    return __builtin_amdgcn_sinf(static_cast<float>(frac_rev(fma(om, ph, quarter))));
}

// Orders this wave's LDS writes before its later reads of other lanes' values.
__device__ __forceinline__ void wave_lds_sync()
{
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

constexpr int mx_waves(int RG) { return RG == 1 ? 4 : 2; }

template <typename InT, int RG>
__global__ void __launch_bounds__(kMxThreads, mx_waves(RG)) k_accumulate_mx(MxArgs a)
{
    __shared__ MxParticle buf_all[kMxThreads];
    extern __shared__ float4 head_all[];                   // [head][threads]
    const Job& j = a.job;
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    MxParticle* buf = buf_all + 64 * wave;
    // this wave's direction, frequency group and particle split
    const int id = (int)blockIdx.x * (kMxThreads / 64) + wave;
    if (id >= a.splits * a.fgroups * j.n_dir) return;      // no barriers below
    const int d = id % j.n_dir, fg = id / j.n_dir % a.fgroups, split = id / j.n_dir / a.fgroups;
    const int64_t p_begin = j.i_begin + (int64_t)split * a.per_split;
    const int64_t p_end = p_begin + a.per_split < j.i_end ? p_begin + a.per_split : j.i_end;

    const int r = lane & 31, half = lane >> 5;
    double om_row[RG];
#pragma unroll
    for (int g = 0; g < RG; ++g) {
        const int k = a.k0 + ((fg * RG + g) * 16 + (r >> 1)) * 16;
        om_row[g] = gload(j.omega, k < j.n_omega ? k : j.n_omega - 1);
    }
    const double quarter_row = (r & 1) ? 0.0 : 0.25;        // even rows cos, odd rows sin
    const double om_col = (double)(r & 15) * j.domega;
    const double quarter_col = r < 16 ? 0.25 : 0.0;         // columns 0..15 cos, 16..31 sin

    const int head = fg == 0 ? a.head : 0;
    float4* hsum = head_all + threadIdx.x;
    for (int k = 0; k < head; ++k) hsum[k * kMxThreads] = make_float4(0.f, 0.f, 0.f, 0.f);

    f32x16 acc[RG][2];
#pragma unroll
    for (int g = 0; g < RG; ++g) {
#pragma unroll
        for (int i = 0; i < 16; ++i) acc[g][0][i] = acc[g][1][i] = 0.f;
    }

    // the next 64 particles' fields are loaded while this 64's products run
    InT f[10];
    auto load = [&](int64_t p0) {
        const int64_t i = p0 + lane < p_end ? p0 + lane : p_end - 1;
#pragma unroll
        for (int c = 0; c < 10; ++c) f[c] = gload(static_cast<const InT*>(j.f[c]), i);
    };
    if (p_begin < p_end) load(p_begin);
    uint32_t turn = (uint32_t)split << 31;                 // sign of the first 16 particles' columns
    for (int64_t p0 = p_begin; p0 < p_end; p0 += 64) {
        const int cnt = p_end - p0 < 64 ? (int)(p_end - p0) : 64;
        uint32_t up[2];                                    // what undoes the columns' sign and scale, FP32 bits
        {
            const int64_t i = p0 + lane < p_end ? p0 + lane : p_end - 1;
            const double t = step_time(j, i);
            float4 geo;
            double ph;
            particle_direction_geometry<0, false>((double)f[0], (double)f[1], (double)f[2], (double)f[3], (double)f[4],
                                                  (double)f[5], (double)f[6], (double)f[7], (double)f[8], (double)f[9],
                                                  t, j.dirs9 + 9 * d, 0.0, geo, ph, j.err);
            const float N = (float)f[9];
            const float F = __builtin_amdgcn_sqrtf(fmaf(N * N, a.g, N * a.g1));
            const bool ok = lane < cnt;
            MxParticle e;
            e.ph = ok ? ph : 0.0;
            const float sign = __builtin_bit_cast(float, 0x3f800000u ^ turn ^ (uint32_t)(lane & 16) << 27);
            e.a1 = ok ? sign * (F * geo.x) : 0.f;
            e.a2 = ok ? sign * (F * geo.y) : 0.f;
            const int x1 = wave_exponent(e.a1), x2 = wave_exponent(e.a2);
            e.a1 = ldexpf(e.a1, kColumnBits - x1);
            e.a2 = ldexpf(e.a2, kColumnBits - x2);
            up[0] = power_bits(x1 - kColumnBits) | turn;
            up[1] = power_bits(x2 - kColumnBits) | turn;
            turn ^= 0x80000000u;
            for (int k = 0; k < head; ++k) {
                const float g0 = gload(reinterpret_cast<const float*>(j.gtab), 2 * (int64_t)k);
                const float g1 = gload(reinterpret_cast<const float*>(j.gtab), 2 * (int64_t)k + 1);
                const float Fk = ok ? __builtin_amdgcn_sqrtf(fmaf(N * N, g0, N * g1)) : 0.f;
                float zr, zi;
                sincos_rev_fast(static_cast<float>(frac_rev(gload(j.omega, k) * ph)), zi, zr);
                const float ur = Fk * zr, ui = Fk * zi;
                float4 v = hsum[k * kMxThreads];
                v.x = fmaf(geo.x, ur, v.x);
                v.y = fmaf(geo.x, ui, v.y);
                v.z = fmaf(geo.y, ur, v.z);
                v.w = fmaf(geo.y, ui, v.w);
                hsum[k * kMxThreads] = v;
            }
            wave_lds_sync();                               // the last 64's reads are done
            buf[lane] = e;
        }
        if (p0 + 64 < p_end) load(p0 + 64);
        wave_lds_sync();
        for (int s = 0; s < cnt; s += 16) {
            const MxParticle* e = buf + s + 8 * half;      // this half wave's 8 of 16 particles
            uint32_t col[2][2][4];                         // [polarization][high, low]
#pragma unroll
            for (int i = 0; i < 8; i += 2) {
                const MxParticle e0 = e[i], e1 = e[i + 1];
                const float c0 = phase_sin(om_col, e0.ph, quarter_col), c1 = phase_sin(om_col, e1.ph, quarter_col);
                split_pair(e0.a1 * c0, e1.a1 * c1, col[0][0][i / 2], col[0][1][i / 2]);
                split_pair(e0.a2 * c0, e1.a2 * c1, col[1][0][i / 2], col[1][1][i / 2]);
            }
            f32x16 sum[2];
            auto add = [&](int g) {
#pragma unroll
                for (int pol = 0; pol < 2; ++pol) {
#pragma unroll
                    for (int i = 0; i < 16; ++i) acc[g][pol][i] = fmaf(sum[pol][i], __builtin_bit_cast(float, up[pol]), acc[g][pol][i]);
                }
            };
#pragma unroll
            for (int g = 0; g < RG; ++g) {
                uint32_t row[2][4];
#pragma unroll
                for (int i = 0; i < 8; i += 2)
                    split_pair(phase_sin(om_row[g], e[i].ph, quarter_row), phase_sin(om_row[g], e[i + 1].ph, quarter_row),
                               row[0][i / 2], row[1][i / 2]);
                if (g > 0) add(g - 1);
                f32x16 zero;
#pragma unroll
                for (int i = 0; i < 16; ++i) zero[i] = 0.f;
#pragma unroll
                for (int part = 0; part < 3; ++part) {     // low high, high low, high high
#pragma unroll
                    for (int pol = 0; pol < 2; ++pol) {
                        const uint32_t(&rp)[4] = row[part == 0];
                        const uint32_t(&cp)[4] = col[pol][part == 1];
                        const u32x4 rw = {rp[0], rp[1], rp[2], rp[3]}, cw = {cp[0], cp[1], cp[2], cp[3]};
                        sum[pol] = __builtin_amdgcn_mfma_f32_32x32x16_f16(__builtin_bit_cast(f16x8, rw),
                                                                          __builtin_bit_cast(f16x8, cw),
                                                                          part == 0 ? zero : sum[pol], 0, 0, 0);
                    }
                }
            }
            add(RG - 1);
            up[0] ^= 0x80000000u;                          // the next 16 columns' sign
            up[1] ^= 0x80000000u;
        }
    }

    // Accumulator i of a lane is row 8 (i / 4) + 4 half + i % 4, column r: rows 2q (cos) and
    // 2q + 1 (sin) are neighbours, and column r ^ 16 is the other of (cos, sin) of the same j.
    // S_re = [cos cos] - [sin sin], S_im = [cos sin] + [sin cos]: one exchange gives the cos
    // columns' lanes S_re and the sin columns' S_im, a second one whole points: of each two q
    // the first to the cos column's lane, the second to the sin column's.
    const bool is_cos = r < 16;
    float4* out = reinterpret_cast<float4*>(a.part) + (int64_t)split * a.n_sub * j.n_dir + d;
#pragma unroll
    for (int g = 0; g < RG; ++g) {
#pragma unroll
        for (int i = 0; i < 16; i += 4) {
            float sv[2][2];                                // [q, q + 1][polarization]
#pragma unroll
            for (int u = 0; u < 2; ++u) {
#pragma unroll
                for (int pol = 0; pol < 2; ++pol) {
                    const float other = __shfl_xor(acc[g][pol][i + 2 * u + 1], 16);
                    sv[u][pol] = is_cos ? acc[g][pol][i + 2 * u] - other : acc[g][pol][i + 2 * u] + other;
                }
            }
            const float t0 = __shfl_xor(is_cos ? sv[1][0] : sv[0][0], 16);
            const float t1 = __shfl_xor(is_cos ? sv[1][1] : sv[0][1], 16);
            const float4 v = is_cos ? make_float4(sv[0][0], t0, sv[0][1], t1) : make_float4(t0, sv[1][0], t1, sv[1][1]);
            const int q = 4 * (i / 4) + 2 * half + (is_cos ? 0 : 1);
            const int k = ((fg * RG + g) * 16 + q) * 16 + (r & 15);
            if (k < a.n_sub && k >= head) out[(int64_t)k * j.n_dir] = v;
        }
    }
    for (int k = 0; k < head; ++k) {
        float4 v = hsum[k * kMxThreads];
#pragma unroll
        for (int m = 32; m > 0; m >>= 1) {
            v.x += __shfl_xor(v.x, m);
            v.y += __shfl_xor(v.y, m);
            v.z += __shfl_xor(v.z, m);
            v.w += __shfl_xor(v.w, m);
        }
        if (lane == 0) out[(int64_t)k * j.n_dir] = v;
    }
}

template <typename InT>
hipError_t launch_mx_t(const MxArgs& a, int rg, hipStream_t st, hipEvent_t ev_start, hipEvent_t ev_stop)
{
    const int64_t waves = (int64_t)a.splits * a.fgroups * a.job.n_dir;
    constexpr int per = kMxThreads / 64;
    const dim3 grid((unsigned)((waves + per - 1) / per)), block(kMxThreads);
    const size_t lds = (size_t)a.head * kMxThreads * sizeof(float4);
    auto go = [&](auto kern) -> hipError_t {
        if (ev_start || ev_stop) {
            MxArgs arg = a;
            void* args[] = {&arg};
            return hipExtLaunchKernel(reinterpret_cast<const void*>(kern), grid, block, args, lds, st, ev_start,
                                      ev_stop, 0);
        }
        hipLaunchKernelGGL(kern, grid, block, lds, st, a);
        return hipGetLastError();
    };
    switch (rg) {
    case 1: return go(k_accumulate_mx<InT, 1>);
    case 2: return go(k_accumulate_mx<InT, 2>);
    case 3: return go(k_accumulate_mx<InT, 3>);
    case 4: return go(k_accumulate_mx<InT, 4>);
    }
    return hipErrorInvalidValue;
}

}  // namespace

int mx_resident_waves(int rg) { return 4 * mx_waves(rg); }

hipError_t launch_accumulate_mx(const MxArgs& a, int dtype, int rg, hipStream_t st, hipEvent_t ev_start,
                                hipEvent_t ev_stop)
{
    return dtype == 0 ? launch_mx_t<float>(a, rg, st, ev_start, ev_stop)
                      : launch_mx_t<double>(a, rg, st, ev_start, ev_stop);
}

}  // namespace rad
