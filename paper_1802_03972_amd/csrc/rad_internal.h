// Internal interface between the host runtime and the gfx950 kernels (not part of the ABI).
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

struct rad_batcher;

namespace rad {

// Particles staged per workgroup chunk (one LDS round).
#ifndef RAD_CHUNK
#define RAD_CHUNK 32
#endif
constexpr int kChunk = RAD_CHUNK;

// One accumulation source: a particle range of one grid (one push, or one batch item).
struct Job {
    const void* f[10];      // x, y, z, bx, by, bz, dbx, dby, dbz, w (element type = kernel InT)
    int64_t i_begin;        // first particle index (into f[])
    int64_t i_end;          // one past the last
    int64_t n_per_step;     // particles per time step (step of element i = i / n_per_step)
    double t0, dt;          // t_j = t0 + j * dt
    const double* dirs9;    // [n_dir][9]: n, e1, e2 (e1, e2 span the plane normal to n)
    const double* omega;    // [n_omega]
    const float2* gtab;     // [n_omega]: (g, 1 - g) of a 1-D shape
    const float* g3;        // [n_dir][n_omega]: g of a 3-D (direction-dependent) shape, or null
    const double* bstep;    // [ceil(n_omega / 16)]: spacing inside each 16-frequency block of a
                            // piecewise-uniform frequency list, or null
    double domega;          // uniform spacing (unused for explicit frequency lists)
    int32_t n_dir, n_omega;
    int32_t tiles_d, tiles_w;
    int* err;               // sticky data-error flag of the grid
};

// Kernel variant bits: how the phase is advanced along the lane's frequencies and where
// the form factor comes from.
constexpr int kVarDirect = 1;   // explicit frequency list: phase from FP64 per term (no walk)
constexpr int kVarShape3 = 2;   // direction-dependent shape factor g(n, omega)
constexpr int kVarBlockStep = 4;  // piecewise-uniform list: frequency walk with a per-block step
// Frequencies per block of a piecewise-uniform list (= frequencies per lane of the variants).
constexpr int kBlockW = 16;

// Lanes of the accumulate kernel's flexible build (groups = 0: the fixed builds).
constexpr int kFlexChunk = 128;   // particles staged at most
struct FlexShape {
    int32_t dirs, blocks;         // tile: directions x blocks of W frequencies
    int32_t slots;                // sets of lanes of a wave that take particles in turn (power of two)
    int32_t groups;               // sets of waves that do (power of two)
    int32_t waves;                // waves of a group: slots * dirs * blocks <= 64 * waves
    int32_t block_stride;         // floats of one block's weights in the F table (>= W)
};

// Arguments of the per-grid accumulate kernel: block b handles tile b % ntiles of split
// b / ntiles, i.e. particles [split * per_split, +per_split) of the job, `chunk` at a time.
struct AccArgs {
    Job job;
    float* part;            // [splits][n_omega][n_dir][4] per-workgroup partial sums
    int32_t splits;
    int64_t per_split;
    int32_t chunk;          // at most kChunk (flexible build: kFlexChunk)
    FlexShape flex;
};

// Arguments of the matrix-core accumulate kernel: frequencies [k0, k0 + n_sub) of the job's grid,
// all with the shape factor g (g1 = 1 - g) but the first `head` of them (at most kMxHead, and only
// with k0 = 0), in fgroups groups of rg x 256; one wave for each (particle split, frequency
// group, direction).
struct MxArgs {
    Job job;
    float* part;            // [splits][n_sub][n_dir][4]
    float g, g1;
    int32_t k0, n_sub, head;
    int32_t fgroups;
    int32_t splits;
    int64_t per_split;
};
constexpr int kMxBlock = 256;   // frequencies of a row group
constexpr int kMxHead = 4;
// What undoes the mean shrink of its sums: 6.8e-8 in each of nine pushes of 3000 to 465000 particles,
// 12 bunches each (standard error 0.1e-8).
constexpr double kMxScale = 1.0 + 6.8e-8;

// Batched launch: every workgroup walks its own list of segments; a segment is a chunk
// range of one (item, tile) and owns one partial tile [TO][TD][4] in the segment buffer.
struct BatchSeg {
    int32_t item;
    int32_t tile;
    int64_t c_begin, c_end;
};

// Fold of one (grid, tile): sum of the listed segments' partial tiles into S.
struct FoldJob {
    double* S;              // grid accumulator, layout [n_omega][n_dir][4]
    int32_t n_dir, n_omega;
    int32_t td, tw;
    int32_t list_begin, list_end;   // into the segment index list
};

// Post-processing variant: one step of tracked particles into per-particle integrals.
struct TrackedArgs {
    const void* f[10];      // x, y, z, bx, by, bz, dbx, dby, dbz, w (w is not used);
                            // n_steps x n_particles elements, step-major
    int64_t n_particles;
    double t;               // time of the first step
    double dt;              // step of the time grid (t_j = t + j dt)
    int32_t n_steps;
    const double* dirs9;
    const double* omega;
    double domega;
    double* T;              // [n_particles][n_omega][n_dir][4] FP64
    bool T_zero;            // T holds zeros
    int* err;
    int32_t n_dir, n_omega;
};

struct LaunchShape {
    int w_per_lane;    // 16 | 32 (16 only for variant != 0)
    int dir_per_wave;  // 16 | 32 | 64
    int waves;         // 1..8
    int variant = 0;   // kVarDirect | kVarShape3 | kVarBlockStep bits
};

inline int tile_dirs(const LaunchShape& s) { return s.dir_per_wave; }
inline int tile_omegas(const LaunchShape& s) { return s.waves * (64 / s.dir_per_wave) * s.w_per_lane; }
inline size_t acc_lds_bytes(const LaunchShape& s)
{
    const size_t td = tile_dirs(s), to = tile_omegas(s);
    return kChunk * td * 16 + kChunk * td * 8 + 11 * kChunk * 8 + kChunk * 8 + kChunk * to * 4;
}

// Limits the FP32 sums in registers of a batcher's launches to `chunks` chunks of kChunk particles
// (0, as created: to a workgroup's range).
void batcher_limit_sums(rad_batcher* b, int chunks);

// LDS of the flexible build: a chunk's arrays, then the accumulators of half the groups.  The table
// of weights starts on 16 bytes, as it is read 16 bytes at a time (an odd chunk of an odd number of
// directions takes 8 bytes over a multiple of 16 before it).
__host__ __device__ inline int flex_weights_at(int dirs, int chunk)
{
    return (chunk * dirs * 24 + kFlexChunk * (11 * 8 + 8) + 15) / 16 * 16;
}
inline size_t flex_lds_bytes(const FlexShape& f, int w, int chunk)
{
    const size_t arrays = flex_weights_at(f.dirs, chunk) + (size_t)chunk * f.blocks * f.block_stride * 4;
    const size_t half = (size_t)(f.groups / 2) * f.waves * 64 * w * 16;
    return arrays > half ? arrays : half;
}

// Sets the calling thread's message returned by rad_last_error().
void set_last_error(const char* msg);

// Launchers (stream-ordered, return hipError_t).  Non-null ev_start / ev_stop are stamped
// with the kernel's own start and end (hipExtLaunchKernel: no separate marker packets on
// the stream, so timing does not slow the launch sequence down).
hipError_t launch_accumulate(const AccArgs& a, int dtype, int precision, const LaunchShape& s,
                             int n_blocks, hipStream_t st, hipEvent_t ev_start = nullptr,
                             hipEvent_t ev_stop = nullptr);
hipError_t launch_accumulate_mx(const MxArgs& a, int dtype, int rg, hipStream_t st, hipEvent_t ev_start = nullptr,
                                hipEvent_t ev_stop = nullptr);
// Waves of the matrix-core kernel with rg row groups (1..4) that one CU holds.
int mx_resident_waves(int rg);
// count = 4 * grid points (FP32 values per split); part is 16-byte aligned.  What is added to the
// points from scale_from on is scaled.
hipError_t launch_fold(const float* part, double* S, int splits, int64_t count, double scale, int64_t scale_from,
                       hipStream_t st, hipEvent_t ev_start = nullptr, hipEvent_t ev_stop = nullptr);
// sum_chunks: chunks of a sum in registers at most (0: whole segments).
hipError_t launch_accumulate_batch(const Job* items, const int32_t* wg_seg_begin, const BatchSeg* segs,
                                   float* seg_part, int sum_chunks, int dtype, int precision,
                                   const LaunchShape& s, int n_blocks, hipStream_t st);
// Kernel attributes only (no launch), so that a later stream capture records launches only.
hipError_t prepare_accumulate_batch(int sum_chunks, int dtype, int precision, const LaunchShape& s);
// n_jobs is read on the device (from n_jobs_dev) so that a captured graph can be replayed
// with different plans; the grid is sized for max_jobs.
hipError_t launch_fold_batch(const int32_t* n_jobs_dev, const FoldJob* jobs, int max_jobs,
                             const int32_t* seg_list, const float* seg_part, int td, int to, hipStream_t st);
// Read-outs.  The result and flag_out (may be null: the data-error flag *err) may be
// page-locked host memory.
hipError_t launch_finalize(const double* S, double* I, int n_dir, int n_omega, double C, const int* err,
                           int* flag_out, hipStream_t st);
hipError_t launch_cartesian(const double* S, const double* dirs9, double* out, int n_dir, int n_omega, const int* err,
                            int* flag_out, hipStream_t st);
// Zeroes p[0 .. n) (16-byte aligned, n even; n = 0: nothing) and the error flag.
hipError_t launch_reset(double* p, int64_t n, int* err, hipStream_t st);
hipError_t launch_trig_probe(const float* in, float* out, int n, hipStream_t st);
hipError_t launch_tracked_accumulate(const TrackedArgs& a, int dtype, bool direct, hipStream_t st);
hipError_t launch_tracked_finalize(const double* T, const double* wts, const double* gk, const double* g3,
                                   int64_t n_particles, int n_dir, int n_omega, double C, double* I, const int* err,
                                   int* flag_out, hipStream_t st);

}  // namespace rad
