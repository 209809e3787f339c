// Host runtime of the C ABI declared in include/rad.h: grid lifetime, validation, launch
// shapes, and the stream-ordered push / fold / read-out sequence.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <atomic>
#include <cmath>
#include <cstdarg>
#include <cstdio>
#include <cstring>
#include <mutex>
#include <string>
#include <vector>

#include "rad.h"
#include "rad_internal.h"

using rad::AccArgs;
using rad::LaunchShape;

namespace {

thread_local std::string t_last_error;

int fail(int code, const char* fmt, ...)
{
    char buf[512];
    va_list ap;
    va_start(ap, fmt);
    vsnprintf(buf, sizeof(buf), fmt, ap);
    va_end(ap);
    t_last_error = buf;
    return code;
}

int hip_fail(hipError_t e, const char* what)
{
    return fail(RAD_ERR_DEVICE, "%s: %s", what, hipGetErrorString(e));
}

#define RAD_HIP(call)                                         \
    do {                                                      \
        hipError_t e_ = (call);                               \
        if (e_ != hipSuccess) return hip_fail(e_, #call);     \
    } while (0)

constexpr double kC = 299792458.0;
constexpr double kQe = 1.602176634e-19;
constexpr double kEps0 = 8.8541878128e-12;
constexpr double kPi = 3.14159265358979323846;

// Normalised Table 1 shape factor |F~(omega)|^2 (F~(0) = 1), evaluated on the host once
// per grid and uploaded as (g, 1 - g) in FP32.
double shape_factor(int shape, double L, double omega)
{
    switch (shape) {
    case RAD_SHAPE_POINT: return 1.0;
    case RAD_SHAPE_GAUSS: {
        const double a = omega * L / kC;
        return std::exp(-a * a);
    }
    default: {
        const double x = 0.5 * omega * L / kC;
        const double s = x == 0.0 ? 1.0 : std::sin(x) / x;
        const double s2 = s * s;
        if (shape == RAD_SHAPE_CIC) return s2;
        if (shape == RAD_SHAPE_TSC) return s2 * s2;
        return s2 * s2 * s2;
    }
    }
}

bool is_shape3(int shape) { return shape >= RAD_SHAPE_CIC3D && shape <= RAD_SHAPE_QSC3D; }

// Cubic cell of side L: product over the axes of the 1-D shape factor at omega * n_c.
double shape_factor3(int shape, double L, const double n[3], double omega)
{
    const int s1 = shape - RAD_SHAPE_CIC3D + RAD_SHAPE_CIC;
    double g = 1.0;
    for (int c = 0; c < 3; ++c) g *= shape_factor(s1, L, omega * std::fabs(n[c]));
    return g;
}

// Orthonormal basis (e1, e2) of the plane normal to unit n.
void normal_basis(const double n[3], double e1[3], double e2[3])
{
    int a = 0;
    if (std::fabs(n[1]) < std::fabs(n[a])) a = 1;
    if (std::fabs(n[2]) < std::fabs(n[a])) a = 2;
    double u[3] = {0, 0, 0};
    u[a] = 1.0;
    const double un = u[0] * n[0] + u[1] * n[1] + u[2] * n[2];
    for (int c = 0; c < 3; ++c) e1[c] = u[c] - un * n[c];
    const double l1 = std::sqrt(e1[0] * e1[0] + e1[1] * e1[1] + e1[2] * e1[2]);
    for (int c = 0; c < 3; ++c) e1[c] /= l1;
    e2[0] = n[1] * e1[2] - n[2] * e1[1];
    e2[1] = n[2] * e1[0] - n[0] * e1[2];
    e2[2] = n[0] * e1[1] - n[1] * e1[0];
    const double l2 = std::sqrt(e2[0] * e2[0] + e2[1] * e2[1] + e2[2] * e2[2]);
    for (int c = 0; c < 3; ++c) e2[c] /= l2;
}

// ---- fixed scratch of the no-allocation push (rad_push_step_noalloc) ----------------
// That entry point keeps its FP32 partial sums in this file-scope device array instead of
// a grid's own buffers.  In host code the name `scratch` is only a host-side handle of the
// symbol, not a device address: the array's address on each GPU is looked up once per
// device (hipGetSymbolAddress, with that device current, when the first grid is created
// on it) and only that address is ever passed to kernels.
constexpr int kScratchDevices = 64;
static __device__ __align__(256) float scratch[RAD_NOALLOC_SCRATCH_BYTES / sizeof(float)];
std::mutex g_scratch_mu;
std::atomic<float*> g_scratch_addr[kScratchDevices];

// Looks up the scratch address on the current device `dev` (once per device).
int scratch_setup(int dev)
{
    if (dev < 0 || dev >= kScratchDevices)
        return fail(RAD_ERR_INVALID_ARG, "device %d beyond the %d devices the library supports", dev, kScratchDevices);
    std::lock_guard<std::mutex> lk(g_scratch_mu);
    if (g_scratch_addr[dev].load(std::memory_order_acquire)) return RAD_OK;
    void* p = nullptr;
    const hipError_t e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
    if (e != hipSuccess) return hip_fail(e, "hipGetSymbolAddress(scratch)");
    if (!p) return fail(RAD_ERR_DEVICE, "no device address for the no-allocation scratch");
    g_scratch_addr[dev].store(static_cast<float*>(p), std::memory_order_release);
    return RAD_OK;
}

// ---- page-locked host buffers of the read-outs ------------------------------------------
// A host read-out's kernel writes its result and the data-error flag into a page-locked buffer,
// the call waits for the stream once and copies the result on.  Through device memory it takes
// a wait for the flag and one for a copy into pageable memory: 482 points 48 us against 15,
// 32768 points 62 against 25, 1048576 points (8.4 MB) 517 against 438; the line below is where
// keeping the buffers costs more memory than the 15 % are worth.  The buffers are shared by all
// grids and threads, are held only during a call, at most kStagesKept are kept, and all are
// given back when the last grid is destroyed.
constexpr size_t kStageHeader = 256;      // the flag's place before the result
constexpr size_t kMaxStageBytes = (size_t)8 << 20;
constexpr size_t kStagesKept = 8;

// Allocating and freeing is no work on a stream, but would end a capture that another thread is in
// the middle of (of the default, global mode).
struct RelaxedCapture {
    hipStreamCaptureMode mode = hipStreamCaptureModeRelaxed;
    RelaxedCapture() { (void)hipThreadExchangeStreamCaptureMode(&mode); }
    ~RelaxedCapture() { (void)hipThreadExchangeStreamCaptureMode(&mode); }
};

class StagePool {
public:
    struct Stage {
        unsigned char* host = nullptr;
        unsigned char* dev = nullptr;     // the same memory as the device addresses it
        size_t bytes = 0;
        int* flag() const { return reinterpret_cast<int*>(host); }
    };
    void retain()
    {
        std::lock_guard<std::mutex> lk(mu_);
        ++users_;
    }
    void drop()
    {
        std::vector<Stage> gone;
        {
            std::lock_guard<std::mutex> lk(mu_);
            if (--users_ == 0) gone.swap(free_);
        }
        RelaxedCapture relaxed;
        for (const Stage& s : gone) (void)hipHostFree(s.host);
    }
    hipError_t take(size_t bytes, Stage* out)
    {
        {
            std::lock_guard<std::mutex> lk(mu_);
            auto best = free_.end();
            for (auto it = free_.begin(); it != free_.end(); ++it)
                if (it->bytes >= bytes && (best == free_.end() || it->bytes < best->bytes)) best = it;
            if (best != free_.end()) {
                *out = *best;
                free_.erase(best);
                return hipSuccess;
            }
        }
        Stage s;
        s.bytes = 64 * 1024;
        while (s.bytes < bytes) s.bytes *= 2;
        RelaxedCapture relaxed;
        hipError_t e = hipHostMalloc((void**)&s.host, s.bytes, hipHostMallocPortable | hipHostMallocMapped);
        if (e != hipSuccess) return e;
        e = hipHostGetDevicePointer((void**)&s.dev, s.host, 0);
        if (e != hipSuccess) {
            (void)hipHostFree(s.host);
            return e;
        }
        *out = s;
        return hipSuccess;
    }
    void give_back(const Stage& s)
    {
        {
            std::lock_guard<std::mutex> lk(mu_);
            if (users_ > 0 && free_.size() < kStagesKept) {
                free_.push_back(s);
                return;
            }
        }
        RelaxedCapture relaxed;
        (void)hipHostFree(s.host);
    }

private:
    std::mutex mu_;
    std::vector<Stage> free_;
    int64_t users_ = 0;
};

StagePool& stages()
{
    static StagePool* pool = new StagePool;   // outlives every grid, also at process end
    return *pool;
}

struct DeviceGuard {
    int prev = -1;
    explicit DeviceGuard(int dev)
    {
        if (hipGetDevice(&prev) != hipSuccess) prev = -1;
        if (prev != dev) (void)hipSetDevice(dev);
    }
    ~DeviceGuard()
    {
        int cur = -1;
        if (prev >= 0 && hipGetDevice(&cur) == hipSuccess && cur != prev) (void)hipSetDevice(prev);
    }
};

}  // namespace

// A range of a grid's frequencies and the kernel that accumulates it.
struct GridPart {
    int k0 = 0, n = 0;        // frequencies [k0, k0 + n)
    bool matrix = false;      // matrix-core kernel (k0 and all below: the general one)
    rad_tile tile{};          // general kernel's launch shape
    rad::FlexShape flex{};    // its flexible build for few directions (groups = 0: not used)
    int flex_chunk = 0;       // and the most particles it stages at a time
    int rg = 0, fgroups = 0;  // matrix kernel: row groups per wave, frequency groups, and
    int head = 0;             // the first frequencies that it sums apart
};

struct rad_grid {
    int device = 0;
    int n_dir = 0, n_omega = 0;
    double omega0 = 0, domega = 0, dt = 0, shape_len = 0;
    int shape = 0, precision = 0;
    double C = 0;
    int cus = 0;
    rad_tile tile{};
    // Where the tile is from: the cost model, a table of measured tiles (rad_hint_tile: the general
    // kernel's fixed tiles take it, other routes stay open) or the caller (rad_set_tile).
    enum TileFrom { kTileDefault, kTileHint, kTileSet } tile_from = kTileDefault;
    double* d_dirs9 = nullptr;
    double* d_omega = nullptr;
    float2* d_gtab = nullptr;
    double* d_S = nullptr;
    // Two partial-sum buffers, used in turn: a push on one stream may start its
    // accumulate while the fold of the previous push (issued on another stream) still
    // reads the other buffer.
    float* d_part[2] = {nullptr, nullptr};
    size_t part_bytes = 0;
    int part_next = 0;
    // Ordering of the work on S and on the partial-sum buffers (order_after, mark_done).
    struct Mark {
        hipEvent_t own = nullptr;
        hipEvent_t ev = nullptr;    // own, or the event that a launch stamped for another mark too
        hipStream_t on = nullptr;   // stream that the marked work was issued on
        bool set = false;           // something was marked
        bool recorded = false;      // ev stands for it (on the null stream: recorded when asked for)
    };
    Mark part_read[2];              // the fold that last read each partial-sum buffer
    Mark last_write;                // the last fold, batched fold, reset or device read-out of S
    int* d_err = nullptr;
    double* d_out = nullptr;
    float* d_g3 = nullptr;     // [n_dir][n_omega] for 3-D shapes
    double* d_bstep = nullptr; // per-block spacing of a piecewise-uniform frequency list
    int variant = 0;           // rad::kVarDirect | rad::kVarShape3
    int const_k0 = 0;          // from this frequency on (n_omega: none) the shape table holds
    float2 const_g{};          // one pair (g, 1 - g)
    std::vector<GridPart> parts;
    bool counted = false;      // among the users of the read-out buffers
    // kernel timing (rad_profile_*)
    bool profiling = false;
    int64_t prof_period = 1;    // time every prof_period-th accumulate launch
    int64_t prof_count = 0;
    std::vector<hipEvent_t> ev_pool;
    std::vector<std::pair<hipEvent_t, hipEvent_t>> ev_acc, ev_fold;
    int64_t prof_updates = 0;
};

namespace {

// Particles handled per workgroup in one launch at most (bounds the FP32 partial sums;
// longer pushes are cut into several launches, each folded into the FP64 accumulator).
constexpr int64_t kMaxPerWorkgroup = 32768;
constexpr int64_t kMinPerSplit = 8;
constexpr int64_t kFewSplits = 32;
constexpr double kSplitCost = 6.0;   // of a split, in particles of one group
constexpr int kMaxWaves = 8;     // of one workgroup

LaunchShape shape_of(const rad_tile& t, int variant = 0)
{
    return LaunchShape{t.w_per_lane, t.dir_per_wave, t.waves, variant};
}

int tiles_d_of(const rad_grid* g, const GridPart& p)
{
    return p.flex.groups ? 1 : (g->n_dir + p.tile.dir_per_wave - 1) / p.tile.dir_per_wave;
}
int tiles_w_of(const GridPart& p)
{
    const int to = p.flex.groups ? p.flex.blocks * p.tile.w_per_lane : rad::tile_omegas(shape_of(p.tile));
    return (p.n + to - 1) / to;
}
int tiles_of(const rad_grid* g, const GridPart& p) { return tiles_d_of(g, p) * tiles_w_of(p); }
constexpr int kFlexResident = 2;   // workgroups of the flexible build per CU (by its LDS)
// Particle splits that run together, rounded down: one more than fits would run alone, after
// all the others.
int max_splits(const rad_grid* g, const GridPart& p)
{
    const int64_t per_split = p.matrix ? (int64_t)g->n_dir * p.fgroups : tiles_of(g, p);
    const int64_t fit = (int64_t)g->cus * (p.matrix ? rad::mx_resident_waves(p.rg)
                                           : p.flex.groups ? kFlexResident : p.tile.wg_per_cu);
    return (int)std::max<int64_t>(1, fit / per_split);
}
size_t split_bytes(const rad_grid* g, const GridPart& p) { return (size_t)p.n * g->n_dir * 4 * sizeof(float); }

// What the general kernel's fixed tiles cost a grid, in cycles of a particle on the scale of
// flex_shape and matrix_shape, for the choice between those routes and this one: lanes outside
// the grid, the set-up that a tile's frequencies and directions share, and the waves that
// registers and LDS let run together.  `tile` (may be null): the tile of that cost.
double fixed_cost(int n_dir, int n_omega, int variant, rad_tile* tile = nullptr)
{
    // Waves per SIMD by registers (128 VGPRs for the walk kernels; 142 to 175 for the others),
    // and the cycles of 16 frequencies of one particle in the hot loop.
    const bool walk = variant == 0 || variant == rad::kVarBlockStep;
    const int slots = 4 * (walk ? 4 : 3);
    const double hot = walk ? 480.0 : 830.0;
    double best = 0.0;
    for (int dpw : {32, 16, 64}) {
        for (int waves = 8; waves >= 1; --waves) {
            const LaunchShape s{16, dpw, waves};
            const int to = rad::tile_omegas(s), per_wave = to / waves;
            if (waves > 1 && to - per_wave >= n_omega) continue;   // a wave without a frequency
            const int resident = std::min(slots / waves, (int)((160 * 1024) / rad::acc_lds_bytes(s)));
            if (resident < 1) continue;
            // issue rate by waves per SIMD (VOP2 loops: 6.2, 3.3 and 3.0 cycles an instruction at
            // one, two and four)
            const double per_simd = resident * waves / 4.0;
            const double rate = per_simd <= 1.0 ? 0.5 * per_simd
                                : per_simd <= 2.0 ? 0.5 + 0.38 * (per_simd - 1.0) : 0.88 + 0.06 * (per_simd - 2.0);
            const double tiles = (double)((n_dir + dpw - 1) / dpw) * ((n_omega + to - 1) / to);
            // geometry 600 cycles per 64 (particle, direction), weights 25 per 64 (particle, frequency)
            const double cost = tiles * (waves * hot + dpw * 9.4 + to * 0.4) / rate;
            if (best > 0.0 && cost >= best) continue;
            best = cost;
            if (tile) *tile = rad_tile{16, dpw, waves, std::min(resident, 16)};
        }
    }
    return best;
}

// Launch shape without a measured entry for the grid.  A simple rule, 32 directions up to 256
// frequencies, else 16, and as many waves as the frequencies fill, gives way to the tile for which
// a push of 50000 particles is faster by a twentieth (the walk kernels) or a tenth (the others), by
// the measured time of a particle on a tile.
//
// The times hold what a formula for the waves' residence missed: a workgroup's waves start on
// the same SIMD each time, so that 3, 5 or 6 of them load the SIMDs unevenly (6 cost what 8 do),
// and more than four waves of the kernels with three waves per SIMD leave room for no second
// workgroup (5 to 8 cost twice what 4 do).  Choosing by such a formula was up to 1.5 times
// slower than the rule: 120000 particles x 56 x 440 of an explicit list 1599 us by the rule, 2399
// by the formula and 1364 here; 64 x 786 1459, 1656 and 1395; 128 x 300 1234, 1312 and 1152.  The
// lines, a twentieth and for the other kernels a tenth, are where the measured choice begins
// to be right in all of 250 grids of 16 to 128 directions and 16 to 1024 frequencies, 20000 and
// 120000 particles: nothing slower than the rule by more than 5 %.
rad_tile default_tile(int n_dir, int n_omega, int variant = 0)
{
    // ns that a particle more costs on one tile of a full chip, by directions (16, 32, 64) and
    // waves (1 to 8), between 20000 and 120000 particles of 128 directions, each tile's own
    // number of frequencies; a push itself costs 8 us and the partial sums
    static const float kWalk[3][8] = {{.346f, .515f, .756f, .833f, 1.248f, 1.415f, 1.418f, 1.478f},
                                      {.476f, .522f, .807f, .879f, 1.336f, 1.444f, 1.470f, 1.526f},
                                      {1.838f, 1.173f, 1.071f, 1.009f, 1.389f, 1.538f, 1.531f, 1.584f}};
    static const float kDirect[3][8] = {{.562f, .929f, 1.338f, 1.469f, 3.275f, 3.279f, 3.280f, 3.290f},
                                        {.715f, .908f, 1.340f, 1.485f, 3.268f, 3.258f, 3.267f, 3.240f},
                                        {1.907f, 1.752f, 1.749f, 1.700f, 3.372f, 3.350f, 3.327f, 3.302f}};
    static const float kCubic[3][8] = {{.471f, .795f, 1.198f, 1.227f, 2.568f, 2.569f, 2.561f, 2.540f},
                                       {.649f, .770f, 1.263f, 1.293f, 2.658f, 2.622f, 2.627f, 2.629f},
                                       {1.881f, 1.573f, 1.483f, 1.418f, 2.761f, 2.724f, 2.693f, 2.690f}};
    const bool walk = variant == 0 || variant == rad::kVarBlockStep;
    const auto& ns = walk ? kWalk : variant & rad::kVarDirect ? kDirect : kCubic;
    // Splits for two rounds of resident workgroups, where that is faster: the other kernels' tiles of
    // three and four waves, whose one round ends unevenly.
    static const float kDirect2[2][2] = {{1.280f, 1.384f}, {1.286f, 1.402f}};
    static const float kCubic2[2][2] = {{1.141f, 1.169f}, {1.170f, 1.230f}};
    constexpr double kCus = 256.0, kParticles = 50000.0;
    auto tile = [](int dpw, int waves) {
        rad_tile t{16, dpw, waves, 0};
        // workgroups that four waves per SIMD and the LDS have room for
        t.wg_per_cu = std::max(2, std::min(std::max(1, 16 / waves), (int)((160 * 1024) / rad::acc_lds_bytes(shape_of(t)))));
        return t;
    };
    auto time = [&](const rad_tile& t, double tile_ns) {
        const int to = rad::tile_omegas(shape_of(t));
        const double tiles = (double)((n_dir + t.dir_per_wave - 1) / t.dir_per_wave) * ((n_omega + to - 1) / to);
        const double fit = kCus * t.wg_per_cu, splits = std::max(1.0, std::floor(fit / tiles));
        const double used = splits * tiles / (std::ceil(splits * tiles / fit) * fit);
        // in ns; the partial sums are written and folded at 5 TB/s
        return 8.0e3 + kParticles * tiles * tile_ns / used + splits * n_dir * n_omega * 16.0 * 0.2e-3;
    };
    const int dpw = n_dir >= 32 && n_omega <= 256 ? 32 : 16, per_wave = 64 / dpw * 16;
    rad_tile best = tile(dpw, std::min(8, std::max(1, (n_omega + per_wave - 1) / per_wave)));
    double best_time = time(best, ns[dpw / 32][best.waves - 1]) / (walk ? 1.05 : 1.1);
    auto consider = [&](const rad_tile& t, double tile_ns) {
        const double c = time(t, tile_ns);
        if (c >= best_time) return;
        best_time = c;
        best = t;
    };
    for (int d : {16, 32, 64}) {
        for (int waves = 1; waves <= 8; ++waves) {
            rad_tile t = tile(d, waves);
            const int to = rad::tile_omegas(shape_of(t));
            if (waves > 1 && to - to / waves >= n_omega) continue;   // a wave without a frequency
            // one round of three such waves is short of the workgroups that it has splits for
            // (48 x 175 of a list 596 us in one round of (16, 3), 486 in two)
            if (walk || d == 64 || waves != 3) consider(t, ns[d / 32][waves - 1]);
            if (!walk && d <= 32 && (waves == 3 || waves == 4)) {
                t.wg_per_cu *= 2;
                consider(t, (variant & rad::kVarDirect ? kDirect2 : kCubic2)[d / 32][waves - 3]);
            }
        }
    }
    return best;
}

// Launch shape of a batch.  The walk kernels keep fixed_cost's: a batch's workgroups take equal
// ranges of all its items, whatever the tile, so that what default_tile adds counts less there
// (of 40 drawn batches the two differ in 10, by -7 to +16 %), and the same shape sums the same
// particles together, so that results stay as they were.
rad_tile batch_tile(int n_dir, int n_omega, int variant)
{
    rad_tile t = default_tile(n_dir, n_omega, variant);
    if (variant == 0 || variant == rad::kVarBlockStep) fixed_cost(n_dir, n_omega, variant, &t);
    return t;
}

int floor_pow2(int x)
{
    int p = 1;
    while (2 * p <= x) p *= 2;
    return p;
}

// The flexible build's lanes for a grid of few directions: all directions x some blocks, up to
// eight waves (four of the kernels with three or two waves per SIMD), particles in turn in what
// is left of a wave and of the workgroup, and as many particles at a time as let two workgroups
// share a CU's LDS.  The blocks per tile are those of the least cost (fixed_cost's scale):
// idle lanes, the geometry that every tile computes, and the barriers of chunks in which a
// wave gets only a few particles, as the weights of many blocks leave LDS for few.  Blocks'
// weights are 20 floats apart where the lanes that read together span several blocks (16 would
// put them in the same banks).
void flex_shape(GridPart& p, int n_dir, int variant, double* cost_out)
{
    const bool walk = variant == 0 || variant == rad::kVarBlockStep, table = !(variant & rad::kVarShape3);
    const int max_waves = walk ? 8 : 4;
    const int nb = (p.n + 15) / 16;
    double best = 0.0;
    for (int blocks = std::min(nb, 64 * max_waves / n_dir); blocks >= 1; --blocks) {
        rad::FlexShape f{};
        f.dirs = n_dir;
        f.blocks = blocks;
        const int pairs = f.dirs * f.blocks;
        f.waves = (pairs + 63) / 64;
        f.slots = pairs <= 32 ? floor_pow2(64 / pairs) : 1;
        f.groups = floor_pow2(max_waves / f.waves);
        f.block_stride = table ? (n_dir < 8 ? 20 : 16) : 0;
        const int per_particle = f.dirs * 24 + f.blocks * f.block_stride * 4;
        const int fit = std::min(rad::kFlexChunk, (78 * 1024 - rad::kFlexChunk * 96) / per_particle);
        if (fit < 1) continue;
        while (f.groups > 1 && f.groups * f.slots > fit) f.groups /= 2;
        while (f.slots > fit) f.slots /= 2;
        const int rounds = fit / (f.groups * f.slots);     // of all slots and groups in a chunk
        // waves beyond a multiple of four share two of the four SIMDs
        const int wg_waves = f.waves * f.groups;
        const double uneven = (wg_waves + 3) / 4 * 4.0 / wg_waves;
        const double cost = (double)((nb + blocks - 1) / blocks) *
                            (f.waves * (walk ? 480.0 : 830.0) / f.slots * (1.0 + 1.0 / rounds) * uneven + n_dir * 9.4 +
                             (table ? blocks * 6.4 : 0.0));
        if (best > 0.0 && cost >= best) continue;
        best = cost;
        p.flex = f;
        p.flex_chunk = rounds * f.groups * f.slots;
    }
    p.tile = rad_tile{16, 16, 1, 1};
    if (cost_out) *cost_out = best;
}

// Row groups per wave and frequency groups of the matrix kernel for n frequencies, and its cost
// on fixed_cost's scale: per 16 particles 420 cycles for the columns and 480 for each row
// group, 450 per 64 particles for the geometry.
double matrix_shape(int n_dir, int n, int* rg, int* fgroups)
{
    const int groups = (n + rad::kMxBlock - 1) / rad::kMxBlock;
    *fgroups = (groups + 3) / 4;
    *rg = (groups + *fgroups - 1) / *fgroups;
    return (double)n_dir * *fgroups * ((420.0 + 480.0 * *rg) / 16.0 + 7.0);
}

// The general kernel's build and shape for a grid's first n frequencies: below kFewDirections
// directions the fixed builds' tiles (16 and more) are mostly empty, and the flexible build is
// used where it costs less.  Push with fold, fixed tiles and flexible: 30000 x 1 x 1000 114 and
// 39 us, 100000 x 2 x 241 112 and 40, 30000 x 2 x 241 of an explicit list 68 and 26, 30000 x 5 x
// 241 48 and 30, cubic cells 66 and 34, 30000 x 8 x 40 29 and 21; 30000 x 15 x 300 is faster in
// fixed tiles (61 and 66).
constexpr int kFewDirections = 16;
void general_part(GridPart& p, const rad_grid* g, int n, double* cost)
{
    double fixed = fixed_cost(g->n_dir, n, g->variant), flex = 0.0;
    p.n = n;
    p.tile = default_tile(g->n_dir, n, g->variant);
    if (g->n_dir < kFewDirections) {
        GridPart f;
        f.n = n;
        flex_shape(f, g->n_dir, g->variant, &flex);
        if (flex < fixed) {
            p = f;
            fixed = flex;
        }
    }
    if (cost) *cost = fixed;
}

// Which kernel accumulates which frequencies.  The matrix kernel takes the frequencies over
// which the shape factor is one constant, and up to kMxHead before them; with more before
// them the general kernel takes those, in whole blocks of 16.  It is used where its waves of
// 256 frequencies of one direction cost less than the general kernel's tiles: from about half
// a wave's 256 frequencies on, from fewer for directions that fill a tile badly (256
// frequencies 0.75 ms against 1.54 for 200000 particles x 128 directions).  A launch shape that the
// caller set takes the whole grid.
void plan_parts(rad_grid* g)
{
    g->parts.clear();
    if (g->tile_from == rad_grid::kTileSet) {
        GridPart set;
        set.n = g->n_omega;
        set.tile = g->tile;
        g->parts.push_back(set);
        return;
    }
    GridPart lo, mx;
    mx.matrix = true;
    mx.head = g->const_k0 <= rad::kMxHead ? g->const_k0 : 0;
    mx.k0 = mx.head ? 0 : (g->const_k0 + 15) / 16 * 16;
    mx.n = g->n_omega - mx.k0;
    if (g->variant == 0 && g->precision == RAD_PHASE_F64 && mx.n >= 16 && g->const_k0 < g->n_omega) {
        double all_cost = 0.0, lo_cost = 0.0;
        GridPart any;
        general_part(any, g, g->n_omega, &all_cost);
        if (mx.k0 > 0) general_part(lo, g, mx.k0, &lo_cost);
        const double mx_cost = matrix_shape(g->n_dir, mx.n, &mx.rg, &mx.fgroups);
        if (lo_cost + mx_cost < 0.9 * all_cost) {
            if (lo.n > 0) g->parts.push_back(lo);
            g->parts.push_back(mx);
            return;
        }
    }
    GridPart all;
    general_part(all, g, g->n_omega, nullptr);
    if (g->tile_from == rad_grid::kTileHint || !all.flex.groups) {
        all = GridPart{};
        all.n = g->n_omega;
        all.tile = g->tile;
    }
    g->parts.push_back(all);
}

int validate_tile(const rad_tile& t)
{
    if (t.w_per_lane != 16 && t.w_per_lane != 32)
        return fail(RAD_ERR_INVALID_ARG, "w_per_lane must be 16 or 32 (got %d)", t.w_per_lane);
    if (t.dir_per_wave != 16 && t.dir_per_wave != 32 && t.dir_per_wave != 64)
        return fail(RAD_ERR_INVALID_ARG, "dir_per_wave must be 16, 32 or 64 (got %d)", t.dir_per_wave);
    if (t.waves < 1 || t.waves > 8)
        return fail(RAD_ERR_INVALID_ARG, "waves must be in 1..8 (got %d)", t.waves);
    if (t.wg_per_cu < 1 || t.wg_per_cu > 16)
        return fail(RAD_ERR_INVALID_ARG, "wg_per_cu must be in 1..16 (got %d)", t.wg_per_cu);
    if (rad::acc_lds_bytes(shape_of(t)) > 160 * 1024)
        return fail(RAD_ERR_INVALID_ARG, "tile needs %zu B of LDS (> 160 KiB)",
                    rad::acc_lds_bytes(shape_of(t)));
    return RAD_OK;
}

// A launch shape, checked, as the grid's.
int apply_tile(rad_grid* g, const rad_tile& t, rad_grid::TileFrom from)
{
    if (int rc = validate_tile(t)) return rc;
    if (g->variant != 0 && t.w_per_lane != 16)
        return fail(RAD_ERR_INVALID_ARG, "grids with a frequency list or a 3-D shape need w_per_lane = 16");
    g->tile = t;
    g->tile_from = from;
    return RAD_OK;
}

int ensure_partials(rad_grid* g)
{
    size_t bytes = 0;
    for (const GridPart& p : g->parts) bytes = std::max(bytes, max_splits(g, p) * split_bytes(g, p));
    if (bytes <= g->part_bytes) return RAD_OK;
    if (g->d_part[0] || g->d_part[1]) {
        RAD_HIP(hipDeviceSynchronize());
        for (int b = 0; b < 2; ++b) {
            if (g->d_part[b]) RAD_HIP(hipFree(g->d_part[b]));
            g->d_part[b] = nullptr;
        }
        g->part_bytes = 0;
    }
    for (int b = 0; b < 2; ++b) {
        if (hipMalloc(&g->d_part[b], bytes) != hipSuccess) {
            g->d_part[b] = nullptr;
            return fail(RAD_ERR_OOM, "cannot allocate 2 x %zu B of partial sums", bytes);
        }
    }
    g->part_bytes = bytes;
    return RAD_OK;
}

int change_tile(rad_grid* g, const rad_tile* t, rad_grid::TileFrom from)
{
    if (!g || !t) return fail(RAD_ERR_INVALID_ARG, "grid and tile must be non-NULL");
    DeviceGuard dg(g->device);
    const rad_tile old = g->tile;
    const rad_grid::TileFrom old_from = g->tile_from;
    int rc = apply_tile(g, *t, from);
    if (rc) return rc;
    plan_parts(g);
    rc = ensure_partials(g);
    if (rc) {
        g->tile = old;
        g->tile_from = old_from;
        plan_parts(g);
    }
    return rc;
}

void release_events(rad_grid* g)
{
    for (auto& e : g->ev_acc) { g->ev_pool.push_back(e.first); g->ev_pool.push_back(e.second); }
    for (auto& e : g->ev_fold) { g->ev_pool.push_back(e.first); g->ev_pool.push_back(e.second); }
    g->ev_acc.clear();
    g->ev_fold.clear();
}

hipError_t take_event(rad_grid* g, hipEvent_t* ev)
{
    if (!g->ev_pool.empty()) {
        *ev = g->ev_pool.back();
        g->ev_pool.pop_back();
        return hipSuccess;
    }
    return hipEventCreate(ev);
}

void free_grid(rad_grid* g)
{
    if (!g) return;
    DeviceGuard dg(g->device);
    release_events(g);
    for (hipEvent_t e : g->ev_pool) (void)hipEventDestroy(e);
    g->ev_pool.clear();
    if (g->d_dirs9) (void)hipFree(g->d_dirs9);
    if (g->d_omega) (void)hipFree(g->d_omega);
    if (g->d_gtab) (void)hipFree(g->d_gtab);
    if (g->d_S) (void)hipFree(g->d_S);
    for (int b = 0; b < 2; ++b) {
        if (g->d_part[b]) (void)hipFree(g->d_part[b]);
        if (g->part_read[b].own) (void)hipEventDestroy(g->part_read[b].own);
    }
    if (g->last_write.own) (void)hipEventDestroy(g->last_write.own);
    if (g->d_err) (void)hipFree(g->d_err);
    if (g->d_out) (void)hipFree(g->d_out);
    if (g->d_g3) (void)hipFree(g->d_g3);
    if (g->d_bstep) (void)hipFree(g->d_bstep);
    if (g->counted) stages().drop();
    delete g;
}

int check_particles(const rad_particles* p)
{
    if (!p) return fail(RAD_ERR_INVALID_ARG, "particles is NULL");
    if (p->dtype != RAD_F32 && p->dtype != RAD_F64)
        return fail(RAD_ERR_INVALID_ARG, "particle dtype must be RAD_F32 or RAD_F64 (got %d)", p->dtype);
    const void* f[10] = {p->x, p->y, p->z, p->bx, p->by, p->bz, p->dbx, p->dby, p->dbz, p->w};
    static const char* names[10] = {"x", "y", "z", "bx", "by", "bz", "dbx", "dby", "dbz", "w"};
    for (int i = 0; i < 10; ++i)
        if (!f[i]) return fail(RAD_ERR_INVALID_ARG, "particle field %s is NULL", names[i]);
    return RAD_OK;
}

void fill_job(rad::Job& j, const rad_grid* g, const rad_particles* p, double t0, int64_t n_per_step,
              const rad_tile& t)
{
    j.f[0] = p->x; j.f[1] = p->y; j.f[2] = p->z;
    j.f[3] = p->bx; j.f[4] = p->by; j.f[5] = p->bz;
    j.f[6] = p->dbx; j.f[7] = p->dby; j.f[8] = p->dbz; j.f[9] = p->w;
    j.n_per_step = n_per_step;
    j.t0 = t0;
    j.dt = g->dt;
    j.dirs9 = g->d_dirs9;
    j.omega = g->d_omega;
    j.gtab = g->d_gtab;
    j.g3 = g->d_g3;
    j.bstep = g->d_bstep;
    j.domega = g->domega;
    j.n_dir = g->n_dir;
    j.n_omega = g->n_omega;
    const int to = rad::tile_omegas(shape_of(t));
    j.tiles_d = (g->n_dir + t.dir_per_wave - 1) / t.dir_per_wave;
    j.tiles_w = (g->n_omega + to - 1) / to;
    j.err = g->d_err;
}

// Cuts particles [0, total) into launches of at most target_splits particle splits of at most
// kMaxPerWorkgroup particles each, and sets a's particle range and its split into workgroups
// for each launch before calling fn() (which returns a status code).
//
// From target_splits full chunks on there is one split for each workgroup that the tile asks
// for, all of the same length to one particle, in chunks of one length.  A smaller push has
// fewer chunks than that: the idle waves first share the chunks' particles (groups of the
// flexible build, up to eight waves a workgroup), then the splits get shorter, down to
// kMinPerSplit particles, to the length of the least time: that of a split times the waves on
// the fullest SIMD, where two take hardly longer than one.  The flexible build of few directions has its groups already; where
// they are one, its splits may be shorter than that as long as there are only kFewSplits of
// them (each is a partial tile to write and to fold: 15 x 540 points, 1500 particles 34 us in
// splits of 3 and 22 in splits of 8; 256 particles 20.6 and 15; 16 particles 11.9 in splits of
// 1 and 13.2 of 8).
// 1024 particles x 16 x 64 points 19.0 -> 8.2 us (128 workgroups of 8 waves instead of 32 of
// one), 2000 x 2 x 241 of an explicit list 22.6 -> 10.7; 50000 x 128 x 256 of a block-stepped
// list, 391 particles a split instead of 13 chunks in 121 of 128 splits, 380 -> 355.
//
// The matrix kernel's splits are whole steps of 16 particles, at least two.
template <typename Fn>
int for_each_launch(const rad_grid* g, AccArgs& a, int64_t total, int64_t target_splits, const GridPart& part, Fn fn)
{
    const int64_t per_launch_cap = target_splits * kMaxPerWorkgroup;
    for (int64_t i0 = 0; i0 < total; i0 += per_launch_cap) {
        const int64_t i1 = std::min(total, i0 + per_launch_cap);
        const int64_t n = i1 - i0;
        int64_t per = (n + target_splits - 1) / target_splits;
        int64_t most = rad::kChunk, step = 1;   // particles of a chunk: at most, and a multiple of
        a.flex = part.flex;
        if (part.matrix) {
            per = std::max<int64_t>(32, (per + 15) / 16 * 16);
        } else if (part.flex.groups) {
            step = part.flex.slots * part.flex.groups;
            most = part.flex_chunk;
            per = std::max({per, step, std::min(kMinPerSplit, (n + kFewSplits - 1) / kFewSplits)});
        } else if (per <= rad::kChunk) {
            int groups = 1;
            const int64_t chunks = (n + rad::kChunk - 1) / rad::kChunk;
            while (2 * groups * part.tile.waves <= kMaxWaves && chunks * 2 * groups <= target_splits) groups *= 2;
            per = rad::kChunk;
            double best = 0.0;
            // for each number of workgroups on a CU the shortest splits that make no more (in 32
            // bits: 64-bit divisions cost a push 0.4 us)
            const int tiles = tiles_of(g, part), particles = (int)n, target = (int)target_splits;
            for (int on_cu = 1; on_cu <= part.tile.wg_per_cu; ++on_cu) {
                const int most = std::min(on_cu * g->cus / tiles, target / groups);
                if (most < 1) continue;
                const int p = std::max((int)kMinPerSplit, (particles + most - 1) / most);
                if (p > rad::kChunk) continue;
                const double load = std::max(2.0, on_cu * groups * part.tile.waves / 4.0);
                const double time = load * ((p + groups - 1) / groups + kSplitCost);
                if (best == 0.0 || time < best) {
                    best = time;
                    per = p;
                }
            }
            if (groups > 1) {
                const LaunchShape ls = shape_of(part.tile);
                a.flex = rad::FlexShape{rad::tile_dirs(ls), rad::tile_omegas(ls) / ls.w_per_lane, 1, groups, ls.waves,
                                        ls.w_per_lane};
            }
        }
        const int64_t chunks = (per + most - 1) / most;
        a.job.i_begin = i0;
        a.job.i_end = i1;
        a.splits = (int32_t)((n + per - 1) / per);
        a.per_split = per;
        a.chunk = (int32_t)(((per + chunks - 1) / chunks + step - 1) / step * step);
        if (int rc = fn()) return rc;
    }
    return RAD_OK;
}

// The launch of one part that for_each_launch prepared in `a`.
hipError_t launch_part(const rad_grid* g, const AccArgs& a, const GridPart& part, int dtype, hipStream_t st,
                       hipEvent_t e0 = nullptr, hipEvent_t e1 = nullptr)
{
    if (!part.matrix)
        return rad::launch_accumulate(a, dtype, g->precision, shape_of(part.tile, g->variant),
                                      a.splits * tiles_of(g, part), st, e0, e1);
    rad::MxArgs m{};
    m.job = a.job;
    m.part = a.part;
    m.g = g->const_g.x;
    m.g1 = g->const_g.y;
    m.k0 = part.k0;
    m.n_sub = part.n;
    m.head = part.head;
    m.fgroups = part.fgroups;
    m.splits = a.splits;
    m.per_split = a.per_split;
    return rad::launch_accumulate_mx(m, dtype, part.rg, st, e0, e1);
}

// Adds a launch's partial sums to the part's range of S ([omega][dir]: a contiguous one).
hipError_t fold_part(const rad_grid* g, const AccArgs& a, const GridPart& part, hipStream_t st,
                     hipEvent_t e0 = nullptr, hipEvent_t e1 = nullptr)
{
    return rad::launch_fold(a.part, g->d_S + (int64_t)part.k0 * g->n_dir * 4, a.splits, (int64_t)part.n * g->n_dir * 4,
                            part.matrix ? rad::kMxScale : 1.0, (int64_t)part.head * g->n_dir, st, e0, e1);
}

// The job of one part: the general kernel sees the frequencies below the part's end.
void part_job(rad::Job& j, const rad_grid* g, const GridPart& part, const rad_particles* p, double t0,
              int64_t n_per_step)
{
    fill_job(j, g, p, t0, n_per_step, part.matrix ? g->tile : part.tile);
    if (part.matrix) return;
    j.n_omega = part.n;
    j.tiles_d = tiles_d_of(g, part);
    j.tiles_w = tiles_w_of(part);
}

bool captures(hipStream_t st, hipError_t* e)
{
    hipStreamCaptureStatus cap = hipStreamCaptureStatusNone;
    *e = st ? hipStreamIsCapturing(st, &cap) : hipSuccess;   // the null stream cannot capture
    return cap != hipStreamCaptureStatusNone;
}

// Calls that read or set the grid's marks, the partial-sum buffers' turn or a plan, or that wait
// for the stream, are of no use in a graph: a replay knows nothing of the marks, and a mark made
// in a capture is no event that later work could wait for.
int refuse_capture(hipStream_t st, const char* call)
{
    hipError_t e;
    const bool capturing = captures(st, &e);
    if (e != hipSuccess) return hip_fail(e, "hipStreamIsCapturing");
    return capturing ? fail(RAD_ERR_INVALID_ARG, "%s cannot be captured (rad_push_step_noalloc can)", call) : RAD_OK;
}

// Work marked on one stream is ordered before later work on another by an event; work on
// the stream of the mark needs none.  On a caller's own stream the event is recorded when the
// work is issued (the stream may be gone when somebody asks).  The null stream is always
// there, so its event is recorded only when another stream asks: a program on the default
// stream pays for no event (a record and the wait for it are 4 to 6 us of host time each, and
// an event stamped by a fold left the GPU idle for 4.7 us before the next push's accumulate).
hipError_t order_after(rad_grid::Mark& m, hipStream_t st)
{
    if (!m.set || m.on == st) return hipSuccess;
    if (!m.recorded) {
        const hipError_t e = hipEventRecord(m.ev, m.on);
        if (e != hipSuccess) return e;
        m.recorded = true;
    }
    return hipStreamWaitEvent(st, m.ev, 0);
}

// Everything issued on `st` so far is marked.  stamped: an event that the last launch on `st`
// stamped (a caller's own stream only), or null to record the mark's own.
hipError_t mark_done(rad_grid::Mark& m, hipStream_t st, hipEvent_t stamped = nullptr)
{
    m.on = st;
    m.set = true;
    m.recorded = st != nullptr;
    m.ev = st && stamped ? stamped : m.own;
    return m.recorded && !stamped ? hipEventRecord(m.ev, st) : hipSuccess;
}

// One launch of a push (accumulate and fold) of one part, as for_each_launch prepared it.
int push_launch(rad_grid* g, const GridPart& part, AccArgs& a, int dtype, hipStream_t st, bool timed_push)
{
    const int b = g->part_next;
    g->part_next ^= 1;
    a.part = g->d_part[b];
    // the fold that last read this buffer must be done before it is overwritten
    RAD_HIP(order_after(g->part_read[b], st));
    hipEvent_t e0 = nullptr, e1 = nullptr, e2 = nullptr, e3 = nullptr;
    // a grid of two parts times both launches of a push, or neither
    if (timed_push || (g->profiling && g->parts.size() == 1 && g->prof_count++ % g->prof_period == 0)) {
        RAD_HIP(take_event(g, &e0));
        RAD_HIP(take_event(g, &e1));
        RAD_HIP(take_event(g, &e2));
        RAD_HIP(take_event(g, &e3));
        g->ev_acc.emplace_back(e0, e1);
        g->ev_fold.emplace_back(e2, e3);
        g->prof_updates += (a.job.i_end - a.job.i_begin) * (int64_t)g->n_dir * part.n;
    }
    hipError_t e = launch_part(g, a, part, dtype, st, e0, e1);
    if (e != hipSuccess) return hip_fail(e, "accumulate launch");
    // The fold runs right after the accumulate on the caller's stream, so it has the
    // whole GPU for its few microseconds (beside the next push's accumulate it would
    // trickle along in the few free wave slots), and after every write of S already issued
    // on another stream.  Where an event is needed (another stream than the null stream)
    // the fold's launch stamps it, without a marker between this fold and the next push's
    // accumulate; a timed fold stamps its timing event, and the mark is recorded after it.
    RAD_HIP(order_after(g->last_write, st));
    const hipEvent_t stamp = e3 || !st ? nullptr : g->part_read[b].own;
    e = fold_part(g, a, part, st, e2, e3 ? e3 : stamp);
    if (e != hipSuccess) return hip_fail(e, "fold launch");
    RAD_HIP(mark_done(g->part_read[b], st, stamp));
    RAD_HIP(mark_done(g->last_write, st, st ? g->part_read[b].own : nullptr));
    return RAD_OK;
}

// Accumulate particles [0, total) (step of element i is i / n_per_step, t = t0 + step*dt).
int push_range(rad_grid* g, double t0, int64_t n_per_step, int64_t total, const rad_particles* p,
               hipStream_t st)
{
    int rc = ensure_partials(g);
    if (rc) return rc;
    const bool timed_push = g->profiling && g->parts.size() > 1 && g->prof_count++ % g->prof_period == 0;
    for (const GridPart& part : g->parts) {
        AccArgs a{};
        part_job(a.job, g, part, p, t0, n_per_step);
        rc = for_each_launch(g, a, total, max_splits(g, part), part, [&]() -> int {
            return push_launch(g, part, a, p->dtype, st, timed_push);
        });
        if (rc) return rc;
    }
    return RAD_OK;
}

int read_err_flag(rad_grid* g, hipStream_t st, int* flag)
{
    RAD_HIP(hipMemcpyAsync(flag, g->d_err, sizeof(int), hipMemcpyDeviceToHost, st));
    RAD_HIP(hipStreamSynchronize(st));
    return RAD_OK;
}

const char* const kBadData = "device detected invalid particle data (non-finite, N < 0 or 1 - beta.n <= 0)";

// Host read-out of `count` doubles: launch(result, flag, stream) writes them and the data-error
// flag.  Up to kMaxStageBytes they go straight to page-locked memory; larger ones through the
// grid's device buffer.  Nothing is written to `out` when the flag is set.
template <typename Launch>
int read_out(rad_grid* g, double* out, size_t count, hipStream_t st, Launch launch)
{
    RAD_HIP(order_after(g->last_write, st));
    const size_t bytes = count * sizeof(double);
    StagePool::Stage sg;
    if (bytes + kStageHeader <= kMaxStageBytes && stages().take(bytes + kStageHeader, &sg) == hipSuccess) {
        hipError_t e = launch(reinterpret_cast<double*>(sg.dev + kStageHeader), reinterpret_cast<int*>(sg.dev), st);
        if (e == hipSuccess) e = hipStreamSynchronize(st);
        // a buffer that a kernel may still write to is not handed on
        if (e != hipSuccess) return hip_fail(e, "read-out");
        const bool bad = *sg.flag() != 0;
        if (!bad) std::memcpy(out, sg.host + kStageHeader, bytes);
        stages().give_back(sg);
        return bad ? fail(RAD_ERR_BAD_DATA, "%s", kBadData) : RAD_OK;
    }
    const hipError_t e = launch(g->d_out, nullptr, st);
    if (e != hipSuccess) return hip_fail(e, "read-out launch");
    int flag = 0;
    if (int rc = read_err_flag(g, st, &flag)) return rc;
    if (flag) return fail(RAD_ERR_BAD_DATA, "%s", kBadData);
    RAD_HIP(hipMemcpyAsync(out, g->d_out, bytes, hipMemcpyDeviceToHost, st));
    RAD_HIP(hipStreamSynchronize(st));
    return RAD_OK;
}

}  // namespace

namespace {

// Validated host-side tables of a grid description: directions with their normal basis
// (n, e1, e2), the frequency list, the walk step, the Eq. 13 prefactor and the
// kernel variant.  check_shape = false skips the shape fields (chosen later).
struct GridTables {
    std::vector<double> dirs9, om;
    std::vector<double> bstep;   // per 16-frequency block spacing (piecewise-uniform lists)
    double domega = 0.0, C = 0.0;
    int variant = 0;
};

// How an explicit frequency list can be evaluated.  A list whose every aligned block of
// kBlockW frequencies is an arithmetic progression (to a few FP64 ulps) runs the frequency
// walk with a per-block step; if the steps also agree and the blocks continue one
// another, the list is one uniform grid.  Otherwise each term takes its own FP64 phase.
int classify_list(const std::vector<double>& om, std::vector<double>& bstep, double& domega)
{
    const int n = (int)om.size(), W = rad::kBlockW;
    const int nb = (n + W - 1) / W;
    bstep.assign((size_t)nb, 0.0);
    auto close = [](double a, double b) {
        const double tol = 16.0 * 2.220446049250313e-16 * std::max(std::fabs(a), std::fabs(b));
        return std::fabs(a - b) <= tol;
    };
    for (int b = 0; b < nb; ++b) {
        const int k0 = b * W, k1 = std::min(n, k0 + W);
        if (k1 - k0 < 2) continue;
        const double st = (om[k1 - 1] - om[k0]) / (double)(k1 - 1 - k0);
        for (int k = k0 + 2; k < k1; ++k)
            if (!close(om[k], om[k0] + (double)(k - k0) * st)) return rad::kVarDirect;
        bstep[b] = st;
    }
    if (n >= 2) {
        const double st = (om[n - 1] - om[0]) / (double)(n - 1);
        bool uniform = true;
        for (int k = 2; k < n && uniform; ++k) uniform = close(om[k], om[0] + (double)k * st);
        if (uniform) {
            domega = st;
            return 0;
        }
    } else {
        domega = 0.0;
        return 0;
    }
    return rad::kVarBlockStep;
}

int prepare_tables(const rad_grid_desc* d, bool check_shape, GridTables& tb)
{
    if (d->n_dir < 1 || !d->dirs) return fail(RAD_ERR_INVALID_ARG, "need n_dir >= 1 and dirs");
    if (d->n_omega < 1) return fail(RAD_ERR_INVALID_ARG, "need n_omega >= 1");
    if (d->omegas) {
        for (int k = 0; k < d->n_omega; ++k)
            if (!(d->omegas[k] >= 0.0) || !std::isfinite(d->omegas[k]))
                return fail(RAD_ERR_INVALID_ARG, "omegas[%d] must be finite and >= 0", k);
    } else if (!(d->omega0 >= 0.0) || !std::isfinite(d->omega0) || !(d->domega >= 0.0) || !std::isfinite(d->domega)) {
        return fail(RAD_ERR_INVALID_ARG, "omega0 and domega must be finite and >= 0");
    }
    if (check_shape) {
        if (d->shape < RAD_SHAPE_POINT || d->shape > RAD_SHAPE_QSC3D)
            return fail(RAD_ERR_INVALID_ARG, "unknown shape %d", d->shape);
        if (d->shape != RAD_SHAPE_POINT && !(d->shape_len > 0.0 && std::isfinite(d->shape_len)))
            return fail(RAD_ERR_INVALID_ARG, "shape_len must be finite and > 0");
    }
    if (!(d->dt > 0.0) || !std::isfinite(d->dt)) return fail(RAD_ERR_INVALID_ARG, "dt must be finite and > 0");
    if (d->precision != RAD_PHASE_F64 && d->precision != RAD_ALL_F32)
        return fail(RAD_ERR_INVALID_ARG, "unknown precision mode %d", d->precision);
    const int64_t points = (int64_t)d->n_dir * d->n_omega;
    if (points > (int64_t)1 << 28) return fail(RAD_ERR_INVALID_ARG, "grid of %lld points too large", (long long)points);
    tb.dirs9.resize((size_t)d->n_dir * 9);
    for (int i = 0; i < d->n_dir; ++i) {
        const double* n = d->dirs + 3 * i;
        const double len = std::sqrt(n[0] * n[0] + n[1] * n[1] + n[2] * n[2]);
        if (!std::isfinite(len) || std::fabs(len - 1.0) > 1e-6)
            return fail(RAD_ERR_INVALID_ARG, "direction %d is not a unit vector (|n| = %.17g)", i, len);
        double* o = tb.dirs9.data() + 9 * i;
        o[0] = n[0]; o[1] = n[1]; o[2] = n[2];
        normal_basis(n, o + 3, o + 6);
    }
    tb.om.resize((size_t)d->n_omega);
    for (int k = 0; k < d->n_omega; ++k) {
        if (d->omegas) {
            tb.om[k] = d->omegas[k];
        } else {
            volatile double kd = (double)k * d->domega;  // one rounding per operation, no fma
            tb.om[k] = d->omega0 + kd;
        }
    }
    tb.domega = d->domega;
    const int list_kind = d->omegas ? classify_list(tb.om, tb.bstep, tb.domega) : 0;
    if (list_kind != rad::kVarBlockStep) tb.bstep.clear();
    if (list_kind == rad::kVarDirect) tb.domega = 0.0;
    const double q = kQe * d->dt;
    tb.C = q * q / (16.0 * kPi * kPi * kPi * kEps0 * kC);
    tb.variant = list_kind | (check_shape && is_shape3(d->shape) ? rad::kVarShape3 : 0);
    return RAD_OK;
}

// What a grid is without a device: its description, and the shape table (g, 1 - g).
void describe_grid(rad_grid* g, const rad_grid_desc* d, const GridTables& tb, int cus, std::vector<float2>& gt)
{
    g->device = d->device;
    g->n_dir = d->n_dir;
    g->n_omega = d->n_omega;
    g->omega0 = d->omega0;
    g->domega = d->domega;
    g->dt = d->dt;
    g->shape = d->shape;
    g->shape_len = d->shape_len;
    g->precision = d->precision;
    g->cus = cus;
    g->C = tb.C;
    g->variant = tb.variant;
    g->domega = tb.domega;
    g->tile = default_tile(d->n_dir, d->n_omega, g->variant);
    g->const_k0 = d->n_omega;
    gt.resize((size_t)d->n_omega);
    for (int k = 0; k < d->n_omega; ++k) {
        const double gg = is_shape3(d->shape) ? 0.0 : shape_factor(d->shape, d->shape_len, tb.om[k]);
        gt[k] = make_float2((float)gg, (float)(1.0 - gg));
    }
    if (!is_shape3(d->shape)) {
        int k = d->n_omega - 1;
        while (k > 0 && gt[k - 1].x == gt[k].x && gt[k - 1].y == gt[k].y) --k;
        g->const_k0 = k;
        g->const_g = gt[d->n_omega - 1];
    }
}

}  // namespace

void rad::set_last_error(const char* msg) { t_last_error = msg ? msg : ""; }

extern "C" {

const char* rad_last_error(void) { return t_last_error.c_str(); }

int rad_device_cus(int32_t device)
{
    int n = 0;
    hipError_t e = hipGetDeviceCount(&n);
    if (e != hipSuccess) return hip_fail(e, "hipGetDeviceCount");
    if (device < 0 || device >= n) return fail(RAD_ERR_INVALID_ARG, "device %d out of range (%d devices)", device, n);
    int cus = 0;
    e = hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, device);
    if (e != hipSuccess) return hip_fail(e, "hipDeviceGetAttribute");
    return cus;
}

int rad_create_grid(rad_grid** out, const rad_grid_desc* d)
{
    if (!out || !d) return fail(RAD_ERR_INVALID_ARG, "out and desc must be non-NULL");
    GridTables tb;
    int vrc = prepare_tables(d, true, tb);
    if (vrc) return vrc;
    const int64_t points = (int64_t)d->n_dir * d->n_omega;
    std::vector<double>& dirs9 = tb.dirs9;
    const int cus = rad_device_cus(d->device);
    if (cus < 0) return cus;

    rad_grid* g = new rad_grid;
    std::vector<double>& om = tb.om;
    std::vector<float2> gt;
    describe_grid(g, d, tb, cus, gt);
    plan_parts(g);
    std::vector<float> g3;
    if (is_shape3(d->shape)) {
        g3.resize((size_t)points);
        for (int i = 0; i < d->n_dir; ++i)
            for (int k = 0; k < d->n_omega; ++k)
                g3[(size_t)i * d->n_omega + k] = (float)shape_factor3(d->shape, d->shape_len, d->dirs + 3 * i, om[k]);
    }

    DeviceGuard dg(g->device);
    if (int rs = scratch_setup(g->device)) {
        free_grid(g);
        return rs;
    }
    const size_t sbytes = (size_t)points * 4 * sizeof(double);
    if (hipMalloc(&g->d_dirs9, dirs9.size() * sizeof(double)) != hipSuccess ||
        hipMalloc(&g->d_omega, om.size() * sizeof(double)) != hipSuccess ||
        hipMalloc(&g->d_gtab, gt.size() * sizeof(float2)) != hipSuccess ||
        hipMalloc(&g->d_S, sbytes) != hipSuccess ||
        hipMalloc(&g->d_err, sizeof(int)) != hipSuccess ||
        hipMalloc(&g->d_out, (size_t)points * 6 * sizeof(double)) != hipSuccess ||
        (!g3.empty() && hipMalloc(&g->d_g3, g3.size() * sizeof(float)) != hipSuccess) ||
        (!tb.bstep.empty() && hipMalloc(&g->d_bstep, tb.bstep.size() * sizeof(double)) != hipSuccess)) {
        free_grid(g);
        return fail(RAD_ERR_OOM, "device allocation failed for a %lld-point grid", (long long)points);
    }
    int rc = ensure_partials(g);
    if (rc) { free_grid(g); return rc; }
    if (hipEventCreateWithFlags(&g->part_read[0].own, hipEventDisableTiming) != hipSuccess ||
        hipEventCreateWithFlags(&g->part_read[1].own, hipEventDisableTiming) != hipSuccess ||
        hipEventCreateWithFlags(&g->last_write.own, hipEventDisableTiming) != hipSuccess) {
        free_grid(g);
        return fail(RAD_ERR_DEVICE, "cannot create the grid's events");
    }
    hipError_t e;
    if ((e = hipMemcpy(g->d_dirs9, dirs9.data(), dirs9.size() * sizeof(double), hipMemcpyHostToDevice)) != hipSuccess ||
        (e = hipMemcpy(g->d_omega, om.data(), om.size() * sizeof(double), hipMemcpyHostToDevice)) != hipSuccess ||
        (e = hipMemcpy(g->d_gtab, gt.data(), gt.size() * sizeof(float2), hipMemcpyHostToDevice)) != hipSuccess ||
        (!g3.empty() && (e = hipMemcpy(g->d_g3, g3.data(), g3.size() * sizeof(float), hipMemcpyHostToDevice)) != hipSuccess) ||
        (!tb.bstep.empty() &&
         (e = hipMemcpy(g->d_bstep, tb.bstep.data(), tb.bstep.size() * sizeof(double), hipMemcpyHostToDevice)) != hipSuccess) ||
        (e = rad::launch_reset(g->d_S, points * 4, g->d_err, nullptr)) != hipSuccess ||
        (e = hipDeviceSynchronize()) != hipSuccess) {
        free_grid(g);
        return hip_fail(e, "grid initialisation");
    }
    stages().retain();
    g->counted = true;
    *out = g;
    return RAD_OK;
}

int rad_destroy_grid(rad_grid* g)
{
    if (!g) return RAD_OK;
    {
        DeviceGuard dg(g->device);
        (void)hipDeviceSynchronize();
    }
    free_grid(g);
    return RAD_OK;
}

int rad_reset(rad_grid* g, void* stream)
{
    if (!g) return fail(RAD_ERR_INVALID_ARG, "grid is NULL");
    DeviceGuard dg(g->device);
    if (int rc = refuse_capture((hipStream_t)stream, "rad_reset")) return rc;
    hipStream_t st = (hipStream_t)stream;
    RAD_HIP(order_after(g->last_write, st));
    hipError_t e = rad::launch_reset(g->d_S, (int64_t)g->n_dir * g->n_omega * 4, g->d_err, st);
    if (e == hipSuccess) e = mark_done(g->last_write, st);
    if (e != hipSuccess) return hip_fail(e, "reset");
    return RAD_OK;
}

int rad_push_step(rad_grid* g, double t, int64_t n_particles, const rad_particles* p, void* stream)
{
    if (!g) return fail(RAD_ERR_INVALID_ARG, "grid is NULL");
    if (n_particles < 0) return fail(RAD_ERR_INVALID_ARG, "n_particles < 0");
    if (!std::isfinite(t)) return fail(RAD_ERR_INVALID_ARG, "t is not finite");
    if (n_particles == 0) return RAD_OK;
    int rc = check_particles(p);
    if (rc) return rc;
    DeviceGuard dg(g->device);
    if ((rc = refuse_capture((hipStream_t)stream, "rad_push_step"))) return rc;
    return push_range(g, t, n_particles, n_particles, p, (hipStream_t)stream);
}

int rad_push_steps(rad_grid* g, double t0, int32_t n_steps, int64_t n_particles,
                   const rad_particles* p, void* stream)
{
    if (!g) return fail(RAD_ERR_INVALID_ARG, "grid is NULL");
    if (n_particles < 0 || n_steps < 0) return fail(RAD_ERR_INVALID_ARG, "negative size");
    if (!std::isfinite(t0)) return fail(RAD_ERR_INVALID_ARG, "t0 is not finite");
    if (n_particles == 0 || n_steps == 0) return RAD_OK;
    int rc = check_particles(p);
    if (rc) return rc;
    DeviceGuard dg(g->device);
    if ((rc = refuse_capture((hipStream_t)stream, "rad_push_steps"))) return rc;
    return push_range(g, t0, n_particles, (int64_t)n_steps * n_particles, p, (hipStream_t)stream);
}

int rad_push_step_noalloc(rad_grid* g, double t, int64_t n_particles, const rad_particles* p, void* stream)
{
    if (!g) return fail(RAD_ERR_INVALID_ARG, "grid is NULL");
    if (n_particles < 0) return fail(RAD_ERR_INVALID_ARG, "n_particles < 0");
    if (!std::isfinite(t)) return fail(RAD_ERR_INVALID_ARG, "t is not finite");
    if (n_particles == 0) return RAD_OK;
    int rc = check_particles(p);
    if (rc) return rc;
    const int64_t count = (int64_t)g->n_omega * g->n_dir * 4;        // FP32 values per split
    const int64_t grid_bytes = count * (int64_t)sizeof(float);
    if (grid_bytes > (int64_t)RAD_NOALLOC_SCRATCH_BYTES)
        return fail(RAD_ERR_INVALID_ARG,
                    "grid of %lld points needs %lld B of partial sums, more than the %zu B no-allocation "
                    "scratch (at most %zu points)", (long long)(count / 4), (long long)grid_bytes,
                    (size_t)RAD_NOALLOC_SCRATCH_BYTES, (size_t)RAD_NOALLOC_SCRATCH_BYTES / 16);
    DeviceGuard dg(g->device);
    float* scr = g->device >= 0 && g->device < kScratchDevices
                     ? g_scratch_addr[g->device].load(std::memory_order_acquire) : nullptr;
    if (!scr) return fail(RAD_ERR_DEVICE, "no-allocation scratch not set up on device %d", g->device);
    hipStream_t st = (hipStream_t)stream;
    // Under stream capture the call records no event and waits on none (a wait on an event
    // recorded outside the capture, or another stream waiting on the capture, would break
    // it): the caller orders the captured push against the grid's other work.
    hipError_t cap_err;
    const bool capturing = captures(st, &cap_err);
    RAD_HIP(cap_err);
    // every fold of this grid runs in issue order: the folds below come after every fold
    // already issued (on any stream), later folds, read-outs and resets after them
    if (!capturing) RAD_HIP(order_after(g->last_write, st));
    for (const GridPart& part : g->parts) {
        AccArgs a{};
        part_job(a.job, g, part, p, t, n_particles);
        a.part = scr;
        const int64_t cap = (int64_t)(RAD_NOALLOC_SCRATCH_BYTES / split_bytes(g, part));
        rc = for_each_launch(g, a, n_particles, std::min<int64_t>(max_splits(g, part), cap), part, [&]() -> int {
            // same stream: a launch's accumulate rewrites the scratch only after the previous
            // launch's fold has read it
            hipError_t e = launch_part(g, a, part, p->dtype, st);
            if (e != hipSuccess) return hip_fail(e, "accumulate launch");
            e = fold_part(g, a, part, st);
            if (e != hipSuccess) return hip_fail(e, "fold launch");
            return RAD_OK;
        });
        if (rc) return rc;
    }
    if (!capturing) RAD_HIP(mark_done(g->last_write, st));
    return RAD_OK;
}

int rad_spectrum_device(rad_grid* g, double* I_dev, void* stream)
{
    if (!g || !I_dev) return fail(RAD_ERR_INVALID_ARG, "grid and output must be non-NULL");
    DeviceGuard dg(g->device);
    if (int rc = refuse_capture((hipStream_t)stream, "rad_spectrum_device")) return rc;
    hipStream_t st = (hipStream_t)stream;
    RAD_HIP(order_after(g->last_write, st));
    hipError_t e = rad::launch_finalize(g->d_S, I_dev, g->n_dir, g->n_omega, g->C, g->d_err, nullptr, st);
    if (e != hipSuccess) return hip_fail(e, "finalize launch");
    // The read-out does not synchronise: later folds and resets, on any stream, must not
    // write S before it has been read, so the read-out becomes the grid's last-write mark.
    RAD_HIP(mark_done(g->last_write, st));
    return RAD_OK;
}

int rad_spectrum(rad_grid* g, double* I_host, void* stream)
{
    if (!g || !I_host) return fail(RAD_ERR_INVALID_ARG, "grid and output must be non-NULL");
    DeviceGuard dg(g->device);
    if (int rc = refuse_capture((hipStream_t)stream, "rad_spectrum")) return rc;
    return read_out(g, I_host, (size_t)g->n_dir * g->n_omega, (hipStream_t)stream, [&](double* out, int* flag_out, hipStream_t st) {
        return rad::launch_finalize(g->d_S, out, g->n_dir, g->n_omega, g->C, g->d_err, flag_out, st);
    });
}

int rad_spectrum_complex(rad_grid* g, double* S_host, void* stream)
{
    if (!g || !S_host) return fail(RAD_ERR_INVALID_ARG, "grid and output must be non-NULL");
    DeviceGuard dg(g->device);
    if (int rc = refuse_capture((hipStream_t)stream, "rad_spectrum_complex")) return rc;
    return read_out(g, S_host, (size_t)g->n_dir * g->n_omega * 6, (hipStream_t)stream, [&](double* out, int* flag_out, hipStream_t st) {
        return rad::launch_cartesian(g->d_S, g->d_dirs9, out, g->n_dir, g->n_omega, g->d_err, flag_out, st);
    });
}

size_t rad_state_size(const rad_grid* g)
{
    return g ? (size_t)g->n_dir * g->n_omega * 4 : 0;
}

int rad_get_state(rad_grid* g, double* state_host, void* stream)
{
    if (!g || !state_host) return fail(RAD_ERR_INVALID_ARG, "grid and state must be non-NULL");
    DeviceGuard dg(g->device);
    if (int rc = refuse_capture((hipStream_t)stream, "rad_get_state")) return rc;
    hipStream_t st = (hipStream_t)stream;
    RAD_HIP(order_after(g->last_write, st));
    int flag = 0;
    int rc = read_err_flag(g, st, &flag);
    if (rc) return rc;
    if (flag) return fail(RAD_ERR_BAD_DATA, "device detected invalid particle data");
    RAD_HIP(hipMemcpyAsync(state_host, g->d_S, rad_state_size(g) * sizeof(double), hipMemcpyDeviceToHost, st));
    RAD_HIP(hipStreamSynchronize(st));
    return RAD_OK;
}

int rad_set_state(rad_grid* g, const double* state_host, void* stream)
{
    if (!g || !state_host) return fail(RAD_ERR_INVALID_ARG, "grid and state must be non-NULL");
    DeviceGuard dg(g->device);
    if (int rc = refuse_capture((hipStream_t)stream, "rad_set_state")) return rc;
    hipStream_t st = (hipStream_t)stream;
    RAD_HIP(order_after(g->last_write, st));
    RAD_HIP(hipMemcpyAsync(g->d_S, state_host, rad_state_size(g) * sizeof(double), hipMemcpyHostToDevice, st));
    hipError_t e = rad::launch_reset(nullptr, 0, g->d_err, st);
    if (e != hipSuccess) return hip_fail(e, "set_state");
    RAD_HIP(hipStreamSynchronize(st));
    return RAD_OK;
}

int rad_grid_variant(const rad_grid* g)
{
    if (!g) return fail(RAD_ERR_INVALID_ARG, "grid is NULL");
    return g->variant;
}

int rad_get_tile(const rad_grid* g, rad_tile* t)
{
    if (!g || !t) return fail(RAD_ERR_INVALID_ARG, "grid and tile must be non-NULL");
    *t = g->tile;
    return RAD_OK;
}

int rad_set_tile(rad_grid* g, const rad_tile* t) { return change_tile(g, t, rad_grid::kTileSet); }

int rad_hint_tile(rad_grid* g, const rad_tile* t) { return change_tile(g, t, rad_grid::kTileHint); }

}  // extern "C"

#include "rad_debug.h"

extern "C" int rad_debug_plan(const rad_grid_desc* d, const rad_tile* tile, int32_t cus, int64_t n_particles,
                              rad_debug_launch* out, int32_t max_launches, int32_t* n_launches)
{
    if (!d || !n_launches || max_launches < 0 || (max_launches > 0 && !out) || cus < 1 || n_particles < 0)
        return fail(RAD_ERR_INVALID_ARG, "bad plan arguments");
    GridTables tb;
    if (int rc = prepare_tables(d, true, tb)) return rc;
    rad_grid g;
    std::vector<float2> gt;
    describe_grid(&g, d, tb, cus, gt);
    if (tile) {
        if (int rc = apply_tile(&g, *tile, rad_grid::kTileSet)) return rc;
    }
    plan_parts(&g);
    int32_t n = 0;
    for (const GridPart& part : g.parts) {
        AccArgs a{};
        for_each_launch(&g, a, n_particles, max_splits(&g, part), part, [&]() -> int {
            if (n < max_launches) {
                rad_debug_launch l{};
                l.kernel = part.matrix ? 2 : a.flex.groups ? 1 : 0;
                l.k0 = part.k0;
                l.n_omega = part.n;
                l.tile = part.tile;
                l.splits = a.splits;
                l.per_split = a.per_split;
                l.chunk = a.chunk;
                if (l.kernel == 1) {
                    l.weights_at = rad::flex_weights_at(a.flex.dirs, a.chunk);
                    l.lds_bytes = (int32_t)rad::flex_lds_bytes(a.flex, part.tile.w_per_lane, a.chunk);
                } else if (l.kernel == 0) {
                    l.lds_bytes = (int32_t)rad::acc_lds_bytes(shape_of(part.tile));
                }
                out[n] = l;
            }
            ++n;
            return RAD_OK;
        });
    }
    *n_launches = n;
    return RAD_OK;
}

extern "C" int rad_debug_trig_probe(const float* in_dev, float* out_dev, int n, void* stream)
{
    if (n < 0 || (n > 0 && (!in_dev || !out_dev))) return fail(RAD_ERR_INVALID_ARG, "bad probe arguments");
    hipError_t e = rad::launch_trig_probe(in_dev, out_dev, n, (hipStream_t)stream);
    if (e != hipSuccess) return hip_fail(e, "trig probe launch");
    return RAD_OK;
}

extern "C" int rad_profile_enable(rad_grid* g, int enable)
{
    if (!g) return fail(RAD_ERR_INVALID_ARG, "grid is NULL");
    DeviceGuard dg(g->device);
    release_events(g);
    g->prof_updates = 0;
    g->profiling = enable > 0;
    g->prof_period = enable > 0 ? enable : 1;
    g->prof_count = 0;
    return RAD_OK;
}

extern "C" int rad_profile_read(rad_grid* g, rad_profile_stats* out)
{
    if (!g || !out) return fail(RAD_ERR_INVALID_ARG, "grid and stats must be non-NULL");
    DeviceGuard dg(g->device);
    rad_profile_stats s{};
    for (auto& e : g->ev_acc) {
        RAD_HIP(hipEventSynchronize(e.second));
        float ms = 0.f;
        RAD_HIP(hipEventElapsedTime(&ms, e.first, e.second));
        s.accumulate_ms += ms;
        s.launches += 1;
    }
    for (auto& e : g->ev_fold) {
        RAD_HIP(hipEventSynchronize(e.second));
        float ms = 0.f;
        RAD_HIP(hipEventElapsedTime(&ms, e.first, e.second));
        s.fold_ms += ms;
    }
    s.updates = g->prof_updates;
    g->prof_updates = 0;
    release_events(g);
    *out = s;
    return RAD_OK;
}

// ---------------------------------------------------------------------------------------
// Batched launches over several grids.
// ---------------------------------------------------------------------------------------
#include <map>
#include <utility>

struct BatchGraphKey {
    int dtype, precision, w, dpw, waves, R, slot;
    bool operator==(const BatchGraphKey& o) const
    {
        return dtype == o.dtype && precision == o.precision && w == o.w && dpw == o.dpw && waves == o.waves &&
               R == o.R && slot == o.slot;
    }
};

struct BatchGraph {
    BatchGraphKey key;
    int64_t gen;
    hipGraphExec_t exec;
};

struct rad_batcher {
    int device = 0;
    int max_items = 0;
    int cus = 0;
    // Two plan buffers (pinned host + device); a plan buffer is rewritten only after the
    // launch that read it two pushes earlier has finished (event `done`).
    struct Slot {
        unsigned char* host = nullptr;
        unsigned char* dev = nullptr;
        size_t cap = 0;
        hipEvent_t done = nullptr;
        bool used = false;
    } slot[2];
    int next = 0;
    float* seg_part = nullptr;
    size_t seg_part_floats = 0;
    bool profiling = false;
    std::vector<std::pair<hipEvent_t, hipEvent_t>> ev_acc, ev_fold;
    std::vector<hipEvent_t> ev_pool;
    int64_t prof_updates = 0;
    // graph mode: captured [plan upload -> accumulate -> fold] per launch configuration
    bool tile_set = false;       // launch shape of the batched kernel (else the built-in
    rad_tile tile{};             // heuristic for the first item's grid shape)
    // A sum in registers covers at most this many chunks (0: no limit but the end of a workgroup's
    // range and of a tile).  The server sets it.
    int sum_chunks = 0;
    bool graph_mode = false;
    hipStream_t cap_stream = nullptr;
    std::vector<BatchGraph> graphs;
    int64_t graph_gen = 0;
    int64_t graph_launches = 0;
    int64_t graph_failures = 0;
};

namespace {

size_t align_up(size_t x, size_t a) { return (x + a - 1) / a * a; }

hipError_t batch_event(rad_batcher* b, hipEvent_t* ev)
{
    if (!b->ev_pool.empty()) {
        *ev = b->ev_pool.back();
        b->ev_pool.pop_back();
        return hipSuccess;
    }
    return hipEventCreate(ev);
}

void batch_release_events(rad_batcher* b)
{
    for (auto& e : b->ev_acc) { b->ev_pool.push_back(e.first); b->ev_pool.push_back(e.second); }
    for (auto& e : b->ev_fold) { b->ev_pool.push_back(e.first); b->ev_pool.push_back(e.second); }
    b->ev_acc.clear();
    b->ev_fold.clear();
}

void free_batcher(rad_batcher* b)
{
    if (!b) return;
    DeviceGuard dg(b->device);
    for (auto& s : b->slot) {
        if (s.done) (void)hipEventSynchronize(s.done);
        if (s.host) (void)hipHostFree(s.host);
        if (s.dev) (void)hipFree(s.dev);
        if (s.done) (void)hipEventDestroy(s.done);
    }
    if (b->seg_part) (void)hipFree(b->seg_part);
    for (auto& ge : b->graphs) (void)hipGraphExecDestroy(ge.exec);
    b->graphs.clear();
    if (b->cap_stream) (void)hipStreamDestroy(b->cap_stream);
    batch_release_events(b);
    for (hipEvent_t e : b->ev_pool) (void)hipEventDestroy(e);
    delete b;
}

struct ItemInfo {
    rad::Job job;
    int64_t chunks = 0;
    int64_t iters = 0;     // tiles * chunks
    int64_t iter_begin = 0;
    rad_grid* grid = nullptr;
};

// One launch's plan over the global iteration range [L0, L1).
struct LaunchPlan {
    std::vector<int32_t> wg_seg_begin;
    std::vector<rad::BatchSeg> segs;
    std::vector<rad::FoldJob> jobs;
    std::vector<int32_t> seg_list;
};

void build_plan(const std::vector<ItemInfo>& items, int64_t L0, int64_t L1, int R, LaunchPlan& pl)
{
    pl = LaunchPlan{};
    const int64_t I = L1 - L0;
    size_t it = 0;
    while (it < items.size() && items[it].iter_begin + items[it].iters <= L0) ++it;
    for (int r = 0; r < R; ++r) {
        pl.wg_seg_begin.push_back((int32_t)pl.segs.size());
        int64_t pos = L0 + I * r / R;
        const int64_t end = L0 + I * (r + 1) / R;
        while (pos < end) {
            while (items[it].iter_begin + items[it].iters <= pos) ++it;
            const ItemInfo& in = items[it];
            const int64_t local = pos - in.iter_begin;
            const int64_t tile = local / in.chunks;
            const int64_t c0 = local % in.chunks;
            const int64_t seg_end = std::min(end, in.iter_begin + (tile + 1) * in.chunks);
            pl.segs.push_back(rad::BatchSeg{(int32_t)it, (int32_t)tile, c0, c0 + (seg_end - pos)});
            pos = seg_end;
        }
    }
    pl.wg_seg_begin.push_back((int32_t)pl.segs.size());
    // fold jobs keyed by (grid, tile), segments listed in segment order.  The tile index is
    // in the batch's launch shape (the items' jobs), not the grid's own single-push shape.
    std::map<std::pair<const rad_grid*, int>, std::vector<int32_t>> groups;
    std::vector<std::pair<const rad_grid*, int>> order;
    std::vector<int> order_tiles_d;
    for (size_t sidx = 0; sidx < pl.segs.size(); ++sidx) {
        const auto& sg = pl.segs[sidx];
        auto key = std::make_pair((const rad_grid*)items[sg.item].grid, (int)sg.tile);
        auto f = groups.find(key);
        if (f == groups.end()) {
            order.push_back(key);
            order_tiles_d.push_back(items[sg.item].job.tiles_d);
            groups[key].push_back((int32_t)sidx);
        } else {
            f->second.push_back((int32_t)sidx);
        }
    }
    for (size_t oi = 0; oi < order.size(); ++oi) {
        const auto& key = order[oi];
        const rad_grid* g = key.first;
        const int tdn = order_tiles_d[oi];
        rad::FoldJob fj{};
        fj.S = g->d_S;
        fj.n_dir = g->n_dir;
        fj.n_omega = g->n_omega;
        fj.td = key.second % tdn;
        fj.tw = key.second / tdn;
        fj.list_begin = (int32_t)pl.seg_list.size();
        for (int32_t sidx : groups[key]) pl.seg_list.push_back(sidx);
        fj.list_end = (int32_t)pl.seg_list.size();
        pl.jobs.push_back(fj);
    }
}

}  // namespace

extern "C" int rad_batcher_create(rad_batcher** out, int32_t device, int32_t max_items)
{
    if (!out) return fail(RAD_ERR_INVALID_ARG, "out is NULL");
    if (max_items < 1 || max_items > (1 << 20)) return fail(RAD_ERR_INVALID_ARG, "max_items must be in 1..2^20");
    const int cus = rad_device_cus(device);
    if (cus < 0) return cus;
    rad_batcher* b = new rad_batcher;
    b->device = device;
    b->max_items = max_items;
    b->cus = cus;
    DeviceGuard dg(device);
    for (auto& s : b->slot) {
        if (hipEventCreateWithFlags(&s.done, hipEventDisableTiming) != hipSuccess) {
            free_batcher(b);
            return fail(RAD_ERR_DEVICE, "cannot create batcher events");
        }
    }
    *out = b;
    return RAD_OK;
}

extern "C" int rad_batcher_destroy(rad_batcher* b)
{
    if (!b) return RAD_OK;
    {
        DeviceGuard dg(b->device);
        (void)hipDeviceSynchronize();
    }
    free_batcher(b);
    return RAD_OK;
}

void rad::batcher_limit_sums(rad_batcher* b, int chunks) { b->sum_chunks = chunks; }

extern "C" int rad_batcher_push(rad_batcher* b, const rad_batch_item* items, int32_t n_items, void* stream)
{
    if (!b) return fail(RAD_ERR_INVALID_ARG, "batcher is NULL");
    if (n_items < 0 || n_items > b->max_items)
        return fail(RAD_ERR_INVALID_ARG, "n_items %d outside 0..%d", n_items, b->max_items);
    if (n_items > 0 && !items) return fail(RAD_ERR_INVALID_ARG, "items is NULL");
    // validation
    std::vector<ItemInfo> info;
    std::vector<const rad_particles*> items_p;
    const rad_grid* g0 = nullptr;
    int dtype = -1;
    for (int32_t i = 0; i < n_items; ++i) {
        const rad_batch_item& itm = items[i];
        if (!itm.grid) return fail(RAD_ERR_INVALID_ARG, "item %d has no grid", i);
        if (itm.n_steps < 0 || itm.n_particles < 0) return fail(RAD_ERR_INVALID_ARG, "item %d has a negative size", i);
        if (!std::isfinite(itm.t0)) return fail(RAD_ERR_INVALID_ARG, "item %d: t0 is not finite", i);
        if (itm.grid->device != b->device)
            return fail(RAD_ERR_INVALID_ARG, "item %d: grid on device %d, batcher on %d", i, itm.grid->device, b->device);
        if (itm.n_steps == 0 || itm.n_particles == 0) continue;
        int rc = check_particles(&itm.p);
        if (rc) return rc;
        if (!g0) {
            g0 = itm.grid;
            dtype = itm.p.dtype;
        }
        if (itm.p.dtype != dtype) return fail(RAD_ERR_INVALID_ARG, "item %d: particle dtype differs within the batch", i);
        if (itm.grid->precision != g0->precision) return fail(RAD_ERR_INVALID_ARG, "item %d: precision mode differs", i);
        if (itm.grid->variant != g0->variant)
            return fail(RAD_ERR_INVALID_ARG, "item %d: frequency-list / 3-D-shape kind differs within the batch", i);
        ItemInfo in;
        in.grid = itm.grid;
        in.job.i_begin = 0;
        in.job.i_end = (int64_t)itm.n_steps * itm.n_particles;
        in.job.n_per_step = itm.n_particles;
        in.job.t0 = itm.t0;
        in.chunks = (in.job.i_end + rad::kChunk - 1) / rad::kChunk;
        info.push_back(in);
        items_p.push_back(&itm.p);
    }
    if (info.empty()) return RAD_OK;
    const rad_tile btile = b->tile_set ? b->tile : batch_tile(g0->n_dir, g0->n_omega, g0->variant);
    if (g0->variant != 0 && btile.w_per_lane != 16)
        return fail(RAD_ERR_INVALID_ARG, "batches of grids with a frequency list or a 3-D shape need w_per_lane = 16");
    for (size_t i = 0; i < info.size(); ++i) {
        ItemInfo& in = info[i];
        const int64_t i_end = in.job.i_end, nps = in.job.n_per_step;
        const double t0 = in.job.t0;
        fill_job(in.job, in.grid, items_p[i], t0, nps, btile);
        in.job.i_begin = 0;
        in.job.i_end = i_end;
        in.iters = in.chunks * (int64_t)in.job.tiles_d * in.job.tiles_w;
    }
    DeviceGuard dg(b->device);
    hipStream_t st = (hipStream_t)stream;
    if (int rc = refuse_capture(st, "rad_batcher_push")) return rc;
    // earlier single-grid folds of these grids must land before the batch fold
    {
        std::vector<rad_grid*> seen;
        for (const auto& in : info) {
            if (std::find(seen.begin(), seen.end(), in.grid) != seen.end()) continue;
            seen.push_back(in.grid);
            RAD_HIP(order_after(in.grid->last_write, st));
        }
    }
    int64_t I = 0;
    for (auto& in : info) {
        in.iter_begin = I;
        I += in.iters;
    }
    const LaunchShape ls = shape_of(btile, g0->variant);
    const int TD = rad::tile_dirs(ls), TO = rad::tile_omegas(ls);
    const int R_target = std::max(1, b->cus * btile.wg_per_cu);
    const int64_t per_launch = (int64_t)R_target * (kMaxPerWorkgroup / rad::kChunk);
    bool launched = false;
    for (int64_t L0 = 0; L0 < I; L0 += per_launch) {
        const int64_t L1 = std::min(I, L0 + per_launch);
        const int R = (int)std::min<int64_t>(R_target, L1 - L0);
        LaunchPlan pl;
        build_plan(info, L0, L1, R, pl);
        // Plan layout: header {n_items, n_segs, n_jobs, R} | items | wg_seg_begin | segs |
        // jobs | seg_list.  In graph mode the capacities (and the launched grid) are fixed
        // so one captured graph serves every plan that fits.
        const int R_fixed = R_target;
        const size_t segs_cap_g = (size_t)R_fixed + 16 * (size_t)b->max_items;
        bool use_graph = b->graph_mode && pl.segs.size() <= segs_cap_g && pl.jobs.size() <= segs_cap_g &&
                         pl.seg_list.size() <= segs_cap_g;
        const int R_launch = use_graph ? R_fixed : R;
        const size_t items_cap = use_graph ? (size_t)b->max_items : info.size();
        const size_t segs_cap = use_graph ? segs_cap_g : pl.segs.size();
        const size_t jobs_cap = use_graph ? segs_cap_g : pl.jobs.size();
        const size_t list_cap = use_graph ? segs_cap_g : pl.seg_list.size();
        const size_t o_hdr = 0;
        const size_t o_items = 16;
        const size_t o_wsb = align_up(o_items + items_cap * sizeof(rad::Job), 16);
        const size_t o_segs = align_up(o_wsb + ((size_t)R_launch + 1) * sizeof(int32_t), 16);
        const size_t o_jobs = align_up(o_segs + segs_cap * sizeof(rad::BatchSeg), 16);
        const size_t o_list = align_up(o_jobs + jobs_cap * sizeof(rad::FoldJob), 16);
        const size_t bytes = align_up(o_list + list_cap * sizeof(int32_t), 16);
        const int slot_index = b->next;
        auto& sl = b->slot[slot_index];
        b->next ^= 1;
        if (sl.used) RAD_HIP(hipEventSynchronize(sl.done));
        if (bytes > sl.cap) {
            if (sl.host) RAD_HIP(hipHostFree(sl.host));
            if (sl.dev) RAD_HIP(hipFree(sl.dev));
            sl.host = nullptr;
            sl.dev = nullptr;
            sl.cap = 0;
            const size_t cap = std::max<size_t>(bytes * 2, 64 * 1024);
            if (hipHostMalloc((void**)&sl.host, cap, hipHostMallocDefault) != hipSuccess ||
                hipMalloc((void**)&sl.dev, cap) != hipSuccess)
                return fail(RAD_ERR_OOM, "cannot allocate a %zu B batch plan", cap);
            sl.cap = cap;
            b->graph_gen += 1;   // captured graphs refer to the old buffers
        }
        const int32_t hdr[4] = {(int32_t)info.size(), (int32_t)pl.segs.size(), (int32_t)pl.jobs.size(), (int32_t)R};
        std::memcpy(sl.host + o_hdr, hdr, sizeof(hdr));
        for (size_t i = 0; i < info.size(); ++i) std::memcpy(sl.host + o_items + i * sizeof(rad::Job), &info[i].job, sizeof(rad::Job));
        {
            int32_t* wsb = reinterpret_cast<int32_t*>(sl.host + o_wsb);
            std::memcpy(wsb, pl.wg_seg_begin.data(), pl.wg_seg_begin.size() * sizeof(int32_t));
            for (int r = R + 1; r <= R_launch; ++r) wsb[r] = (int32_t)pl.segs.size();   // idle workgroups
        }
        std::memcpy(sl.host + o_segs, pl.segs.data(), pl.segs.size() * sizeof(rad::BatchSeg));
        std::memcpy(sl.host + o_jobs, pl.jobs.data(), pl.jobs.size() * sizeof(rad::FoldJob));
        std::memcpy(sl.host + o_list, pl.seg_list.data(), pl.seg_list.size() * sizeof(int32_t));
        // segment scratch
        const size_t need = segs_cap * (size_t)TD * TO * 4;
        if (need > b->seg_part_floats) {
            if (b->seg_part) {
                RAD_HIP(hipDeviceSynchronize());
                RAD_HIP(hipFree(b->seg_part));
                b->seg_part = nullptr;
                b->seg_part_floats = 0;
            }
            const size_t alloc = need + need / 4;
            if (hipMalloc((void**)&b->seg_part, alloc * sizeof(float)) != hipSuccess)
                return fail(RAD_ERR_OOM, "cannot allocate %zu B of batch partial sums", alloc * sizeof(float));
            b->seg_part_floats = alloc;
            b->graph_gen += 1;
        }
        const rad::Job* d_items = reinterpret_cast<const rad::Job*>(sl.dev + o_items);
        const int32_t* d_wsb = reinterpret_cast<const int32_t*>(sl.dev + o_wsb);
        const rad::BatchSeg* d_segs = reinterpret_cast<const rad::BatchSeg*>(sl.dev + o_segs);
        const int32_t* d_njobs = reinterpret_cast<const int32_t*>(sl.dev + o_hdr) + 2;
        const rad::FoldJob* d_jobs = reinterpret_cast<const rad::FoldJob*>(sl.dev + o_jobs);
        const int32_t* d_list = reinterpret_cast<const int32_t*>(sl.dev + o_list);
        hipGraphExec_t exec = nullptr;
        if (use_graph) {
            const BatchGraphKey key{dtype, g0->precision * 16 + ls.variant, ls.w_per_lane, ls.dir_per_wave, ls.waves,
                                    R_launch, slot_index};
            for (auto& ge : b->graphs)
                if (ge.key == key && ge.gen == b->graph_gen) exec = ge.exec;
            if (!exec) {
                // capture [plan upload -> persistent accumulate -> fold] on the batcher's own stream
                hipGraph_t graph = nullptr;
                hipError_t e = rad::prepare_accumulate_batch(b->sum_chunks, dtype, g0->precision, ls);
                if (e == hipSuccess) e = hipStreamBeginCapture(b->cap_stream, hipStreamCaptureModeThreadLocal);
                if (e == hipSuccess) {
                    hipError_t e1 = hipMemcpyAsync(sl.dev, sl.host, bytes, hipMemcpyHostToDevice, b->cap_stream);
                    if (e1 == hipSuccess)
                        e1 = rad::launch_accumulate_batch(d_items, d_wsb, d_segs, b->seg_part, b->sum_chunks, dtype,
                                                          g0->precision, ls, R_launch, b->cap_stream);
                    if (e1 == hipSuccess)
                        e1 = rad::launch_fold_batch(d_njobs, d_jobs, (int)jobs_cap, d_list, b->seg_part, TD, TO,
                                                    b->cap_stream);
                    hipError_t e2 = hipStreamEndCapture(b->cap_stream, &graph);
                    e = e1 != hipSuccess ? e1 : e2;
                }
                if (e == hipSuccess) e = hipGraphInstantiate(&exec, graph, nullptr, nullptr, 0);
                if (graph) (void)hipGraphDestroy(graph);
                if (e != hipSuccess) {
                    (void)hipGetLastError();
                    exec = nullptr;
                    b->graph_mode = false;   // fall back to direct launches from now on
                    b->graph_failures += 1;
                } else {
                    b->graphs.push_back(BatchGraph{key, b->graph_gen, exec});
                }
            }
            use_graph = exec != nullptr;
        }
        hipEvent_t e0 = nullptr, e1 = nullptr, e2 = nullptr, e3 = nullptr;
        if (b->profiling) {
            RAD_HIP(batch_event(b, &e0));
            RAD_HIP(batch_event(b, &e1));
            RAD_HIP(batch_event(b, &e2));
            RAD_HIP(batch_event(b, &e3));
            b->ev_acc.emplace_back(e0, e1);
            b->ev_fold.emplace_back(e2, e3);
            for (const auto& sg : pl.segs) {
                const ItemInfo& in = info[sg.item];
                const int64_t lo = sg.c_begin * rad::kChunk;
                const int64_t hi = std::min(in.job.i_end, sg.c_end * rad::kChunk);
                const int td = sg.tile % in.job.tiles_d, tw = sg.tile / in.job.tiles_d;
                const int64_t nd = std::min(TD, in.job.n_dir - td * TD);
                const int64_t no = std::min(TO, in.job.n_omega - tw * TO);
                b->prof_updates += (hi - lo) * nd * no;   // in-grid terms only
            }
        }
        if (use_graph) {
            // timing of a replay covers the whole graph (upload, accumulate and fold)
            if (b->profiling) RAD_HIP(hipEventRecord(e0, st));
            RAD_HIP(hipGraphLaunch(exec, st));
            b->graph_launches += 1;
            if (b->profiling) {
                RAD_HIP(hipEventRecord(e1, st));
                RAD_HIP(hipEventRecord(e2, st));
                RAD_HIP(hipEventRecord(e3, st));
            }
        } else {
            RAD_HIP(hipMemcpyAsync(sl.dev, sl.host, bytes, hipMemcpyHostToDevice, st));
            if (b->profiling) RAD_HIP(hipEventRecord(e0, st));
            hipError_t e = rad::launch_accumulate_batch(d_items, d_wsb, d_segs, b->seg_part, b->sum_chunks, dtype,
                                                        g0->precision, ls, R_launch, st);
            if (e != hipSuccess) return hip_fail(e, "batch accumulate launch");
            if (b->profiling) {
                RAD_HIP(hipEventRecord(e1, st));
                RAD_HIP(hipEventRecord(e2, st));
            }
            e = rad::launch_fold_batch(d_njobs, d_jobs, (int)jobs_cap, d_list, b->seg_part, TD, TO, st);
            if (e != hipSuccess) return hip_fail(e, "batch fold launch");
            if (b->profiling) RAD_HIP(hipEventRecord(e3, st));
        }
        RAD_HIP(hipEventRecord(sl.done, st));
        sl.used = true;
        launched = true;
    }
    // Later single-grid folds (on whatever stream pushes them), resets and read-outs must
    // come after this batch's fold.
    if (launched) {
        std::vector<rad_grid*> seen;
        for (const auto& in : info) {
            rad_grid* g = in.grid;
            if (std::find(seen.begin(), seen.end(), g) != seen.end()) continue;
            seen.push_back(g);
            RAD_HIP(mark_done(g->last_write, st));
        }
    }
    return RAD_OK;
}

extern "C" int rad_batcher_profile_enable(rad_batcher* b, int enable)
{
    if (!b) return fail(RAD_ERR_INVALID_ARG, "batcher is NULL");
    batch_release_events(b);
    b->prof_updates = 0;
    b->profiling = enable != 0;
    return RAD_OK;
}

extern "C" int rad_batcher_profile_read(rad_batcher* b, rad_profile_stats* out)
{
    if (!b || !out) return fail(RAD_ERR_INVALID_ARG, "batcher and stats must be non-NULL");
    DeviceGuard dg(b->device);
    rad_profile_stats s{};
    for (auto& e : b->ev_acc) {
        RAD_HIP(hipEventSynchronize(e.second));
        float ms = 0.f;
        RAD_HIP(hipEventElapsedTime(&ms, e.first, e.second));
        s.accumulate_ms += ms;
        s.launches += 1;
    }
    for (auto& e : b->ev_fold) {
        RAD_HIP(hipEventSynchronize(e.second));
        float ms = 0.f;
        RAD_HIP(hipEventElapsedTime(&ms, e.first, e.second));
        s.fold_ms += ms;
    }
    s.updates = b->prof_updates;
    b->prof_updates = 0;
    batch_release_events(b);
    *out = s;
    return RAD_OK;
}

extern "C" int rad_batcher_set_graph(rad_batcher* b, int enable)
{
    if (!b) return fail(RAD_ERR_INVALID_ARG, "batcher is NULL");
    DeviceGuard dg(b->device);
    if (enable && !b->cap_stream) {
        if (hipStreamCreateWithFlags(&b->cap_stream, hipStreamNonBlocking) != hipSuccess)
            return fail(RAD_ERR_DEVICE, "cannot create the capture stream");
    }
    b->graph_mode = enable != 0;
    return RAD_OK;
}

extern "C" int rad_batcher_graph_stats(rad_batcher* b, int64_t* graphs, int64_t* launches, int64_t* failures)
{
    if (!b) return fail(RAD_ERR_INVALID_ARG, "batcher is NULL");
    if (graphs) *graphs = (int64_t)b->graphs.size();
    if (launches) *launches = b->graph_launches;
    if (failures) *failures = b->graph_failures;
    return RAD_OK;
}

extern "C" int rad_batcher_set_tile(rad_batcher* b, const rad_tile* t)
{
    if (!b) return fail(RAD_ERR_INVALID_ARG, "batcher is NULL");
    if (!t) {
        b->tile_set = false;
        return RAD_OK;
    }
    int rc = validate_tile(*t);
    if (rc) return rc;
    b->tile = *t;
    b->tile_set = true;
    return RAD_OK;
}

extern "C" int rad_batcher_get_tile(rad_batcher* b, rad_tile* t)
{
    if (!b || !t) return fail(RAD_ERR_INVALID_ARG, "batcher and tile must be non-NULL");
    if (!b->tile_set) return fail(RAD_ERR_INVALID_ARG, "no launch shape set (the heuristic for the first item's grid is used)");
    *t = b->tile;
    return RAD_OK;
}

// ---------------------------------------------------------------------------------------
// Post-processing variant: tracked particles with per-particle time integrals.
// ---------------------------------------------------------------------------------------
struct rad_tracked {
    int device = 0;
    int64_t n_particles = 0;
    int n_dir = 0, n_omega = 0;
    double domega = 0, dt = 0, C = 0;
    bool direct = false;
    std::vector<double> dirs, om;
    double* d_dirs9 = nullptr;
    double* d_omega = nullptr;
    double* d_T = nullptr;
    // d_T holds zeros when the work issued so far has run: the next push need not read it.
    // What a captured graph does to it is not seen here, so a capture ends the use of this.
    bool T_zero = false;
    bool captured = false;
    double* d_wg = nullptr;    // n_particles weights, then up to n_dir * n_omega shape factors
    double* d_I = nullptr;
    bool counted = false;      // among the users of the read-out buffers
    int* d_err = nullptr;
};

namespace {

void free_tracked(rad_tracked* tr)
{
    if (!tr) return;
    DeviceGuard dg(tr->device);
    for (double* p : {tr->d_dirs9, tr->d_omega, tr->d_T, tr->d_wg, tr->d_I})
        if (p) (void)hipFree(p);
    if (tr->d_err) (void)hipFree(tr->d_err);
    if (tr->counted) stages().drop();
    delete tr;
}

}  // namespace

extern "C" int rad_tracked_create(rad_tracked** out, const rad_grid_desc* d, int64_t n_particles)
{
    if (!out || !d) return fail(RAD_ERR_INVALID_ARG, "out and desc must be non-NULL");
    if (n_particles < 1) return fail(RAD_ERR_INVALID_ARG, "need n_particles >= 1");
    if (d->precision != RAD_PHASE_F64) return fail(RAD_ERR_INVALID_ARG, "tracked particles use the FP64-phase mode");
    GridTables tb;
    int rc = prepare_tables(d, false, tb);
    if (rc) return rc;
    const int64_t points = (int64_t)d->n_dir * d->n_omega;
    // 32 B per particle and grid point; refuse sizes whose byte count would not fit
    if (n_particles > ((int64_t)1 << 50) / (points * 32))
        return fail(RAD_ERR_INVALID_ARG, "%lld tracked particles x %lld points is too large",
                    (long long)n_particles, (long long)points);
    rad_tracked* tr = new rad_tracked;
    tr->device = d->device;
    tr->n_particles = n_particles;
    tr->n_dir = d->n_dir;
    tr->n_omega = d->n_omega;
    tr->domega = tb.domega;
    tr->dt = d->dt;
    tr->C = tb.C;
    // any non-uniform list takes the per-term phase here (tracked sets are small)
    tr->direct = (tb.variant & (rad::kVarDirect | rad::kVarBlockStep)) != 0;
    if (tr->direct) tr->domega = 0.0;
    tr->dirs.assign(d->dirs, d->dirs + 3 * (size_t)d->n_dir);
    tr->om = tb.om;
    DeviceGuard dg(d->device);
    const size_t tbytes = (size_t)n_particles * points * 4 * sizeof(double);
    if (hipMalloc(&tr->d_dirs9, tb.dirs9.size() * sizeof(double)) != hipSuccess ||
        hipMalloc(&tr->d_omega, tb.om.size() * sizeof(double)) != hipSuccess ||
        hipMalloc(&tr->d_T, tbytes) != hipSuccess ||
        hipMalloc(&tr->d_wg, ((size_t)n_particles + points) * sizeof(double)) != hipSuccess ||
        hipMalloc(&tr->d_I, (size_t)points * sizeof(double)) != hipSuccess ||
        hipMalloc(&tr->d_err, sizeof(int)) != hipSuccess) {
        free_tracked(tr);
        return fail(RAD_ERR_OOM, "cannot allocate %zu B of per-particle integrals", tbytes);
    }
    hipError_t e;
    if ((e = hipMemcpy(tr->d_dirs9, tb.dirs9.data(), tb.dirs9.size() * sizeof(double), hipMemcpyHostToDevice)) != hipSuccess ||
        (e = hipMemcpy(tr->d_omega, tb.om.data(), tb.om.size() * sizeof(double), hipMemcpyHostToDevice)) != hipSuccess ||
        (e = rad::launch_reset(tr->d_T, (int64_t)(tbytes / sizeof(double)), tr->d_err, nullptr)) != hipSuccess || (e = hipDeviceSynchronize()) != hipSuccess) {
        free_tracked(tr);
        return hip_fail(e, "tracked initialisation");
    }
    stages().retain();
    tr->counted = true;
    tr->T_zero = true;
    *out = tr;
    return RAD_OK;
}

extern "C" int rad_tracked_destroy(rad_tracked* tr)
{
    if (!tr) return RAD_OK;
    {
        DeviceGuard dg(tr->device);
        (void)hipDeviceSynchronize();
    }
    free_tracked(tr);
    return RAD_OK;
}

namespace {

int note_capture(rad_tracked* tr, hipStream_t st)
{
    hipError_t e;
    const bool capturing = captures(st, &e);
    RAD_HIP(e);
    if (capturing) {
        tr->captured = true;
        tr->T_zero = false;
    }
    return RAD_OK;
}

}  // namespace

extern "C" int rad_tracked_reset(rad_tracked* tr, void* stream)
{
    if (!tr) return fail(RAD_ERR_INVALID_ARG, "tracked is NULL");
    DeviceGuard dg(tr->device);
    hipStream_t st = (hipStream_t)stream;
    hipError_t e = rad::launch_reset(tr->d_T, tr->n_particles * tr->n_dir * tr->n_omega * 4, tr->d_err, st);
    if (e != hipSuccess) return hip_fail(e, "tracked reset");
    if (int rc = note_capture(tr, st)) return rc;
    tr->T_zero = !tr->captured;
    return RAD_OK;
}

namespace {

int tracked_push(rad_tracked* tr, double t0, int32_t n_steps, const rad_particles* p, void* stream)
{
    if (!tr) return fail(RAD_ERR_INVALID_ARG, "tracked is NULL");
    if (!std::isfinite(t0)) return fail(RAD_ERR_INVALID_ARG, "t is not finite");
    if (n_steps < 0) return fail(RAD_ERR_INVALID_ARG, "negative step count");
    if (!p) return fail(RAD_ERR_INVALID_ARG, "particles is NULL");
    if (n_steps == 0) return RAD_OK;
    rad_particles q = *p;
    if (!q.w) q.w = q.x;   // the weight field is not read here
    int rc = check_particles(&q);
    if (rc) return rc;
    DeviceGuard dg(tr->device);
    rad::TrackedArgs a{};
    a.f[0] = p->x; a.f[1] = p->y; a.f[2] = p->z;
    a.f[3] = p->bx; a.f[4] = p->by; a.f[5] = p->bz;
    a.f[6] = p->dbx; a.f[7] = p->dby; a.f[8] = p->dbz; a.f[9] = nullptr;
    a.n_particles = tr->n_particles;
    a.t = t0;
    a.dt = tr->dt;
    a.n_steps = n_steps;
    a.dirs9 = tr->d_dirs9;
    a.omega = tr->d_omega;
    a.domega = tr->domega;
    if ((rc = note_capture(tr, (hipStream_t)stream))) return rc;
    a.T = tr->d_T;
    a.T_zero = tr->T_zero;
    tr->T_zero = false;
    a.err = tr->d_err;
    a.n_dir = tr->n_dir;
    a.n_omega = tr->n_omega;
    hipError_t e = rad::launch_tracked_accumulate(a, p->dtype, tr->direct, (hipStream_t)stream);
    if (e != hipSuccess) return hip_fail(e, "tracked accumulate launch");
    return RAD_OK;
}

}  // namespace

extern "C" int rad_tracked_push_step(rad_tracked* tr, double t, const rad_particles* p, void* stream)
{
    return tracked_push(tr, t, 1, p, stream);
}

namespace rad {
int tracked_step_group();   // rad_kernels.hip
}

extern "C" int rad_tracked_step_group(void) { return rad::tracked_step_group(); }

extern "C" int rad_tracked_push_steps(rad_tracked* tr, double t0, int32_t n_steps, const rad_particles* p,
                                      void* stream)
{
    return tracked_push(tr, t0, n_steps, p, stream);
}

extern "C" int rad_tracked_spectrum(rad_tracked* tr, const double* weights_host, int32_t shape, double shape_len,
                                    double* I_host, void* stream)
{
    if (!tr || !weights_host || !I_host) return fail(RAD_ERR_INVALID_ARG, "NULL argument");
    if (shape < RAD_SHAPE_POINT || shape > RAD_SHAPE_QSC3D) return fail(RAD_ERR_INVALID_ARG, "unknown shape %d", shape);
    if (shape != RAD_SHAPE_POINT && !(shape_len > 0.0 && std::isfinite(shape_len)))
        return fail(RAD_ERR_INVALID_ARG, "shape_len must be finite and > 0");
    for (int64_t m = 0; m < tr->n_particles; ++m)
        if (!(weights_host[m] >= 0.0) || !std::isfinite(weights_host[m]))
            return fail(RAD_ERR_INVALID_ARG, "weight %lld must be finite and >= 0", (long long)m);
    DeviceGuard dg(tr->device);
    hipStream_t st = (hipStream_t)stream;
    if (int rc = refuse_capture(st, "rad_tracked_spectrum")) return rc;
    const bool s3 = is_shape3(shape);
    // weights, then the shape factors, as the device buffer holds them
    const size_t points = (size_t)tr->n_dir * tr->n_omega, n_g = s3 ? points : (size_t)tr->n_omega;
    const size_t in_bytes = ((size_t)tr->n_particles + n_g) * sizeof(double), out_bytes = points * sizeof(double);
    auto inputs = [&](double* dst) {
        std::memcpy(dst, weights_host, (size_t)tr->n_particles * sizeof(double));
        double* g = dst + tr->n_particles;
        for (int d = 0; d < (s3 ? tr->n_dir : 1); ++d)
            for (int k = 0; k < tr->n_omega; ++k)
                g[(size_t)d * tr->n_omega + k] = s3 ? shape_factor3(shape, shape_len, tr->dirs.data() + 3 * d, tr->om[k])
                                                    : shape_factor(shape, shape_len, tr->om[k]);
    };
    const double* d_g = tr->d_wg + tr->n_particles;
    auto launch = [&](double* out, int* flag_out) {
        return rad::launch_tracked_finalize(tr->d_T, tr->d_wg, s3 ? nullptr : d_g, s3 ? d_g : nullptr, tr->n_particles,
                                            tr->n_dir, tr->n_omega, tr->C, out, tr->d_err, flag_out, st);
    };
    // Up to kMaxStageBytes the inputs leave from one page-locked buffer in one copy, and the
    // flag and the result come back in it; the result by way of device memory, since its
    // writes are single values (see k_tracked_finalize).
    StagePool::Stage sg;
    const size_t in_place = kStageHeader + (out_bytes + 255) / 256 * 256;
    if (in_place + in_bytes <= kMaxStageBytes && stages().take(in_place + in_bytes, &sg) == hipSuccess) {
        inputs(reinterpret_cast<double*>(sg.host + in_place));
        hipError_t e = hipMemcpyAsync(tr->d_wg, sg.host + in_place, in_bytes, hipMemcpyHostToDevice, st);
        if (e == hipSuccess) e = launch(tr->d_I, reinterpret_cast<int*>(sg.dev));
        if (e == hipSuccess) e = hipMemcpyAsync(sg.host + kStageHeader, tr->d_I, out_bytes, hipMemcpyDeviceToHost, st);
        if (e == hipSuccess) e = hipStreamSynchronize(st);
        if (e != hipSuccess) return hip_fail(e, "tracked read-out");
        const bool bad = *sg.flag() != 0;
        if (!bad) std::memcpy(I_host, sg.host + kStageHeader, out_bytes);
        stages().give_back(sg);
        return bad ? fail(RAD_ERR_BAD_DATA, "%s", kBadData) : RAD_OK;
    }
    std::vector<double> in((size_t)tr->n_particles + n_g);
    inputs(in.data());
    RAD_HIP(hipMemcpyAsync(tr->d_wg, in.data(), in_bytes, hipMemcpyHostToDevice, st));
    const hipError_t e = launch(tr->d_I, nullptr);
    if (e != hipSuccess) return hip_fail(e, "tracked finalize launch");
    int flag = 0;
    RAD_HIP(hipMemcpyAsync(&flag, tr->d_err, sizeof(int), hipMemcpyDeviceToHost, st));
    RAD_HIP(hipStreamSynchronize(st));
    if (flag) return fail(RAD_ERR_BAD_DATA, "%s", kBadData);
    RAD_HIP(hipMemcpyAsync(I_host, tr->d_I, out_bytes, hipMemcpyDeviceToHost, st));
    RAD_HIP(hipStreamSynchronize(st));
    return RAD_OK;
}
