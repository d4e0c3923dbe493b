// Time-domain deposit (Algorithm 2 with the piecewise-linear interpolation of
// Sec. "Interpolation"), forward pass.
//
// Work decomposition (one GPU's share of the paper's detector decomposition):
//   * a pre-pass (for many pushed particles the pusher) writes, for every (particle, sample), the
//     sample's arrival base d (the two large, cancelling terms of the arrival time, carried in double-double and
//     rounded once), flags particles whose arrival times are not provably increasing and finds
//     each particle's max |r|^2; a pixel table holds each pixel's constants;
//   * fast path (k_sweep, particles whose arrival times provably increase): for each pixel the grid
//     points of the window are looked up among the samples, not the samples among the grid points.
//     A block takes a particle in steps of 256 samples (128 in FP64), finds from the arrival times at the steps'
//     ends which steps hold window grid points for its 128 pixels, stages those steps' samples in
//     LDS and gives every lane one (pixel, grid point) pair: the lane finds the sample interval of
//     its grid point, evaluates the field at the interval's two ends and adds the interpolated
//     value to the trace.  Arrival times are formed where that needs them: at the steps' ends and,
//     per grid point, at about four samples, instead of at every sample (bunch workload: 21 samples
//     per grid point inside the window and 71 % of the samples outside it; precision workload: 99 %
//     outside).  Steps with many grid points per sample form every arrival time and field once
//     instead;
//   * careful path (k_careful, particles the pre-pass could not clear): lanes own pixels; the
//     skip rules of lw_deposit_td are applied interval by interval, crossings go to a queue in LDS
//     that is drained 64 entries at a time, one per lane (see Wave::drain): the field at the
//     interval's two ends and the interpolated values at its grid points, added to the trace.  An
//     interval holding more than kLongRun grid points (an observer grid much finer than the samples)
//     is deposited by the whole wavefront, 64 grid points per pass.
// The field is therefore evaluated only at samples that the interpolation reads.  Every decision
// and weight uses one arrival-time value per (sample, pixel): every path evaluates it with the
// same operations (tau_eval), and the field with one function, so a contribution's bits do not
// depend on the path that finds it.  LW_CULL asks for what the fast path does anyway.
//
// Arrival-time forms (exact geometry): the polynomials in the pixel variable b hold the path term's series
// (first order with single-precision fields, third order with double ones; valid where
// |r|^2 <= 1e-8 |x_m|^2 over the whole trajectory) for pixels at the reference distance
// (|x_m| of the first pixel), evaluated to a lower degree where the terms above it are provably
// negligible for the particle and the tile's pixels (kModeRecLow); a tile whose pixels
// sit at another distance, or a particle outside the series bound, evaluates arrival_tau per
// pixel instead (series or square-root form), from the same d.
//
// Fast path condition (checked per particle by the pre-pass): every sample usable and
// every step shorter than c*dt by a margin well above the rounding of tau, which makes
// tau strictly increasing for every pixel (|x - r_i| - |x - r_{i-1}| >= -|r_i - r_{i-1}|).
#include "lw_internal.h"

#include <algorithm>
#include <cmath>
#include <type_traits>

namespace lw {
namespace {

constexpr int kPPL = 2;                 // pixels per lane
constexpr int kTilePix = 64 * kPPL;     // pixels per tile
constexpr int kPixBits = 7;
static_assert((1 << kPixBits) == kTilePix, "tile of 128 pixels");
constexpr int kBlockThreads = 64;
// queue ring: up to 63 pending entries plus one push (at most 64 crossings: one sample's pixels
// of one half of the tile)
constexpr uint32_t kQCap = 128;
// intervals with more grid points than this are deposited by the whole wavefront
constexpr int kLongRun = 8;
// Fast path: a particle's samples are split into segments of at most kSegIntervals intervals, into more of them
// where that leaves fewer than kFillBlocks blocks; particles per block: one until there are kTargetBlocks
// blocks (some 20 to 30 rounds of the resident ones), then up to kMaxPartsPerGroup.  Few of a bunch's particles may
// pass the window (1 in 70 of the precision workload, whose (particle, tile) units took 2.8 ms each, a quarter of the
// sweep with most of the chip idle at its end): a block looks its particles through first, and a unit is
// short.  Precision cut 35.8 -> 29.1 ms, 1000-electron bunch FP64 3.42 -> 2.68 ms (4096 intervals: 3.2).
constexpr int64_t kSegIntervals = 4096, kSegIntervals64 = 2048;
constexpr int64_t kTargetBlocks = 16384;
// trajectories of one step are light, and a block's own start (pixels, counters) outweighs them: fewer blocks then.  254 draws
// of up to 128 samples, 1 to 1e5 particles, 1 to 2e4 pixels: 5 % faster in the mean than with kTargetBlocks (8192 blocks
// 3 %, 2048 6 %, with more of them slower); 15077 particles of 8 samples, 160 pixels, most out of the window 333 -> 110 us
constexpr int64_t kTargetBlocksShort = 4096;
constexpr int kMaxPartsPerGroup = 64;  // at most a wavefront's lanes
constexpr int64_t kFillBlocks = 2048;
// particles per block of the careful path
constexpr int kMaxPartsCareful = 4;
// most particles, and particles times tiles, of a launch
constexpr int64_t kMaxParticles = int64_t(1) << 23, kMaxUnits = int64_t(1) << 26;
// samples per block of the pre-pass: at most kPrepassChunk, less where that leaves fewer than
// kPrepassBlocks blocks (one electron of 20001 samples: 65 us in 3 blocks)
constexpr int kPrepassChunk = 8192;
constexpr int64_t kPrepassBlocks = 2048;
// pixel table: kPT doubles per pixel (o, px, py, ok, nx, ny, nz, D, invD, padding), at most
// kPixTabMax pixels per pass (its share of the workspace); larger grids take several passes
constexpr int kPT = 16;
constexpr int64_t kPixTabMax = 16384;
static_assert(kPixTabMax % kTilePix == 0, "whole tiles per pixel pass");

// scan modes: polynomials (degree 3 or 5 in b, exact geometry), far field (tau = d + b),
// or arrival_tau per pixel in one of its forms
constexpr int kModeRec3 = 0, kModeRec5 = 1, kModeFar = 2;
// arrival_tau per pixel with the form of each pixel (series where rb2 |x_m|^-2 <= kSeriesBound)
constexpr int kModeMixed = 6;
// polynomials evaluated to a lower degree (RecLayout::LOW: 2 of 3 with single-precision
// fields, 3 of 5 with double ones) where tail_negligible holds for the particle and the tile
constexpr int kModeRecLow = 7;

// Degrees of the arrival time as a polynomial in the pixel variable (exact geometry), and the lower one of kModeRecLow
template <int GEOM, bool F64>
struct RecLayout {
    static constexpr int DEG = GEOM == LW_GEOM_FARFIELD ? 0 : (F64 ? 5 : 3);
    static constexpr int LOW = GEOM == LW_GEOM_FARFIELD ? 0 : (F64 ? 3 : 2);
};

// number of window grid points <= tau: clamp(floor(tau) + 1, 0, n_obs)
__device__ __forceinline__ int64_t grid_count(double tau, double n_obs)
{
    return (int64_t)fmin(fmax(floor(tau) + 1.0, 0.0), n_obs);
}

// |r|^2 with the operation order of the pre-pass
__device__ __forceinline__ double sq3(double x, double y, double z) { return fma(z, z, fma(y, y, x * x)); }

// value of lane src (wavefront-uniform src) of a double / float / double register
__device__ __forceinline__ double readlane_double(double v, int src)
{
    const uint64_t b = (uint64_t)__double_as_longlong(v);
    const uint32_t lo = __builtin_amdgcn_readlane((uint32_t)b, src);
    const uint32_t hi = __builtin_amdgcn_readlane((uint32_t)(b >> 32), src);
    return __longlong_as_double((long long)(((uint64_t)hi << 32) | lo));
}
__device__ __forceinline__ float readlane_t(float v, int src)
{
    return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), src));
}
__device__ __forceinline__ double readlane_t(double v, int src) { return readlane_double(v, src); }

__device__ __forceinline__ double uniform_double(double v)
{
    const uint64_t b = (uint64_t)__double_as_longlong(v);
    const uint32_t lo = __builtin_amdgcn_readfirstlane((uint32_t)b);
    const uint32_t hi = __builtin_amdgcn_readfirstlane((uint32_t)(b >> 32));
    return __longlong_as_double((long long)(((uint64_t)hi << 32) | lo));
}

// The arrival bases are written by an earlier launch and only read while the deposit kernel runs, so
// a wavefront-uniform sample's is read through the constant address space: with the address in
// scalar registers these become scalar loads.
typedef const __attribute__((address_space(4))) double *cdptr;
__device__ __forceinline__ cdptr uniform_ptr(const double *p)
{
    const uint64_t b = (uint64_t)reinterpret_cast<uintptr_t>(p);
    const uint32_t lo = __builtin_amdgcn_readfirstlane((uint32_t)b);
    const uint32_t hi = __builtin_amdgcn_readfirstlane((uint32_t)(b >> 32));
    return (cdptr)(((uint64_t)hi << 32) | lo);
}

// ---------------------------------------------------------------------------------------------
// Pixel table and the arrival time

// What a launch starts from, in one kernel (six launches of their own were 15 of one electron's 57 us): zeros in the
// trace (n_trace 16-byte elements and n_tail 4-byte ones behind them), the counters, the particles' flags and bounds
// (n_p), and the pixel table's rows [0, n_rows): the pixels [0, n_pix), then padding rows (all zero, not usable) up to
// the end of the last tile, whose arrival times stay finite.
struct SetupShape {
    int64_t n_trace, n_tail, n_p, n_pix, n_rows;
    double C;
};
__global__ __launch_bounds__(256) void k_setup(uint4 *__restrict__ trace, unsigned long long *__restrict__ diag,
                                               int *__restrict__ pflag, unsigned long long *__restrict__ rmax2,
                                               const double *__restrict__ x_det, double *__restrict__ pt, SetupShape sh)
{
    const int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x, step = (int64_t)gridDim.x * blockDim.x;
    for (int64_t j = t; j < sh.n_trace; j += step) trace[j] = make_uint4(0, 0, 0, 0);
    if (t < sh.n_tail) ((uint32_t *)(trace + sh.n_trace))[t] = 0;
    if (diag && t < 4) diag[t] = 0;
    for (int64_t j = t; j < sh.n_p; j += step) {
        pflag[j] = 0;
        rmax2[j] = 0;
    }
    for (int64_t m = t; m < sh.n_rows; m += step) {
        double *o = pt + m * kPT;
        if (m >= sh.n_pix) {
#pragma unroll
            for (int j = 0; j < kPT; ++j) o[j] = 0.0;
            continue;
        }
        const PixC p = pix_const(x_det, m, sh.C);
        o[0] = p.o;
        o[1] = p.px;
        o[2] = p.py;
        o[3] = p.g.ok ? 1.0 : 0.0;
        o[4] = p.g.nx;
        o[5] = p.g.ny;
        o[6] = p.g.nz;
        o[7] = p.g.D;
        o[8] = p.g.invD;
#pragma unroll
        for (int j = 9; j < kPT; ++j) o[j] = 0.0;
    }
}

// a pixel's constants from its table row (per lane, or wavefront-uniform through scalar loads)
template <typename P>
__device__ __forceinline__ PixC pixc_row(P row)
{
    PixC p;
    p.o = row[0];
    p.px = row[1];
    p.py = row[2];
    p.g.ok = row[3] != 0.0;
    p.g.nx = row[4];
    p.g.ny = row[5];
    p.g.nz = row[6];
    p.g.D = row[7];
    p.g.invD = row[8];
    return p;
}

// The values of a sample that a scan mode's arrival time takes (N of them; X: offset of the position):
//   far field:             d, x, y, z
//   polynomials:           c_0 .. c_{DEG-1}, x, y, z (the leading coefficient is the same for every sample)
//   kModeMixed:            x, y, z, d
template <int GEOM, bool F64, int MODE>
struct ScanVals {
    using L = RecLayout<GEOM, F64>;
    static constexpr int N = (MODE == kModeFar || MODE == kModeMixed) ? 4 : L::DEG + 3;
    static constexpr int X = MODE == kModeFar ? 1 : (MODE == kModeMixed ? 0 : L::DEG);
};
template <int GEOM, bool F64, int MODE>
__device__ __forceinline__ void scan_vals(double d, double x, double y, double z, double C, double Dref, double *v)
{
    using V = ScanVals<GEOM, F64, MODE>;
    v[V::X] = x;
    v[V::X + 1] = y;
    v[V::X + 2] = z;
    if constexpr (MODE == kModeFar) {
        v[0] = d;
    } else if constexpr (MODE == kModeMixed) {
        v[3] = d;
    } else {
        constexpr int DEG = RecLayout<GEOM, F64>::DEG, LOW = RecLayout<GEOM, F64>::LOW;
        double c[DEG + 1];
        tau_poly<DEG>(d, x, y, z, C, Dref, c);
#pragma unroll
        for (int j = 0; j < DEG; ++j) v[j] = MODE == kModeRecLow && j > LOW ? 0.0 : c[j];
    }
}

// Arrival time of one (sample, pixel) in scan mode MODE from the sample's values v (scan_vals) and the
// pixel constants P: far field tau = d + b; polynomials tau = sum_j c_j b^j (c_DEG = cK; up to
// j = LOW in kModeRecLow); else
// arrival_tau in the pixel's form (series where rb2 |x_m|^-2 <= kSeriesBound).  A (sample, pixel)
// gets the same bits wherever it is evaluated.
template <int GEOM, bool F64, int MODE>
__device__ __forceinline__ double tau_eval(const PixC &P, const double *v, double cK, double rb2, double C)
{
    if constexpr (MODE == kModeFar) {
        return pix_b(P, v[1], v[2], v[3]) + v[0];
    } else if constexpr (MODE == kModeRec3 || MODE == kModeRec5 || MODE == kModeRecLow) {
        constexpr int DEG = RecLayout<GEOM, F64>::DEG, LOW = RecLayout<GEOM, F64>::LOW;
        const double b = pix_b(P, v[DEG], v[DEG + 1], v[DEG + 2]);
        double u;
        if constexpr (MODE == kModeRecLow) {
            u = fma(b, v[LOW], v[LOW - 1]);
#pragma unroll
            for (int j = LOW - 2; j >= 0; --j) u = fma(b, u, v[j]);
        } else {
            u = fma(b, cK, v[DEG - 1]);
#pragma unroll
            for (int j = DEG - 2; j >= 0; --j) u = fma(b, u, v[j]);
        }
        return u;
    } else {
        constexpr int FORM = F64 ? kTauSeries : kTauShort;
        const double x = v[0], y = v[1], z = v[2], rr = sq3(x, y, z);
        if (rb2 * (P.g.invD * P.g.invD) <= kSeriesBound) return arrival_tau<GEOM, FORM>(P, v[3], x, y, z, rr, C);
        return arrival_tau<GEOM, kTauSqrt>(P, v[3], x, y, z, rr, C);
    }
}

inline size_t align_up(size_t v, size_t a) { return (v + a - 1) / a * a; }

struct DepWs {
    double *pt;                 // [kPixTabMax][kPT] pixel table of the current pass
    int *pflag;                 // [n_p] see k_prepass
    unsigned long long *rmax2;  // [n_p] bits of max_i |r_i|^2 (non-negative doubles order as integers)
    double *d;                  // [n_p][n_s] arrival bases
};

constexpr size_t kPixTabBytes = (size_t)kPixTabMax * kPT * sizeof(double);

// pixel table, flags, bounds and arrival bases
size_t ws_bytes_for(int64_t n_p, int64_t ns)
{
    const size_t np = (size_t)std::max<int64_t>(n_p, 1), nsz = (size_t)std::max<int64_t>(ns, 1);
    return kPixTabBytes + align_up(np * sizeof(int), 256) + align_up(np * sizeof(unsigned long long), 256) +
           align_up(np * nsz * sizeof(double), 256);
}

DepWs carve(void *ws, int64_t n_p)
{
    DepWs w;
    char *p = (char *)ws;
    w.pt = (double *)p;
    p += kPixTabBytes;
    w.pflag = (int *)p;
    p += align_up((size_t)std::max<int64_t>(n_p, 1) * sizeof(int), 256);
    w.rmax2 = (unsigned long long *)p;
    p += align_up((size_t)std::max<int64_t>(n_p, 1) * sizeof(unsigned long long), 256);
    w.d = (double *)p;
    return w;
}

// Whether dense particles (at least kGatherDensity grid points per interval at a pixel in the middle of the detector) of
// short trajectories go to k_gather, and what that is decided by: their number, their grid points and the windows these
// touch, and in at most 512 bins of windows how many particles overlap.  The rule compares estimates of both kernels'
// times, fitted to 240 drawn calls of 1 to 1e5 particles of 2 to 1000 samples on 1 to 3000 pixels (k_gather: nine of ten
// within 0.46 to 1.26 of the measured times; k_sweep without its cost of the trace's zeros and the launches):
//   k_gather  5 us, 6 ns a window and pixel, 5 ps more for each particle to look at, 2.2 us a particle that
//             the fullest window takes (one after the other), 4.1 us a particle and window on 1536 resident blocks
//   k_sweep   13 ps a grid point (FP64 20), 10 ns a particle and tile, and of one block's particles and pixels,
//             kDensePix at a time, 1 us and 1.7 ns a grid point
// and takes k_gather where it is faster by half: in 77 of the draws, where k_sweep takes 1.07 to 19 times as long.  By their
// density alone k_gather would be the slower one in 144 of the draws, up to 58 times.  Where k_sweep keeps them, the rule
// and the idle launch cost 4 us (calls too small for k_gather on any account have neither).
constexpr double kGatherDensity = 1.0;
constexpr float kGatherMargin = 1.5f;
constexpr int64_t kGatherSamples = 1024;  // longest trajectory (every sample that bounds a window is evaluated)
constexpr int kGatherBins = 512, kRuleBlocks = 64;
constexpr int64_t kGatherBlocks = 4095;  // odd, so that no block takes the same window of every pixel (an idle block takes 0.7 ns)
struct GatherRule {
    int64_t n_p;           // blocks from this one on are the rule's
    const double *x_mid;
    double n_obs;
    int64_t n_win, window, bin;  // windows of a pixel, grid points of a window and a bin
    float fixed, per_most, per_window, per_point, per_particle, per_pass, per_mean;  // us
    // of the fullest window's particles, the windows, points and particles
    __host__ __device__ __forceinline__ bool gathered(float most, float windows, float points, float particles) const
    {
        const float gather = fixed + per_most * most + per_window * windows;
        const float sweep = per_point * points + per_particle * particles + per_pass + per_mean * points / fmaxf(particles, 1.0f);
        return kGatherMargin * gather < sweep;
    }
};
// In the padding of the pixel table (zero at the start of a pixel pass): the tenth and eleventh elements of row j hold the
// changes of the overlap at bins 4 j to 4 j + 3, the first row's others the rest
struct GatherStats {
    double *pt;
    __device__ __forceinline__ int *step(int j) const { return (int *)(pt + (int64_t)(j >> 2) * kPT + 9) + (j & 3); }
    __device__ __forceinline__ unsigned long long *sum(int i) const { return (unsigned long long *)(pt + 11 + i); }  // points, windows, particles
    __device__ __forceinline__ unsigned *blocks() const { return (unsigned *)(pt + 14); }
};
// the decision: 1 where k_gather takes the dense particles
__device__ __forceinline__ const int *gather_flag(const double *pt) { return (const int *)(pt + kPT - 1); }
static_assert(kGatherBins <= 4 * kTilePix, "bins in the rows of the first tile");

template <typename T>
__device__ __forceinline__ T load_shared_by_blocks(const T *p)
{
    return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// Block b of n_blocks (of 256 threads): flags the dense particles; the last block to end decides.  In blocks of their own beside
// the pre-pass's: added up there, particle by particle, the sums took 60 ns a particle.
__device__ __forceinline__ void gather_rule(const GatherRule &rule, int b, int n_blocks, const double *__restrict__ r,
                                            int64_t n_samples, int64_t sample0, double t_start, double dt, double t0,
                                            double dt_obs, double C, int geom, int *__restrict__ pflag, double *pt)
{
    __shared__ int s_step[kGatherBins];
    __shared__ unsigned long long s_sum[3];
    __shared__ bool s_last;
    const int tid = threadIdx.x;
    for (int j = tid; j < kGatherBins; j += 256) s_step[j] = 0;
    if (tid < 3) s_sum[tid] = 0ull;
    __syncthreads();
    const PixC P = pix_const(rule.x_mid, 0, C);
    unsigned long long v[3] = {0ull, 0ull, 0ull};
    for (int64_t k = (int64_t)b * 256 + tid; k < rule.n_p; k += (int64_t)n_blocks * 256) {
        // by the first and last arrival times
        auto tau = [&](int64_t i) {
            const double *ri = r + 3 * (k * n_samples + i);
            const double d = arrival_base(t_start, dt, (double)(sample0 + i), t0, dt_obs, ri[2]);
            return geom == LW_GEOM_EXACT ? arrival_tau<LW_GEOM_EXACT, kTauSqrt>(P, d, ri[0], ri[1], ri[2], 0.0, C)
                                         : arrival_tau<LW_GEOM_FARFIELD, kTauSqrt>(P, d, ri[0], ri[1], ri[2], 0.0, C);
        };
        const double ta = tau(0), tb = tau(n_samples - 1);
        if (!(tb - ta >= kGatherDensity * (double)(n_samples - 1))) continue;
        atomicOr(pflag + k, 2);
        const int64_t c0 = grid_count(ta, rule.n_obs), c1 = grid_count(tb, rule.n_obs);
        if (c1 <= c0) continue;
        v[0] += (unsigned long long)(c1 - c0);
        v[1] += (unsigned long long)((c1 - 1) / rule.window - c0 / rule.window + 1);
        v[2] += 1ull;
        atomicAdd(s_step + (int)(c0 / rule.bin), 1);
        const int64_t after = (c1 - 1) / rule.bin + 1;
        if (after < kGatherBins) atomicAdd(s_step + (int)after, -1);
    }
    for (int i = 0; i < 3; ++i) {
        for (int off = 32; off > 0; off >>= 1) v[i] += __shfl_xor(v[i], off);
        if ((tid & 63) == 0) atomicAdd(s_sum + i, v[i]);
    }
    __syncthreads();
    const GatherStats st{pt};
    for (int j = tid; j < kGatherBins; j += 256)
        if (s_step[j]) atomicAdd(st.step(j), s_step[j]);
    if (tid < 3 && s_sum[tid]) atomicAdd(st.sum(tid), s_sum[tid]);
    __threadfence();
    __syncthreads();
    if (tid == 0) s_last = atomicAdd(st.blocks(), 1u) == (unsigned)n_blocks - 1u;
    __syncthreads();
    if (!s_last || tid >= 64) return;
    __threadfence();
    // a lane takes neighbouring bins: their running sums, raised by what precedes the lane
    constexpr int kPer = kGatherBins / 64;
    int sum = 0, most = -0x7fffffff;
    for (int j = 0; j < kPer; ++j) {
        sum += load_shared_by_blocks(st.step(kPer * tid + j));
        most = max(most, sum);
    }
    int upto = sum;
    for (int off = 1; off < 64; off <<= 1) {
        const int o = __shfl_up(upto, off);
        if (tid >= off) upto += o;
    }
    most += upto - sum;
    for (int off = 32; off > 0; off >>= 1) most = max(most, __shfl_xor(most, off));
    if (tid == 0) {
        auto sum_of = [&](int i) { return (float)load_shared_by_blocks(st.sum(i)); };
        *const_cast<int *>(gather_flag(pt)) = rule.gathered((float)most, sum_of(1), sum_of(0), sum_of(2)) ? 1 : 0;
    }
}

// ---------------------------------------------------------------------------------------------
// pre-pass: one block per (particle, chunk of samples): arrival bases, per-particle max |r|^2 and the flags: 1 for the
// careful path, 2 for a dense particle (gather_rule), 0 else.  Bound by memory: 72 bytes of a
// sample read, 8 written (with the polynomial's coefficients and the position stored beside the base, 64 or 80 written,
// the pre-pass of 2000 x 20001 samples took 1.75 ms, now 0.79; the coefficients are formed where a step's samples are
// staged instead)
__global__ __launch_bounds__(256) void k_prepass(const double *__restrict__ r, const double *__restrict__ beta,
                                                 const double *__restrict__ beta_dot, int64_t n_samples, int chunk,
                                                 int64_t sample0, double t_start, double dt, double t0,
                                                 double dt_obs, double C, double *__restrict__ base,
                                                 int *__restrict__ pflag, unsigned long long *__restrict__ rmax2,
                                                 int geom, GatherRule rule, double *pt)
{
    __shared__ unsigned long long s_max[4];
    __shared__ int s_bad[4];
    const int64_t k = blockIdx.x;
    if (k >= rule.n_p) {
        if (blockIdx.y == 0)
            gather_rule(rule, (int)(k - rule.n_p), (int)(gridDim.x - rule.n_p), r, n_samples, sample0, t_start, dt, t0, dt_obs, C, geom,
                        pflag, pt);
        return;
    }
    const int64_t i_begin = (int64_t)blockIdx.y * chunk;
    const int64_t i_end = std::min<int64_t>(i_begin + chunk, n_samples);
    const double cdt_step = kC * dt;
    double mx = 0.0;
    int bad = 0;
    for (int64_t i = i_begin + threadIdx.x; i < i_end; i += blockDim.x) {
        const int64_t s = k * n_samples + i;
        const double *ri = r + 3 * s, *bi = beta + 3 * s, *di = beta_dot + 3 * s;
        const double x = ri[0], y = ri[1], z = ri[2];
        // sample i of the arrays is sample sample0 + i of the trajectory (spans of a longer one)
        const double d = arrival_base(t_start, dt, (double)(sample0 + i), t0, dt_obs, z);
        base[s] = d;
        const double rr = sq3(x, y, z);
        bool b = !sample_usable(ri, bi, di);
        if (!b) {
            mx = fmax(mx, rr);
            if (i > 0) {
                const double dx = x - ri[-3], dy = y - ri[-2], dz = z - ri[-1];
                b = interval_slow(d, x, y, z, sqrt(dx * dx + dy * dy + dz * dz), cdt_step, C);
            }
        }
        bad |= b ? 1 : 0;
    }
    // block reduction
    for (int off = 32; off > 0; off >>= 1) {
        mx = fmax(mx, __shfl_xor(mx, off));
        bad |= __shfl_xor(bad, off);
    }
    const int wv = threadIdx.x >> 6;
    if ((threadIdx.x & 63) == 0) {
        s_max[wv] = (unsigned long long)__double_as_longlong(mx);
        s_bad[wv] = bad;
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        unsigned long long m = 0;
        int bb = 0;
        for (int w = 0; w < (int)(blockDim.x >> 6); ++w) {
            m = std::max(m, s_max[w]);
            bb |= s_bad[w];
        }
        atomicMax(rmax2 + k, m);
        if (bb) atomicOr(pflag + k, 1);
    }
}

template <typename T>
__global__ void k_fill(T *__restrict__ p, int64_t n)
{
    for (int64_t j = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; j < n; j += (int64_t)gridDim.x * blockDim.x)
        p[j] = (T)0;
}

// ---------------------------------------------------------------------------------------------
struct DepShape {
    int64_t n_particles, n_samples, n_pix, n_obs;
    int64_t n_tiles, n_groups, parts_per_group;
    double C;  // 1/(c dt_obs)
    int fmask;
};

// contribution v to element j of the trace, row `row` (the row only matters in kAccFixed; the
// order-independent modes are FP64 only)
template <int ACC, typename T>
__device__ __forceinline__ void put(T *E, const DetAcc &det, size_t j, size_t row, T v)
{
    if constexpr (ACC == kAccFloat) {
        atomic_add(E + j, v);
    } else if constexpr (ACC == kAccMaxAbs) {
        atomicMax((unsigned long long *)E + j, (unsigned long long)__double_as_longlong(fabs(v)));
    } else {
        // |v * scale| < 2^62 by the choice of scale, and any term below 2^63 is taken, so a
        // last-bit difference between the two passes' v cannot drop one (a NaN scale drops
        // all: the row is NaN in the result).  The sign-extended term is added to the 128-bit
        // sum as its low word and, with the carry out of the low word, its high word.
        const double t = v * det.scale[row];
        const long long n = fabs(t) < 0x1p63 ? (long long)__builtin_rint(t) : 0ll;
        if (n != 0) {
            const unsigned long long un = (unsigned long long)n;
            const unsigned long long old = atomicAdd((unsigned long long *)E + j, un);
            const long long dh = (n < 0 ? -1ll : 0ll) + (old + un < old ? 1ll : 0ll);
            if (dh != 0) atomicAdd(det.hi + j, (unsigned long long)dh);
        }
    }
}

// Per-wavefront state of the careful path (k_careful): lanes own pixels (kPPL each); a particle's
// samples are taken one at a time, with the skip rules applied per interval; crossings are queued
// in LDS and drained 64 at a time, each lane adding one interval's grid points to the trace with
// global atomics (ACC: how a contribution is added to the trace).
template <typename T, int GEOM, int ACC = kAccFloat>
struct Wave {
    const double *__restrict__ r;
    const double *__restrict__ beta;
    const double *__restrict__ beta_dot;
    const double *__restrict__ charge;
    const double *__restrict__ x_det;
    const double *__restrict__ base;  // arrival bases
    const double *__restrict__ pt;    // pixel table of this pass
    T *__restrict__ E;
    DepShape sh;
    double cK;   // leading coefficient of the polynomials
    double Dref; // the polynomials' pixel distance
    double rb2;  // the current particle's bound of |r|^2 over its whole trajectory
    int lane;
    int64_t tile, k0;
    uint2 *q;          // queue ring in LDS: {sample index, (particle - k0) << kPixBits | pixel in tile}
    double2 *qt;       // the entry's arrival times {tau_{i-1}, tau_i}
    double *sv;        // the scan values of 64 samples in LDS [value][sample]
    PixC pc[kPPL];     // constants of this lane's pixels (lane + 64 h)
    uint32_t qh, qn;   // queue ring head and length
    DetAcc det;        // high words and row scales (ACC == kAccFixed)

    __device__ __forceinline__ static uint32_t qwrap(uint32_t v) { return v >= kQCap ? v - kQCap : v; }

    // Arrival time of pixel h from the scan values v of a sample (wavefront-uniform)
    template <int MODE>
    __device__ __forceinline__ double tau_of(int h, const double *v) const
    {
        return tau_eval<GEOM, sizeof(T) == 8, MODE>(pc[h], v, cK, rb2, sh.C);
    }

    // the scan values of samples i0 .. i0 + 63 of particle k (up to the last one's) into sv: a sample's coefficients are
    // formed by one lane, not by all of them in turn (2 particles x 2001 samples, 128 pixels, FP64: 5.53 -> 5.19 ms)
    template <int MODE>
    __device__ __forceinline__ void stage_scan(int64_t k, int64_t i0) const
    {
        __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");  // the values before are read
        __builtin_amdgcn_wave_barrier();
        const size_t s = (size_t)k * sh.n_samples + (size_t)std::min<int64_t>(i0 + lane, sh.n_samples - 1);
        double v[ScanVals<GEOM, sizeof(T) == 8, MODE>::N];
        scan_vals<GEOM, sizeof(T) == 8, MODE>(base[s], r[3 * s], r[3 * s + 1], r[3 * s + 2], sh.C, Dref, v);
#pragma unroll
        for (int c = 0; c < ScanVals<GEOM, sizeof(T) == 8, MODE>::N; ++c) sv[64 * c + lane] = v[c];
        __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
        __builtin_amdgcn_wave_barrier();
    }

    // Evaluate the cnt oldest queued crossings (lane j takes entry j).
    __device__ void drain(uint32_t cnt)
    {
        __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
        __builtin_amdgcn_wave_barrier();
        const bool act = (uint32_t)lane < cnt;
        const uint32_t slot = qwrap(qh + (uint32_t)lane);
        const uint2 e = act ? q[slot] : make_uint2(1u, 0u);
        const double2 tt = act ? qt[slot] : make_double2(0.0, 1.0);
        const int ml0 = (int)(e.y & (uint32_t)(kTilePix - 1));
        // far field: the entry's pixel direction from the pixel table
        PixGeo g;
        if (GEOM == LW_GEOM_FARFIELD) {
            g = pixc_row(pt + (size_t)(tile * kTilePix + ml0) * kPT).g;
        } else {
            g.nx = g.ny = 0.0;
            g.nz = g.D = g.invD = 1.0;
            g.ok = true;
        }
        // the entry's interval: fields at both ends and grid points [u0, u1)
        const double ta = tt.x, tb = tt.y;
        int u0 = 0, u1 = 0;
        T idt = (T)0, eax = (T)0, eay = (T)0, eaz = (T)0, ebx = (T)0, eby = (T)0, ebz = (T)0;
        if (act) {
            const uint32_t i = e.x, kl = e.y;
            const int64_t k = k0 + (int64_t)(kl >> kPixBits);
            const int ml = ml0;
            const int64_t m = tile * kTilePix + ml;
            // both samples of the interval, each value loaded once (all loads issued first)
            const size_t sa = ((size_t)k * sh.n_samples + i - 1) * 3;
            const double *ra = r + sa, *ba = beta + sa, *da = beta_dot + sa;
            const double rax = ra[0], ray = ra[1], raz = ra[2], rbx = ra[3], rby = ra[4], rbz = ra[5];
            const double bax = ba[0], bay = ba[1], baz = ba[2], bbx = ba[3], bby = ba[4], bbz = ba[5];
            const double dax = da[0], day = da[1], daz = da[2], dbx = da[3], dby = da[4], dbz = da[5];
            const double q = charge ? charge[k] : -kQe;
            const double *xm = x_det + 3 * m;
            lw_field<T, GEOM>(g, xm, rax, ray, raz, bax, bay, baz, dax, day, daz, q, sh.fmask, eax, eay, eaz);
            lw_field<T, GEOM>(g, xm, rbx, rby, rbz, bbx, bby, bbz, dbx, dby, dbz, q, sh.fmask, ebx, eby, ebz);
            // grid indices fit in 32 bits (n_obs < 2^31, checked on the host)
            const double nob = (double)sh.n_obs;
            u0 = (int)fmin(fmax(floor(ta) + 1.0, 0.0), nob);
            u1 = (int)fmin(fmax(floor(tb) + 1.0, 0.0), nob);
            // interpolation weight w = (u - ta)/(tb - ta), in the precision of the trace
            idt = sizeof(T) == 4 ? (T)__builtin_amdgcn_rcpf((float)(tb - ta)) : (T)(1.0 / (tb - ta));
            if (u1 - u0 <= kLongRun) {
                for (int u = u0; u < u1; ++u) {
                    const T w = (T)((double)u - ta) * idt, w1 = (T)1 - w;
                    const size_t row = (size_t)m * 3, j = row * sh.n_obs + u;
                    put<ACC>(E, det, j, row, w1 * eax + w * ebx);
                    put<ACC>(E, det, j + sh.n_obs, row + 1, w1 * eay + w * eby);
                    put<ACC>(E, det, j + 2 * sh.n_obs, row + 2, w1 * eaz + w * ebz);
                }
            }
        }
        // intervals holding many grid points (a grid much finer than the sample spacing): the
        // whole wavefront deposits them one at a time, 64 consecutive grid points per pass
        uint64_t longm = __ballot(act && u1 - u0 > kLongRun);
        while (longm) {
            const int src = (int)__builtin_ctzll(longm);
            longm &= longm - 1;
            const double sta = readlane_double(ta, src);
            const int su0 = __builtin_amdgcn_readlane(u0, src), su1 = __builtin_amdgcn_readlane(u1, src);
            const int sml = __builtin_amdgcn_readlane(ml0, src);
            const T sidt = readlane_t(idt, src);
            const T sax = readlane_t(eax, src), say = readlane_t(eay, src), saz = readlane_t(eaz, src);
            const T sbx = readlane_t(ebx, src), sby = readlane_t(eby, src), sbz = readlane_t(ebz, src);
            // 64-bit index: su1 may sit within 64 of the largest int (n_obs up to 2^31 - 1)
            for (int64_t u = (int64_t)su0 + lane; u < su1; u += 64) {
                const T w = (T)((double)u - sta) * sidt, w1 = (T)1 - w;
                const size_t row = (size_t)(tile * kTilePix + sml) * 3, j = row * sh.n_obs + u;
                put<ACC>(E, det, j, row, w1 * sax + w * sbx);
                put<ACC>(E, det, j + sh.n_obs, row + 1, w1 * say + w * sby);
                put<ACC>(E, det, j + 2 * sh.n_obs, row + 2, w1 * saz + w * sbz);
            }
        }
        // the entries are read: later pushes may take their slots
        __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
        __builtin_amdgcn_wave_barrier();
        qh = __builtin_amdgcn_readfirstlane(qwrap(qh + cnt));
        qn = __builtin_amdgcn_readfirstlane(qn - cnt);
    }

    // Append the lanes with `hit` set (callers drain before kTilePix more can arrive).
    __device__ __forceinline__ void push(bool hit, uint64_t mask, uint32_t i, uint32_t tag, double ta, double tb)
    {
        if (hit) {
            const uint32_t slot = qwrap(qh + qn + lanes_below(mask));
            q[slot] = make_uint2(i, tag);
            qt[slot] = make_double2(ta, tb);
        }
        qn = __builtin_amdgcn_readfirstlane(qn + (uint32_t)__popcll(mask));  // wavefront-uniform
    }

    __device__ __forceinline__ void pump()
    {
        while (qn >= 64) drain(64);
    }

    // Careful path: the skip rules of lw_deposit_td interval by interval, pixel h of this lane,
    // with the arrival times of the fast path's MODE (the same values wherever a particle takes
    // the fast path in one span and the careful path in another).
    template <int MODE, int H>
    __device__ __forceinline__ void careful_particle(bool lane_ok, bool pix_in, int64_t m, int64_t k,
                                                     unsigned long long &c0, unsigned long long &c1,
                                                     unsigned long long &c2, unsigned long long &c3)
    {
        constexpr int NV = ScanVals<GEOM, sizeof(T) == 8, MODE>::N;
        const int64_t ns = sh.n_samples;
        const double nob = (double)sh.n_obs;
        const double q = charge ? charge[k] : -kQe;
        bool prev_ok = false;
        double tprev = 0.0;
        const uint32_t tag = ((uint32_t)(k - k0) << kPixBits) | (uint32_t)(lane + 64 * H);
        for (int64_t i = 0; i < ns; ++i) {
            const size_t s = (size_t)k * ns + i;
            if ((i & 63) == 0) stage_scan<MODE>(k, i);
            double v[NV];
#pragma unroll
            for (int c = 0; c < NV; ++c) v[c] = sv[64 * c + (i & 63)];
            const double x = r[3 * s], y = r[3 * s + 1], z = r[3 * s + 2];
            bool ok = lane_ok && sample_usable(r + 3 * s, beta + 3 * s, beta_dot + 3 * s);
            const double tv = tau_of<MODE>(H, v);
            double tau = NAN;
            if (ok) {
                tau = tv;
                T ex, ey, ez;
                lw_field<T, GEOM>(pc[H].g, x_det + 3 * m, x, y, z, beta[3 * s], beta[3 * s + 1], beta[3 * s + 2],
                                  beta_dot[3 * s], beta_dot[3 * s + 1], beta_dot[3 * s + 2], q, sh.fmask, ex, ey, ez);
                ok = isfinite(tau) && isfinite((double)ex) && isfinite((double)ey) && isfinite((double)ez);
            }
            bool hit = false;
            if (i > 0 && pix_in) {
                if (!ok || !prev_ok) {
                    c1 += 1;
                } else if (!(tau > tprev)) {
                    c0 += 1;
                } else {
                    const int64_t fa = grid_count(tprev, nob), fb = grid_count(tau, nob);
                    c3 += (unsigned long long)(fb - fa);
                    c2 += (unsigned long long)((int64_t)(floor(tau) - floor(tprev)) - (fb - fa));
                    hit = fb > fa;
                }
            }
            const uint64_t mask = __ballot(hit);
            if (mask) {
                push(hit, mask, (uint32_t)i, tag, tprev, tau);
                pump();
            }
            prev_ok = ok;
            tprev = tau;
        }
    }

    // One particle in scan mode MODE, both pixels of this lane
    template <int MODE>
    __device__ __forceinline__ void particle(const bool *lane_ok, const bool *pix_in, const int64_t *m, int64_t k,
                                             unsigned long long &c0, unsigned long long &c1, unsigned long long &c2,
                                             unsigned long long &c3)
    {
        static_assert(kPPL == 2, "careful path written for two pixels per lane");
        careful_particle<MODE, 0>(lane_ok[0], pix_in[0], m[0], k, c0, c1, c2, c3);
        careful_particle<MODE, 1>(lane_ok[1], pix_in[1], m[1], k, c0, c1, c2, c3);
    }
};

// careful path: the particles the pre-pass flagged (a wavefront whose group holds none exits)
template <typename T, int GEOM, int ACC>
__global__ __launch_bounds__(kBlockThreads) __attribute__((amdgpu_waves_per_eu(3))) void k_careful(
    const double *__restrict__ r, const double *__restrict__ beta, const double *__restrict__ beta_dot,
    const double *__restrict__ charge, const double *__restrict__ x_det, const double *__restrict__ base,
    const double *__restrict__ pt, const int *__restrict__ pflag, const unsigned long long *__restrict__ rmax2,
    const double *__restrict__ rbound2, T *__restrict__ E, unsigned long long *__restrict__ diag, DepShape sh, DetAcc det)
{
    constexpr bool kF64 = sizeof(T) == 8;
    constexpr int kRec = kF64 ? kModeRec5 : kModeRec3;
    // block -> (particle group, tile) as in k_sweep
    const int64_t b = blockIdx.x;
    const int64_t xcd = b & 7, slot = b >> 3;
    const int64_t grp = (slot / sh.n_tiles) * 8 + xcd;
    const int64_t tile = slot % sh.n_tiles;
    const int64_t k0 = grp * sh.parts_per_group;
    const int64_t k1 = grp < sh.n_groups ? std::min(k0 + sh.parts_per_group, sh.n_particles) : k0;
    {
        bool any = false;
        for (int64_t k = k0 + (threadIdx.x & 63); k < k1; k += 64) any |= (pflag[k] & 1) != 0;
        if (__ballot(any) == 0) return;  // whole block (one wavefront)
    }
    __shared__ uint2 q_all[kQCap];
    __shared__ double2 qt_all[kQCap];
    __shared__ double sv_all[64 * ScanVals<GEOM, kF64, GEOM == LW_GEOM_FARFIELD ? kModeFar : kRec>::N];
    __shared__ unsigned long long red[4];
    const int lane = threadIdx.x & 63;
    if (threadIdx.x < 4) red[threadIdx.x] = 0ull;
    __syncthreads();

    Wave<T, GEOM, ACC> w;
    int64_t m[kPPL];
    bool pix_in[kPPL], lane_ok[kPPL];
    double id2 = 0.0, s2 = 0.0;
    const double Dref = pix_geo(x_det, 0).D;  // the polynomials' pixel distance
    bool far_off = false;                     // a pixel of this wavefront at another distance
#pragma unroll
    for (int h = 0; h < kPPL; ++h) {
        m[h] = tile * kTilePix + 64 * h + lane;
        pix_in[h] = m[h] < sh.n_pix;
        w.pc[h] = pixc_row(pt + (pix_in[h] ? m[h] : 0) * kPT);
        lane_ok[h] = pix_in[h] && w.pc[h].g.ok;
        if (lane_ok[h]) {
            id2 = fmax(id2, w.pc[h].g.invD * w.pc[h].g.invD);
            s2 = fmax(s2, 2.0 * (1.0 - w.pc[h].g.nz));
            far_off |= !(fabs(w.pc[h].g.D - Dref) <= kSameDistance * Dref);
        }
    }
    for (int off = 32; off > 0; off >>= 1) {
        id2 = fmax(id2, __shfl_xor(id2, off));
        s2 = fmax(s2, __shfl_xor(s2, off));
    }
    const double invD2max = uniform_double(id2), s2max = uniform_double(s2);
    const bool rec_ok = GEOM == LW_GEOM_EXACT && __ballot(far_off) == 0;
    {
        double c[6];
        if (kF64)
            tau_poly<5>(0.0, 0.0, 0.0, 0.0, sh.C, Dref, c);
        else
            tau_poly<3>(0.0, 0.0, 0.0, 0.0, sh.C, Dref, c);
        w.cK = c[kF64 ? 5 : 3];
    }

    w.r = r;
    w.beta = beta;
    w.beta_dot = beta_dot;
    w.charge = charge;
    w.x_det = x_det;
    w.base = base;
    w.Dref = Dref;
    w.pt = pt;
    w.E = E;
    if constexpr (ACC != kAccFloat) w.det = det;
    w.sh = sh;
    w.lane = lane;
    w.tile = tile;
    w.k0 = k0;
    w.q = q_all;
    w.qt = qt_all;
    w.sv = sv_all;
    w.qh = 0;
    w.qn = 0;

    unsigned long long c0 = 0, c1 = 0, c2 = 0, c3 = 0;
    for (int64_t k = k0; k < k1; ++k) {
        if (!(pflag[k] & 1)) continue;  // fast path: k_sweep, k_gather
        // series forms where |r|^2 <= 1e-8 |x_m|^2 over the whole trajectory (the max over the
        // whole trajectory when given, else over the samples of this call), decided per pixel
        w.rb2 = rbound2 ? rbound2[k] : __longlong_as_double((long long)rmax2[k]);
        const bool all_ser = GEOM == LW_GEOM_EXACT && w.rb2 * invD2max <= kSeriesBound;
        if (GEOM == LW_GEOM_FARFIELD)
            w.template particle<kModeFar>(lane_ok, pix_in, m, k, c0, c1, c2, c3);
        else if (all_ser && rec_ok) {
            if (tail_negligible<kF64>(w.rb2, s2max, sh.C, w.cK, Dref))
                w.template particle<kModeRecLow>(lane_ok, pix_in, m, k, c0, c1, c2, c3);
            else
                w.template particle<kRec>(lane_ok, pix_in, m, k, c0, c1, c2, c3);
        } else
            w.template particle<kModeMixed>(lane_ok, pix_in, m, k, c0, c1, c2, c3);
    }
    while (w.qn > 0) w.drain(w.qn < 64 ? w.qn : 64);

    // counters: block reduction in LDS, then one global atomic per counter
    if (c0) atomicAdd(&red[0], c0);
    if (c1) atomicAdd(&red[1], c1);
    if (c2) atomicAdd(&red[2], c2);
    if (c3) atomicAdd(&red[3], c3);
    __syncthreads();
    if (diag && threadIdx.x < 4 && red[threadIdx.x]) atomicAdd(diag + threadIdx.x, red[threadIdx.x]);
}

// ---------------------------------------------------------------------------------------------
// Fast path.  A block owns a tile of kTilePix pixels and a group of particles (and, where there are
// few of those, a segment of the samples).  For each particle:
//   * a mask of the steps (H intervals) that hold window grid points for some pixel of the tile, from the
//     arrival times at the steps' boundaries alone, lanes over pixels (arrival times increase on this path);
//   * per such step the samples are staged in LDS (scan values, beta, 1/|beta|, beta_dot), in a ring that holds this
//     step's and the one's before, and every pixel's grid points counted;
//   * sparse steps (deposit_points): lanes over (pixel, grid point) pairs.  A lane finds
//     the interval of its grid point (bracket from the pixel's arrival times at five samples of the step, then
//     three-point interpolation), evaluates the field at its two ends and adds the interpolated
//     value to the trace;
//   * dense steps (deposit_dense; at least kDensePoints grid points per interval of a whole step): per pixel, lanes
//     over samples form every arrival time and field of the step in LDS, then lanes over grid
//     points interpolate.
// The interval found is the one with tau_{i-1} < u <= tau_i whichever way it is found, and the
// contribution's arithmetic is the same in both, so a contribution has the same bits.
//
// The traces' atomics set the time: they leave the chip's L2 as requests of at most 64 bytes, and the memory side takes
// 18-20 billion of those a second whatever they hold (285 G floats/s in aligned groups of 16, 98 G/s in runs of 8
// at any place).  A step of the bunch workload has 12 grid points a pixel, 7.1 to a request; so the last points of
// a step wait for the next one where that completes their 64 bytes, which is what the second half of the ring is
// for: 12.8 to a request.  2000 x 20001 samples, 4096 pixels, mixed: 51.3 -> 34.5 ms,
// 6.4e8 requests; with whole requests per wavefront (lanes idle where a step starts or ends inside one) the same.
// The ring's 512 samples (as many as two blocks a compute unit have LDS for) in three steps of 170 intervals or four of
// 127 hold points back longer: 6.15e8 requests, but the steps' own work is there 1.5 or 2 times, 38.7 and 46.1 ms of
// the whole deposit and spectrum instead of 37.6.  (Pixels on the axis have 5 points in 255 intervals.)
template <typename T>
struct SweepCfg {
    static constexpr int NT = sizeof(T) == 8 ? 128 : 256;  // samples of a step, neighbouring steps sharing one
    static constexpr int H = NT - 1;                       // intervals of a step
    static constexpr int R = 2 * NT;                       // ring
    static constexpr int kThreads = 2 * NT;
    static constexpr int G = 64 / (int)sizeof(T);  // elements per request
    static constexpr int kDensePix = sizeof(T) == 8 ? 1 : 2;  // pixels of a dense step at a time
};
constexpr int kSteps = 64;      // steps per mask
// Grid points of a live pixel, per interval of a whole step, from which a step is dense: forming every arrival time and
// field of a step takes a pixel about the same time however few its intervals are.  427 particles of 2 samples, 5687 pixels, at
// most one point each: 1859 us with the step's own intervals in the rule, 507 so.
constexpr float kDensePoints = 0.6f;

template <typename T, int GEOM>
struct SweepLds {
    using Cfg = SweepCfg<T>;
    static constexpr int NP = GEOM == LW_GEOM_FARFIELD ? 2 : (RecLayout<GEOM, sizeof(T) == 8>::DEG + 3) / 2;  // pairs of scan values
    static constexpr int PX = GEOM == LW_GEOM_FARFIELD ? 8 : 6;  // doubles per pixel: o, px, py, then x_m or n, 1/|x_m|
    double2 rec[NP][Cfg::R];  // sample i at i mod R
    double2 be[2][Cfg::R];    // beta_x, beta_y; beta_z, 1/|beta| (0 at rest)
    T acc[3][Cfg::R];         // beta_dot
    double2 px[kTilePix][PX / 2];
    // a pixel's arrival times at the first sample of a step, a quarter, half and three quarters of it and the last,
    // of this step (its parity) and the one before
    double node[2][5][kTilePix];
    double tau[Cfg::kDensePix][Cfg::NT];  // dense steps: the current pixels' arrival times
    T e[Cfg::kDensePix][3][Cfg::NT];      // and fields
    int ulo[kTilePix];       // a pixel's first grid point to deposit
    // of the tile half's pixels before this one: grid points to deposit, those held back by the step before
    int cum[2][kTilePix];
    int tot[2][2], fresh[2];
    int hit[kMaxPartsPerGroup];  // scan mode + 1 of the group's particles that the segment deposits
    uint64_t okm[2];             // usable pixels
    uint64_t live[2];  // pixels with grid points in the step
    uint64_t mask[Cfg::kThreads / 64];
    unsigned long long red[4];
};

template <typename T, int GEOM, int ACC>
struct Sweep {
    static constexpr bool F64 = sizeof(T) == 8;
    using Cfg = SweepCfg<T>;
    using Lds = SweepLds<T, GEOM>;
    Lds &s;
    const double *__restrict__ pt;  // the tile's rows of the pixel table
    T *__restrict__ E;              // the tile's first trace row
    const DepShape &sh;
    DetAcc det;  // from the tile's first trace row
    double cK, Dref, rb2, q;
    int tid;

    // a pixel's constants in the arrival time of MODE
    template <int MODE>
    __device__ __forceinline__ PixC pixel(int p) const
    {
        if constexpr (MODE == kModeMixed) return pixc_row(pt + (size_t)p * kPT);
        PixC P;
        const double2 a = s.px[p][0];
        P.o = a.x;
        P.px = a.y;
        P.py = s.px[p][1].x;
        return P;
    }
    // arrival time of staged sample i at a pixel
    template <int MODE>
    __device__ __forceinline__ double tau_at(const PixC &P, int i) const
    {
        const int j = i & (Cfg::R - 1);
        double v[2 * Lds::NP];
#pragma unroll
        for (int c = 0; c < Lds::NP; ++c) {
            if (2 * c >= ScanVals<GEOM, F64, MODE>::N) break;
            const double2 d = s.rec[c][j];
            v[2 * c] = d.x;
            v[2 * c + 1] = d.y;
        }
        return tau_eval<GEOM, F64, MODE>(P, v, cK, rb2, sh.C);
    }
    // field of staged sample i at pixel p
    template <int MODE>
    __device__ __forceinline__ void field_at(int p, int i, T &ex, T &ey, T &ez) const
    {
        constexpr int X = ScanVals<GEOM, F64, MODE>::X;
        const int j = i & (Cfg::R - 1);
        double v[2 * Lds::NP];
#pragma unroll
        for (int c = X / 2; c <= (X + 2) / 2; ++c) {
            const double2 d = s.rec[c][j];
            v[2 * c] = d.x;
            v[2 * c + 1] = d.y;
        }
        const double2 b01 = s.be[0][j], b23 = s.be[1][j];
        const double2 g1 = s.px[p][1], g2 = s.px[p][2];
        const double xm[3] = {g1.y, g2.x, g2.y};
        PixGeo g;
        g.nx = g1.y;
        g.ny = g2.x;
        g.nz = g2.y;
        if constexpr (GEOM == LW_GEOM_FARFIELD) g.invD = s.px[p][3].x;
        lw_field_ib<T, GEOM>(g, xm, v[X], v[X + 1], v[X + 2], b01.x, b01.y, b23.x, b23.y, s.acc[0][j], s.acc[1][j],
                             s.acc[2][j], q, sh.fmask, ex, ey, ez);
    }
    __device__ __forceinline__ void add(int p, int64_t u, T w, const T *a, const T *b) const
    {
        const T w1 = (T)1 - w;
        const size_t j = (size_t)p * 3 * (size_t)sh.n_obs + (size_t)u;
#pragma unroll
        for (int c = 0; c < 3; ++c)
            put<ACC>(E, det, j + (size_t)c * (size_t)sh.n_obs, 3 * p + c, w1 * a[c] + w * b[c]);
    }
    __device__ __forceinline__ static T inverse(double dt)  // 1/(tau_i - tau_{i-1})
    {
        return F64 ? (T)(1.0 / dt) : (T)__builtin_amdgcn_rcpf((float)dt);
    }
    // the last grid point <= u whose element starts a request (of the pixel's first component; the tile's first
    // element does, 3 kTilePix rows being a multiple of G)
    __device__ __forceinline__ int64_t request_start(int p, int64_t u) const
    {
        const int64_t off = (int64_t)(((uint64_t)p * 3 * (uint64_t)sh.n_obs) & (Cfg::G - 1));
        return ((u + off) & ~(int64_t)(Cfg::G - 1)) - off;
    }

    // Stage samples i0 + 1 .. i0 + n of a particle, and i0 unless the ring holds it (base, rk, bk, dk: its arrival
    // bases, r, beta, beta_dot)
    template <int MODE>
    __device__ __forceinline__ void stage(const double *base, const double *rk, const double *bk, const double *dk, int i0, int n,
                                          bool prev) const
    {
        const int t = tid & (Cfg::NT - 1);
        if (t > n || (t == 0 && prev)) return;
        const int64_t i = i0 + t;
        const int j = (int)i & (Cfg::R - 1);
        if (tid < Cfg::NT) {
            double v[2 * Lds::NP];
            scan_vals<GEOM, F64, MODE>(base[i], rk[3 * i], rk[3 * i + 1], rk[3 * i + 2], sh.C, Dref, v);
#pragma unroll
            for (int c = 0; c < Lds::NP; ++c)
                if (2 * c < ScanVals<GEOM, F64, MODE>::N) s.rec[c][j] = make_double2(v[2 * c], v[2 * c + 1]);
        } else {
            const double bx = bk[3 * i], by = bk[3 * i + 1], bz = bk[3 * i + 2];
            s.be[0][j] = make_double2(bx, by);
            s.be[1][j] = make_double2(bz, inv_beta<T>(bx, by, bz));
#pragma unroll
            for (int c = 0; c < 3; ++c) s.acc[c][j] = (T)dk[3 * i + c];
        }
    }

    // (pixel, grid point) pairs, one per lane: `total` of them, tot0 at the tile's first half of the pixels, pixel p's
    // from ulo[p] on.  The step's samples are i0 .. i0 + n; those of the step before hold the points held back.
    template <int MODE>
    __device__ __forceinline__ void deposit_points(const int *cum, int i0, int n, bool prev, int par, int tot0, int total) const
    {
        for (int it = tid; it < total; it += Cfg::kThreads) {
            int p = it >= tot0 ? 64 : 0;
            const int r = it >= tot0 ? it - tot0 : it;
#pragma unroll
            for (int b = 32; b > 0; b >>= 1)
                if (cum[p + b] <= r) p += b;
            const int u = s.ulo[p] + (r - cum[p]);
            const PixC P = pixel<MODE>(p);
            const double ud = (double)u;
            // the step and the quarter of it that hold the crossing
            const bool old = prev && !(ud > s.node[par][0][p]);
            const double (*nd)[kTilePix] = s.node[old ? par ^ 1 : par];
            const int lo0 = old ? i0 - Cfg::H : i0, len = old ? Cfg::H : n;
            int j = ud > nd[2][p] ? 2 : 0;
            j += ud > nd[j + 1][p] ? 1 : 0;
            int lo = lo0 + ((j * len) >> 2), hi = lo0 + (((j + 1) * len) >> 2);
            double ta = nd[j][p], tb = nd[j + 1][p];
            float ya = (float)(ta - ud), yb = (float)(tb - ud);  // ya < 0 <= yb
            // (a first guess that is a parabola through the node beyond as well saved no arrival time)
            int g = lo + (int)rintf((float)(hi - lo) * (-ya * __builtin_amdgcn_rcpf(yb - ya)));
            for (int k = 0; hi - lo > 1; ++k) {
                g = min(max(g, lo + 1), hi - 1);
                const double tg = tau_at<MODE>(P, g);
                const float yg = (float)(tg - ud), fl = (float)(g - lo), fr = (float)(hi - g);
                // slope at g of the parabola through the bracket's ends and g
                const float d = ((yg - ya) * fr * __builtin_amdgcn_rcpf(fl) + (yb - yg) * fl * __builtin_amdgcn_rcpf(fr)) *
                                __builtin_amdgcn_rcpf(fl + fr);
                const float x = __builtin_amdgcn_fmed3f(-yg * __builtin_amdgcn_rcpf(d), -1e3f, 1e3f);  // from g
                if (tg >= ud) {
                    hi = g;
                    tb = tg;
                    yb = yg;
                    g += (int)floorf(x);
                } else {
                    lo = g;
                    ta = tg;
                    ya = yg;
                    g += (int)ceilf(x);
                }
                if (k >= 4) g = (lo + hi) >> 1;
            }
            T a[3], b[3];
            field_at<MODE>(p, lo, a[0], a[1], a[2]);
            field_at<MODE>(p, hi, b[0], b[1], b[2]);
            add(p, u, (T)(ud - ta) * inverse(tb - ta), a, b);
        }
    }

    // Every pixel's intervals of the step, kDensePix pixels at a time
    template <int MODE>
    __device__ __forceinline__ void deposit_dense(int i0, int n, int par) const
    {
        const double nob = (double)sh.n_obs;
        constexpr int kShare = Cfg::kThreads / Cfg::kDensePix;
        const int hb = tid / kShare, t = tid % kShare;
        uint64_t left[2] = {s.live[0], s.live[1]};
        auto pop = [&]() {
            const int h = left[0] ? 0 : 1;
            if (!left[h]) return -1;
            const int p = 64 * h + (int)__builtin_ctzll(left[h]);
            left[h] &= left[h] - 1;
            return p;
        };
        while (left[0] | left[1]) {  // the same in every thread
            int p = pop();
            if constexpr (Cfg::kDensePix == 2) {
                const int pb = pop();
                if (hb) p = pb;
            }
            __syncthreads();  // the previous pixels' fields are read
            if (p >= 0 && t <= n) {
                s.tau[hb][t] = tau_at<MODE>(pixel<MODE>(p), i0 + t);
                T x, y, z;
                field_at<MODE>(p, i0 + t, x, y, z);
                s.e[hb][0][t] = x;
                s.e[hb][1][t] = y;
                s.e[hb][2][t] = z;
            }
            __syncthreads();
            if (p < 0) continue;
            const int64_t u0 = grid_count(s.node[par][0][p], nob), u1 = grid_count(s.node[par][4][p], nob);
            const double *tau = s.tau[hb];
            for (int64_t u = request_start(p, u0) + t; u < u1; u += kShare) {
                if (u < u0) continue;
                const double ud = (double)u;
                int lo = 0, hi = n;
                double ta = tau[0], tb = tau[n];
                for (int k = 0; hi - lo > 1; ++k) {
                    int g = lo + (int)((float)(hi - lo) * ((float)(ud - ta) * __builtin_amdgcn_rcpf((float)(tb - ta))));
                    g = (k & 3) == 3 ? (lo + hi) >> 1 : min(max(g, lo + 1), hi - 1);
                    const double tg = tau[g];
                    if (tg >= ud) {
                        hi = g;
                        tb = tg;
                    } else {
                        lo = g;
                        ta = tg;
                    }
                }
                const T a[3] = {s.e[hb][0][lo], s.e[hb][1][lo], s.e[hb][2][lo]};
                const T b[3] = {s.e[hb][0][hi], s.e[hb][1][hi], s.e[hb][2][hi]};
                add(p, u, (T)(ud - ta) * inverse(tb - ta), a, b);
            }
        }
    }

    // One particle's steps [st0, st1) (the same in every thread): base, rk, bk, dk as in stage
    template <int MODE>
    __device__ __forceinline__ void particle(const double *base, const double *rk, const double *bk, const double *dk, int st0,
                                             int st1, bool lane_ok) const
    {
        constexpr int kWaves = Cfg::kThreads / 64;
        const int ns = (int)sh.n_samples;
        const double nob = (double)sh.n_obs;
        const int lane = tid & 63, wv = __builtin_amdgcn_readfirstlane(tid >> 6);
        const int p = tid & (kTilePix - 1);
        int last = -2;        // the step staged last
        int64_t unext = 0;    // thread p < kTilePix: pixel p's first grid point not yet deposited
        for (int c0 = st0; c0 < st1; c0 += kSteps) {
            // steps of this chunk with window grid points at some pixel: pairs of wavefronts (pixels) take
            // equal shares of the steps
            const int c1 = min(c0 + kSteps, st1), share = (c1 - c0 + kWaves / 2 - 1) / (kWaves / 2);
            const int a = min(c0 + (wv >> 1) * share, c1), b = min(a + share, c1);
            uint64_t mask = 0;
            if (c1 == c0 + 1 && st1 == st0 + 1) {
                mask = 1;  // one step: the look through the particles has told
            } else if (a < b) {
                const PixC P = pixel<MODE>(p);
                auto count = [&](int st) {  // window grid points up to the first sample of step st
                    const int64_t i = min((int64_t)st * Cfg::H, (int64_t)ns - 1);
                    const cdptr sd = uniform_ptr(base + i), sr = uniform_ptr(rk + 3 * i);
                    double v[2 * Lds::NP];
                    scan_vals<GEOM, F64, MODE>(sd[0], sr[0], sr[1], sr[2], sh.C, Dref, v);
                    return grid_count(tau_eval<GEOM, F64, MODE>(P, v, cK, rb2, sh.C), nob);
                };
                int64_t prev = count(a);
                if (__ballot(lane_ok && count(b) != prev) != 0) {
                    for (int st = a; st < b; ++st) {
                        const int64_t next = count(st + 1);
                        if (__ballot(lane_ok && next != prev) != 0) mask |= 1ull << (st - c0);
                        prev = next;
                    }
                }
            }
            __syncthreads();  // the previous chunk's masks are read
            if (lane == 0) s.mask[wv] = mask;
            __syncthreads();
            mask = 0;
#pragma unroll
            for (int v = 0; v < kWaves; ++v) mask |= s.mask[v];
            while (mask) {
                const int st = c0 + (int)__builtin_ctzll(mask);
                mask &= mask - 1;
                const bool prev = last == st - 1;
                const bool more = st + 1 < c1 && ((mask >> (st + 1 - c0)) & 1);  // the next step follows
                const int par = st & 1, i0 = st * Cfg::H;
                const int n = min(Cfg::H, ns - 1 - i0);  // intervals
                stage<MODE>(base, rk, bk, dk, i0, n, prev);
                __syncthreads();
                if (tid < kTilePix) {
                    double tl = 0.0, th = 0.0;
                    if (lane_ok) {
                        const PixC P = pixel<MODE>(p);
                        tl = tau_at<MODE>(P, i0);
                        th = tau_at<MODE>(P, i0 + n);
                    }
                    s.node[par][0][p] = tl;
                    s.node[par][4][p] = th;
                    const int64_t cl = grid_count(tl, nob), ch = grid_count(th, nob);
                    const int64_t u0 = prev ? unext : cl;
                    // points from the last request's start on wait for the next step, if all of them are this step's
                    const int64_t cut = request_start(p, ch);
                    const int64_t u1 = more && cut >= cl ? cut : ch;
                    s.ulo[p] = (int)u0;
                    // counts above 2^20 make the step dense, where they are not used
                    const int fresh = (int)min(ch - cl, (int64_t)1 << 20), held = (int)(cl - u0);
                    const int cnt = (int)min(u1 - u0, (int64_t)1 << 20);
                    int sum = cnt, sumh = held, sumf = fresh;
#pragma unroll
                    for (int off = 1; off < 64; off <<= 1) {
                        const int o = __shfl_up(sum, off), oh = __shfl_up(sumh, off), of = __shfl_up(sumf, off);
                        if (lane >= off) {
                            sum += o;
                            sumh += oh;
                            sumf += of;
                        }
                    }
                    s.cum[0][p] = sum - cnt;
                    s.cum[1][p] = sumh - held;
                    const uint64_t live = __ballot(fresh > 0);
                    if (lane == 63) {
                        s.tot[0][wv] = sum;
                        s.tot[1][wv] = sumh;
                        s.fresh[wv] = sumf;
                        s.live[wv] = live;
                    }
                    unext = u1;
                }
                for (int c = tid / kTilePix; c >= 1 && c <= 3; c += Cfg::kThreads / kTilePix - 1)
                    s.node[par][c][p] = lane_ok ? tau_at<MODE>(pixel<MODE>(p), i0 + ((c * n) >> 2)) : 0.0;
                __syncthreads();
                const bool dense = (float)(s.fresh[0] + s.fresh[1]) >=
                                   kDensePoints * (float)((__popcll(s.live[0]) + __popcll(s.live[1])) * Cfg::H);
                const int d = dense ? 1 : 0, tot0 = s.tot[d][0], total = tot0 + s.tot[d][1];
                deposit_points<MODE>(s.cum[d], i0, n, prev, par, tot0, total);
                if (dense) {
                    if (tid < kTilePix) unext = grid_count(s.node[par][4][p], nob);
                    deposit_dense<MODE>(i0, n, par);
                }
                last = st;
                __syncthreads();  // the step is read
            }
        }
    }
};

// segments of the samples, in steps
struct SweepShape {
    int n_seg, per_seg, n_steps;
};

template <typename T, int GEOM, int ACC>
__global__ __launch_bounds__(SweepCfg<T>::kThreads) __attribute__((amdgpu_waves_per_eu(sizeof(T) == 4 ? 4 : 3))) void k_sweep(
    const double *__restrict__ r, const double *__restrict__ beta, const double *__restrict__ beta_dot,
    const double *__restrict__ charge, const double *__restrict__ x_det, const double *__restrict__ base,
    const double *__restrict__ pt, const int *__restrict__ pflag, const unsigned long long *__restrict__ rmax2,
    const double *__restrict__ rbound2, T *__restrict__ E, unsigned long long *__restrict__ diag, DepShape sh, SweepShape sw,
    DetAcc det)
{
    constexpr bool kF64 = sizeof(T) == 8;
    constexpr int kRec = kF64 ? kModeRec5 : kModeRec3;
    __shared__ SweepLds<T, GEOM> lds;
    const int tid = threadIdx.x, p = tid & (kTilePix - 1);
    // block -> (particle group and segment, tile); blocks go to the 8 XCDs round robin, and all tiles
    // of a group run on one XCD at once, so that they share its samples in that L2
    const int64_t b = blockIdx.x;
    const int64_t xcd = b & 7, slot = b >> 3;
    const int64_t unit = (slot / sh.n_tiles) * 8 + xcd;
    const int64_t tile = slot % sh.n_tiles;
    const int64_t grp = unit / sw.n_seg;
    const int seg = (int)(unit - grp * sw.n_seg);
    if (grp >= sh.n_groups) return;  // padding block
    const int64_t k0 = grp * sh.parts_per_group, k1 = std::min(k0 + sh.parts_per_group, sh.n_particles);
    const int st0 = seg * sw.per_seg, st1 = min(st0 + sw.per_seg, sw.n_steps);
    const int others = *gather_flag(pt) ? 3 : 1;  // flags of other kernels' particles
    {
        // no particle of the group is this kernel's (a group is at most a wavefront's lanes)
        const int64_t k = k0 + (tid & 63);
        if (__ballot(k < k1 && (pflag[k] & others) == 0) == 0) return;
    }

    if (tid < 4) lds.red[tid] = 0ull;
    const int64_t m = tile * kTilePix + p;
    const bool pix_in = m < sh.n_pix;
    const double Dref = pix_geo(x_det, 0).D;  // the polynomials' pixel distance
    bool lane_ok, far_off = false;
    double id2 = 0.0, s2 = 0.0;
    {
        // rows past the pass's last pixel are zero padding (not usable)
        const PixC pc = pixc_row(pt + m * kPT);
        lane_ok = pix_in && pc.g.ok;
        if (tid < kTilePix) {
            double g0 = pc.g.nx, g1 = pc.g.ny, g2 = pc.g.nz;
            if (GEOM == LW_GEOM_EXACT) {
                g0 = pix_in ? x_det[3 * m] : 0.0;
                g1 = pix_in ? x_det[3 * m + 1] : 0.0;
                g2 = pix_in ? x_det[3 * m + 2] : 0.0;
            }
            lds.px[p][0] = make_double2(pc.o, pc.px);
            lds.px[p][1] = make_double2(pc.py, g0);
            lds.px[p][2] = make_double2(g1, g2);
            if constexpr (GEOM == LW_GEOM_FARFIELD) lds.px[p][3] = make_double2(pc.g.invD, 0.0);
        }
        if (lane_ok) {
            id2 = pc.g.invD * pc.g.invD;
            s2 = fmax(0.0, 2.0 * (1.0 - pc.g.nz));
            far_off = !(fabs(pc.g.D - Dref) <= kSameDistance * Dref);
        }
    }
    // over the tile's pixels: its two halves are wavefronts 0, 1 (and again the later ones)
    for (int off = 32; off > 0; off >>= 1) {
        id2 = fmax(id2, __shfl_xor(id2, off));
        s2 = fmax(s2, __shfl_xor(s2, off));
    }
    const uint64_t off_mask = __ballot(far_off), ok_mask = __ballot(lane_ok);
    if ((tid & 63) == 0 && tid < kTilePix) {
        lds.node[0][0][tid >> 6] = id2;
        lds.node[0][1][tid >> 6] = s2;
        lds.mask[tid >> 6] = off_mask;
        lds.okm[tid >> 6] = ok_mask;
    }
    __syncthreads();
    const double invD2max = fmax(lds.node[0][0][0], lds.node[0][0][1]), s2max = fmax(lds.node[0][1][0], lds.node[0][1][1]);
    const bool rec_ok = GEOM == LW_GEOM_EXACT && (lds.mask[0] | lds.mask[1]) == 0;

    const size_t row0 = (size_t)(tile * kTilePix) * 3;
    if constexpr (ACC != kAccFloat) {
        det.hi += row0 * (size_t)sh.n_obs;
        det.scale += row0;
    }
    Sweep<T, GEOM, ACC> w{lds, pt + (size_t)(tile * kTilePix) * kPT, E + row0 * (size_t)sh.n_obs, sh, det, 0.0, Dref, 0.0, 0.0, tid};
    {
        double c[6];
        tau_poly<kF64 ? 5 : 3>(0.0, 0.0, 0.0, 0.0, sh.C, Dref, c);
        w.cK = c[kF64 ? 5 : 3];
    }
    const double nob = (double)sh.n_obs;
    unsigned long long c1 = 0, c2 = 0, c3 = 0;
    // the particle's constants, then f with its scan mode
    auto with_mode = [&](int64_t k, auto f) {
        // series forms where |r|^2 <= 1e-8 |x_m|^2 over the whole trajectory (the max over the
        // whole trajectory when given, else over the samples of this call), decided per pixel
        w.rb2 = rbound2 ? rbound2[k] : __longlong_as_double((long long)rmax2[k]);
        w.q = charge ? charge[k] : -kQe;
        if constexpr (GEOM == LW_GEOM_FARFIELD) {
            f(std::integral_constant<int, kModeFar>{});
        } else {
            const bool all_ser = w.rb2 * invD2max <= kSeriesBound;
            if (all_ser && rec_ok) {
                if (tail_negligible<kF64>(w.rb2, s2max, sh.C, w.cK, Dref))
                    f(std::integral_constant<int, kModeRecLow>{});
                else
                    f(std::integral_constant<int, kRec>{});
            } else
                f(std::integral_constant<int, kModeMixed>{});
        }
    };
    // the group's particles whose arrival times pass window grid points within the segment, at some pixel: a
    // wavefront per particle, lanes over pixels; and the counters, which follow from the first and last arrival times
    const int nk = (int)(k1 - k0), lane = tid & 63;
    for (int kk = __builtin_amdgcn_readfirstlane(tid >> 6); kk < nk; kk += SweepCfg<T>::kThreads / 64) {
        const int64_t k = k0 + kk;
        int hit = 0;
        if ((pflag[k] & others) == 0) {  // else careful path (k_careful) or dense (k_gather)
            const size_t s0 = (size_t)k * sh.n_samples;
            with_mode(k, [&](auto mode) {
                constexpr int MODE = decltype(mode)::value;
                const int64_t ie[3] = {std::min<int64_t>((int64_t)st0 * SweepCfg<T>::H, sh.n_samples - 1),
                                       std::min<int64_t>((int64_t)st1 * SweepCfg<T>::H, sh.n_samples - 1), sh.n_samples - 1};
                const int ne = seg == 0 && ie[1] < ie[2] ? 3 : 2;
                double v[3][ScanVals<GEOM, kF64, MODE>::N];
#pragma unroll
                for (int e = 0; e < 3; ++e) {
                    if (e >= ne) break;
                    const cdptr sd = uniform_ptr(base + s0 + ie[e]), sr = uniform_ptr(r + 3 * (s0 + ie[e]));
                    scan_vals<GEOM, kF64, MODE>(sd[0], sr[0], sr[1], sr[2], sh.C, Dref, v[e]);
                }
                bool any = false;
#pragma unroll
                for (int h = 0; h < 2; ++h) {
                    const bool in = tile * kTilePix + 64 * h + lane < sh.n_pix, ok = (lds.okm[h] >> lane) & 1;
                    const PixC P = w.template pixel<MODE>(64 * h + lane);
                    const double t0 = tau_eval<GEOM, kF64, MODE>(P, v[0], w.cK, w.rb2, sh.C);
                    const double t1 = tau_eval<GEOM, kF64, MODE>(P, v[1], w.cK, w.rb2, sh.C);
                    any |= ok && grid_count(t1, nob) != grid_count(t0, nob);
                    if (seg == 0 && ok) {
                        const double te = ne == 3 ? tau_eval<GEOM, kF64, MODE>(P, v[2], w.cK, w.rb2, sh.C) : t1;
                        const int64_t inside = grid_count(te, nob) - grid_count(t0, nob);
                        c3 += (unsigned long long)inside;
                        c2 += (unsigned long long)((int64_t)(floor(te) - floor(t0)) - inside);
                    } else if (seg == 0 && in) {
                        c1 += (unsigned long long)(sh.n_samples - 1);
                    }
                }
                hit = __ballot(any) != 0 ? MODE + 1 : 0;
            });
        }
        if (lane == 0) lds.hit[kk] = hit;
    }
    __syncthreads();
    for (int kk = 0; kk < nk; ++kk) {
        if (!lds.hit[kk]) continue;
        const int64_t k = k0 + kk;
        const size_t s0 = (size_t)k * sh.n_samples;
        with_mode(k, [&](auto mode) {
            w.template particle<decltype(mode)::value>(base + s0, r + 3 * s0, beta + 3 * s0, beta_dot + 3 * s0, st0, st1, lane_ok);
        });
    }

    // counters: block reduction in LDS, then one global atomic per counter
    if (c1) atomicAdd(&lds.red[1], c1);
    if (c2) atomicAdd(&lds.red[2], c2);
    if (c3) atomicAdd(&lds.red[3], c3);
    __syncthreads();
    if (diag && tid < 4 && lds.red[tid]) atomicAdd(diag + tid, lds.red[tid]);
}

// ---------------------------------------------------------------------------------------------
// Dense particles (gather_rule) of short trajectories: an observer grid much finer than the samples, where a particle's
// points run over thousands of grid points.  A block owns a window of grid points of one pixel, finds the particles whose
// arrival times pass it, forms their arrival times and fields at the samples that bound it and adds the interpolated values to
// its grid points in registers: one read and write of the trace instead of three atomics per point, which bound k_sweep here
// (18 G requests/s).  1280 particles x 101 samples on 2^20 points, one pixel, mixed: 174 -> 140 us.  Four wavefronts per
// SIMD: with three (139 registers instead of 128) 43851 particles x 22 samples on 526165 points, 3 pixels, 2814 us, so 2347.
template <typename T>
struct GatherCfg {
    static constexpr int U = 16 / (int)sizeof(T);  // grid points per thread (twice that: 20 us more, half: 30 more)
    static constexpr int W = 256 * U;
};

template <typename T, int GEOM>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(4))) void k_gather(const double *__restrict__ r, const double *__restrict__ beta,
                                                const double *__restrict__ beta_dot, const double *__restrict__ charge,
                                                const double *__restrict__ x_det, const double *__restrict__ base,
                                                const double *__restrict__ pt, const int *__restrict__ pflag,
                                                const unsigned long long *__restrict__ rmax2,
                                                const double *__restrict__ rbound2, T *__restrict__ E,
                                                unsigned long long *__restrict__ diag, DepShape sh)
{
    constexpr bool kF64 = sizeof(T) == 8;
    constexpr int kRec = kF64 ? kModeRec5 : kModeRec3, U = GatherCfg<T>::U, W = GatherCfg<T>::W;
    if (*gather_flag(pt) == 0) return;
    __shared__ double s_tau[256];
    __shared__ T s_e[3][256];
    __shared__ int s_list[256], s_cnt[4];
    __shared__ double s_red[2][2];
    __shared__ uint64_t s_far[2];
    const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
    const double Dref = pix_geo(x_det, 0).D, nob = (double)sh.n_obs;
    const int ns = (int)sh.n_samples;
    double cK;
    {
        double c[6];
        tau_poly<kF64 ? 5 : 3>(0.0, 0.0, 0.0, 0.0, sh.C, Dref, c);
        cK = c[kF64 ? 5 : 3];
    }
    const int64_t n_win = (sh.n_obs + W - 1) / W;
    for (int64_t item = blockIdx.x; item < n_win * sh.n_pix; item += gridDim.x) {
        const int64_t m = item / n_win, U0 = (item - m * n_win) * W, U1 = std::min<int64_t>(U0 + W, sh.n_obs);
        const PixC P = pixc_row(pt + m * kPT);
        const bool counts = diag && U0 == 0;  // the first window's blocks keep the counters
        if (!P.g.ok && !counts) continue;
        const double xm[3] = {x_det[3 * m], x_det[3 * m + 1], x_det[3 * m + 2]};
        unsigned long long n_bad = 0, n_out = 0, n_in = 0;
        // the pixel's tile decides the arrival-time form, as in k_sweep
        __syncthreads();  // the previous window is done with
        if (tid < kTilePix) {
            const int64_t mt = m / kTilePix * kTilePix + tid;
            const PixC pc = pixc_row(pt + mt * kPT);  // padding rows: not usable
            const bool ok = mt < sh.n_pix && pc.g.ok;
            double id2 = ok ? pc.g.invD * pc.g.invD : 0.0, s2 = ok ? fmax(0.0, 2.0 * (1.0 - pc.g.nz)) : 0.0;
            const uint64_t far = __ballot(ok && !(fabs(pc.g.D - Dref) <= kSameDistance * Dref));
            for (int off = 32; off > 0; off >>= 1) {
                id2 = fmax(id2, __shfl_xor(id2, off));
                s2 = fmax(s2, __shfl_xor(s2, off));
            }
            if (lane == 0) {
                s_red[wv][0] = id2;
                s_red[wv][1] = s2;
                s_far[wv] = far;
            }
        }
        __syncthreads();
        const double invD2max = fmax(s_red[0][0], s_red[1][0]), s2max = fmax(s_red[0][1], s_red[1][1]);
        const bool rec_ok = GEOM == LW_GEOM_EXACT && (s_far[0] | s_far[1]) == 0;
        auto with_mode = [&](int64_t k, auto f) {
            const double rb2 = rbound2 ? rbound2[k] : __longlong_as_double((long long)rmax2[k]);
            if constexpr (GEOM == LW_GEOM_FARFIELD) {
                f(std::integral_constant<int, kModeFar>{}, rb2);
            } else {
                if (rb2 * invD2max <= kSeriesBound && rec_ok) {
                    if (tail_negligible<kF64>(rb2, s2max, sh.C, cK, Dref))
                        f(std::integral_constant<int, kModeRecLow>{}, rb2);
                    else
                        f(std::integral_constant<int, kRec>{}, rb2);
                } else
                    f(std::integral_constant<int, kModeMixed>{}, rb2);
            }
        };
        auto tau_of = [&](auto mode, double rb2, int64_t s) {  // of sample s (of all particles)
            constexpr int MODE = decltype(mode)::value;
            double v[ScanVals<GEOM, kF64, MODE>::N];
            scan_vals<GEOM, kF64, MODE>(base[s], r[3 * s], r[3 * s + 1], r[3 * s + 2], sh.C, Dref, v);
            return tau_eval<GEOM, kF64, MODE>(P, v, cK, rb2, sh.C);
        };
        T acc[U][3];
#pragma unroll
        for (int q = 0; q < U; ++q) acc[q][0] = acc[q][1] = acc[q][2] = (T)0;
        bool any = false;  // the same in every thread
        for (int64_t kb = 0; kb < sh.n_particles; kb += 256) {
            const int64_t k = kb + tid;
            bool hit = false;
            if (k < sh.n_particles && pflag[k] == 2 && P.g.ok) {
                with_mode(k, [&](auto mode, double rb2) {
                    const double t0 = tau_of(mode, rb2, k * ns), t1 = tau_of(mode, rb2, k * ns + ns - 1);
                    const int64_t c0 = grid_count(t0, nob), c1 = grid_count(t1, nob);
                    hit = c1 > c0 && c1 > U0 && c0 < U1;
                    n_in += (unsigned long long)(c1 - c0);
                    n_out += (unsigned long long)((int64_t)(floor(t1) - floor(t0)) - (c1 - c0));
                });
            } else if (k < sh.n_particles && pflag[k] == 2) {
                n_bad += (unsigned long long)(ns - 1);
            }
            const uint64_t hm = __ballot(hit);
            __syncthreads();  // the previous list is done with
            if (lane == 0) s_cnt[wv] = (int)__popcll(hm);
            __syncthreads();
            int before = 0, total = 0;
            for (int v = 0; v < 4; ++v) {
                before += v < wv ? s_cnt[v] : 0;
                total += s_cnt[v];
            }
            if (hit) s_list[before + (int)lanes_below(hm)] = tid;
            __syncthreads();
            any |= total > 0;
            for (int e = 0; e < total; ++e) {
                const int64_t kk = kb + s_list[e], s0 = kk * ns;
                const double q = charge ? charge[kk] : -kQe;
                with_mode(kk, [&](auto mode, double rb2) {
                    for (int j0 = 0; j0 + 1 < ns; j0 += 255) {
                        const int n = min(255, ns - 1 - j0);
                        __syncthreads();  // the previous samples are read
                        if (tid <= n) s_tau[tid] = tau_of(mode, rb2, s0 + j0 + tid);
                        __syncthreads();
                        const int64_t c0 = grid_count(s_tau[0], nob), c1 = grid_count(s_tau[n], nob);
                        if (c1 <= U0) continue;
                        if (c0 >= U1) break;
                        // fields at the samples of intervals that reach into the window
                        if (tid <= n && s_tau[min(tid + 1, n)] >= (double)U0 && s_tau[max(tid - 1, 0)] < (double)U1) {
                            const int64_t s = s0 + j0 + tid;
                            const double bx = beta[3 * s], by = beta[3 * s + 1], bz = beta[3 * s + 2];
                            T x, y, z;
                            lw_field_ib<T, GEOM>(P.g, xm, r[3 * s], r[3 * s + 1], r[3 * s + 2], bx, by, bz, inv_beta<T>(bx, by, bz),
                                                 (T)beta_dot[3 * s], (T)beta_dot[3 * s + 1], (T)beta_dot[3 * s + 2], q, sh.fmask, x,
                                                 y, z);
                            s_e[0][tid] = x;
                            s_e[1][tid] = y;
                            s_e[2][tid] = z;
                        }
                        __syncthreads();
#pragma unroll
                        for (int i = 0; i < U; ++i) {
                            const int64_t u = U0 + tid + 256 * i;
                            if (u < c0 || u >= c1) continue;  // c1 <= n_obs
                            const double ud = (double)u;
                            int lo = 0, hi = n;
                            double ta = s_tau[0], tb = s_tau[n];
                            for (int it = 0; hi - lo > 1; ++it) {
                                int g = lo + (int)((float)(hi - lo) * ((float)(ud - ta) * __builtin_amdgcn_rcpf((float)(tb - ta))));
                                g = (it & 3) == 3 ? (lo + hi) >> 1 : min(max(g, lo + 1), hi - 1);
                                const double tg = s_tau[g];
                                if (tg >= ud) {
                                    hi = g;
                                    tb = tg;
                                } else {
                                    lo = g;
                                    ta = tg;
                                }
                            }
                            const T inv = kF64 ? (T)(1.0 / (tb - ta)) : (T)__builtin_amdgcn_rcpf((float)(tb - ta));
                            const T w = (T)(ud - ta) * inv, w1 = (T)1 - w;
#pragma unroll
                            for (int c = 0; c < 3; ++c) acc[i][c] += w1 * s_e[c][lo] + w * s_e[c][hi];
                        }
                    }
                });
            }
        }
        if (counts) {
            for (int off = 32; off > 0; off >>= 1) {
                n_bad += __shfl_xor(n_bad, off);
                n_out += __shfl_xor(n_out, off);
                n_in += __shfl_xor(n_in, off);
            }
            if (lane == 0) {
                if (n_bad) atomicAdd(diag + 1, n_bad);
                if (n_out) atomicAdd(diag + 2, n_out);
                if (n_in) atomicAdd(diag + 3, n_in);
            }
        }
        if (!any) continue;
#pragma unroll
        for (int i = 0; i < U; ++i) {
            const int64_t u = U0 + tid + 256 * i;
            if (u >= U1) continue;
            T *o = E + (size_t)m * 3 * (size_t)sh.n_obs + (size_t)u;
#pragma unroll
            for (int c = 0; c < 3; ++c) o[(size_t)c * (size_t)sh.n_obs] += acc[i][c];
        }
    }
}

// Row scales of the fixed-point pass from the first pass's max |v| per element (bits of a
// non-negative double): scale = 2^(62 - e) where max < 2^e, so every |v| * scale < 2^62.  A row
// that received nothing takes 1; a row with a non-finite contribution takes NaN and is NaN in the
// result.
__global__ __launch_bounds__(256) void k_det_scale(const unsigned long long *__restrict__ mx, int64_t n_rows,
                                                   int64_t n_obs, double *__restrict__ scale)
{
    __shared__ unsigned long long red[256];
    for (int64_t row = blockIdx.x; row < n_rows; row += gridDim.x) {
        const unsigned long long *p = mx + (size_t)row * (size_t)n_obs;
        unsigned long long v = 0;
        for (int64_t u = threadIdx.x; u < n_obs; u += 256) v = p[u] > v ? p[u] : v;
        red[threadIdx.x] = v;
        __syncthreads();
        for (int h = 128; h > 0; h >>= 1) {
            if ((int)threadIdx.x < h && red[threadIdx.x + h] > red[threadIdx.x]) red[threadIdx.x] = red[threadIdx.x + h];
            __syncthreads();
        }
        if (threadIdx.x == 0) {
            const double M = __longlong_as_double((long long)red[0]);
            double sc = 1.0;
            if (!isfinite(M)) {
                sc = NAN;
            } else if (M > 0.0) {
                int e;
                frexp(M, &e);
                sc = ldexp(1.0, 62 - e < 1023 ? 62 - e : 1023);
            }
            scale[row] = sc;
        }
        __syncthreads();
    }
}

// The 128-bit sums (low words in E, high words in hi) to doubles, in place, then divided by the
// row's power of two.  A sum that fits in 64 bits converts with one rounding; a larger one is
// hi 2^64 + lo through the fma, where the rounding of lo (at most 2^10) is at most half an ulp of
// the result (|result| >= 2^63): at most one ulp in all.
__global__ __launch_bounds__(256) void k_det_finish(double *__restrict__ E, const unsigned long long *__restrict__ hi,
                                                    const double *__restrict__ scale, int64_t n_rows, int64_t n_obs)
{
    const size_t n = (size_t)n_rows * (size_t)n_obs;
    for (size_t j = (size_t)blockIdx.x * blockDim.x + threadIdx.x; j < n; j += (size_t)gridDim.x * blockDim.x) {
        const double sc = scale[j / (size_t)n_obs];
        const unsigned long long lo = (unsigned long long)__double_as_longlong(E[j]);
        const long long h = (long long)hi[j], sl = (long long)lo;
        const double v = h == (sl < 0 ? -1ll : 0ll) ? (double)sl : fma((double)h, 0x1p64, (double)lo);
        E[j] = isnan(sc) ? NAN : v * (1.0 / sc);
    }
}

}  // namespace

size_t det_acc_bytes(int64_t n_pix, int64_t n_obs)
{
    return align_up((size_t)n_pix * 3 * (size_t)n_obs * 8, 256) + align_up((size_t)n_pix * 3 * 8, 256);
}

// Two deposits with the same per-contribution values: the first finds max |v| per trace element,
// the second adds the contributions as 128-bit fixed-point integers scaled per row by the first's
// maximum; the integer sums do not depend on the order in which the atomics land.
lw_status launch_deposit_det(const lw_traj_t *t, const lw_grid_t *gr, int fmask, int geom, double *E, int64_t *diag,
                             void *acc, void *ws, size_t ws_bytes, hipStream_t s)
{
    const int64_t rows = gr->n_pix * 3, n_obs = gr->n_obs;
    const size_t n_el = (size_t)rows * (size_t)n_obs;
    double *scale = (double *)((char *)acc + align_up(n_el * 8, 256));
    const DetAcc det{(unsigned long long *)acc, scale};
    const bool boris = t->kind == LW_TRAJ_BORIS;
    auto pass = [&](int mode, int64_t *dg) {
        return boris ? launch_deposit_boris(t, gr, LW_PREC_FP64, fmask, geom, false, E, dg, ws, ws_bytes, s, mode, det)
                     : launch_deposit(t, gr, LW_PREC_FP64, fmask, geom, false, E, dg, ws, ws_bytes, s, 0, nullptr, mode,
                                      det);
    };
    if (n_el == 0) return pass(kAccFixed, diag);  // nothing to deposit: the diag reset only
    lw_status st = pass(kAccMaxAbs, nullptr);
    if (st != LW_OK) return st;
    k_det_scale<<<(unsigned)std::min<int64_t>(rows, 65536), 256, 0, s>>>((const unsigned long long *)E, rows, n_obs,
                                                                        scale);
    const unsigned blocks = (unsigned)std::min<size_t>((n_el + 255) / 256, 65536);
    k_fill<unsigned long long><<<blocks, 256, 0, s>>>(det.hi, (int64_t)n_el);
    if ((st = check_launch("lw_deposit_td_det")) != LW_OK) return st;
    if ((st = pass(kAccFixed, diag)) != LW_OK) return st;
    k_det_finish<<<blocks, 256, 0, s>>>(E, det.hi, scale, rows, n_obs);
    return check_launch("lw_deposit_td_det");
}

size_t deposit_ws_bytes(int64_t n_particles, int64_t n_samples)
{
    return ws_bytes_for(n_particles, n_samples);
}

// Particles from which the pusher leaves the arrival bases: its chains take longer for them, the pre-pass reads every
// sample again.  Deposit of pushed trajectories of 10001 samples, bases from the pre-pass and from the pusher: 500
// particles 2.82 and 2.88 ms, 1000 2.84 and 2.82, 1500 3.10 and 2.99, 2048 3.22 and 2.99, 8192 4.57 and 3.24; of 1001
// samples 1500 464 and 456 us, 8192 833 and 668.
constexpr int64_t kPrePushed = 1500;

// whether k_gather may take dense particles: whole short trajectories (every span of a longer one takes the same path)
// on a grid that is long against them
static bool gather_allowed(int64_t ns, bool whole, int64_t n_obs, int acc_mode)
{
    return acc_mode == kAccFloat && whole && ns >= 2 && ns <= kGatherSamples && n_obs >= 4 * ns;
}

DepositPre deposit_pre(void *ws, int64_t n_p, int64_t ns, bool whole, const lw_grid_t *gr, int acc_mode)
{
    DepositPre pre;
    pre.whole = whole;
    if (gather_allowed(ns, whole, gr->n_obs, acc_mode) || n_p < kPrePushed) return pre;
    const DepWs w = carve(ws, n_p);
    pre.base = w.d;
    pre.pflag = w.pflag;
    pre.t0 = gr->t0;
    pre.dt_obs = gr->dt_obs;
    pre.C = 1.0 / (kC * gr->dt_obs);
    return pre;
}

lw_status launch_deposit(const lw_traj_t *t, const lw_grid_t *gr, int prec, int fmask, int geom, bool accumulate,
                         void *E, int64_t *diag, void *ws, size_t ws_bytes, hipStream_t s, int64_t sample0,
                         const double *rbound2, int acc_mode, DetAcc det, const DepositPre *pre)
{
    const int64_t n_p = t->n_particles, ns = t->n_samples, n_pix = gr->n_pix, n_obs = gr->n_obs;
    const bool cull = (geom & LW_CULL) != 0;
    geom &= ~LW_CULL;
    const size_t trace_elems = (size_t)n_pix * 3 * (size_t)n_obs;
    const bool f64 = prec == LW_PREC_FP64, prepassed = pre && pre->base;
    if (acc_mode != kAccFloat && (!f64 || cull))
        return fail(LW_E_UNSUPPORTED, "lw_deposit_td_det: FP64 without culling only");
    if (n_obs > 0x7fffffff) return fail(LW_E_SHAPE, "lw_deposit_td: n_obs must be below 2^31");
    if (ns > 0x7fffffff) return fail(LW_E_SHAPE, "lw_deposit_td: too many samples");
    const double C = 1.0 / (kC * gr->dt_obs);
    // the trace's and counters' zeros (accumulate: none), with the setup of the first launch
    SetupShape su{0, 0, 0, 0, 0, C};
    unsigned long long *diag0 = nullptr;
    if (!accumulate) {
        const size_t words = trace_elems * (f64 ? 2 : 1);
        su.n_trace = (int64_t)(words / 4);
        su.n_tail = (int64_t)(words % 4);
        diag0 = (unsigned long long *)diag;
    }
    auto setup = [&](const DepWs *w, const double *xd) {
        const int64_t most = std::max({su.n_trace, su.n_p, su.n_rows, (int64_t)1});
        k_setup<<<(unsigned)std::min<int64_t>((most + 255) / 256, 16384), 256, 0, s>>>(
            (uint4 *)E, diag0, w ? w->pflag : nullptr, w ? w->rmax2 : nullptr, xd, w ? w->pt : nullptr, su);
        su.n_trace = su.n_tail = 0;
        diag0 = nullptr;
    };
    if (n_p == 0 || n_pix == 0 || ns == 0) {
        if (!accumulate) setup(nullptr, nullptr);
        return check_launch("deposit fill");
    }
    // particles per launch: all of them, or as many as the workspace holds arrival bases for and the grids
    // reach: those count their threads in 32 bits (256 per particle in the pre-pass, 16 per particle and tile in
    // k_careful, 8 per particle, tile and segment in k_sweep)
    const int64_t most_tiles = (std::min<int64_t>(n_pix, kPixTabMax) + kTilePix - 1) / kTilePix;
    int64_t chunk = std::min<int64_t>({n_p, kMaxParticles, std::max<int64_t>(1, kMaxUnits / most_tiles)});
    while (chunk > 1 && ws_bytes_for(chunk, ns) > ws_bytes) chunk = std::max<int64_t>(1, chunk / 2);
    if (ws_bytes_for(chunk, ns) > ws_bytes)
        return fail(LW_E_WORKSPACE, "lw_deposit_td: workspace of %zu bytes holds no particle (%zu needed)", ws_bytes,
                    ws_bytes_for(1, ns));
    if (prepassed && (chunk < n_p || !rbound2))
        return fail(LW_E_WORKSPACE, "lw_deposit_td: pushed arrival bases of a part of the particles");
    const int64_t n_chunks_s = (ns + kPrepassChunk - 1) / kPrepassChunk;
    if (n_chunks_s > 65535) return fail(LW_E_SHAPE, "lw_deposit_td: too many samples");
    // pixel passes of at most kPixTabMax pixels (the pixel table's share of the workspace); each
    // pass is a deposit of its own pixels (its first pixel is the reference)
    for (int64_t m0 = 0; m0 < n_pix; m0 += kPixTabMax) {
        const int64_t npx = std::min<int64_t>(kPixTabMax, n_pix - m0);
        const double *xd = gr->x_det + 3 * m0;
        void *Ep = f64 ? (void *)((double *)E + (size_t)m0 * 3 * (size_t)n_obs)
                       : (void *)((float *)E + (size_t)m0 * 3 * (size_t)n_obs);
        // the pass's rows of the order-independent accumulators
        const DetAcc dp{det.hi ? det.hi + (size_t)m0 * 3 * (size_t)n_obs : nullptr,
                        det.scale ? det.scale + (size_t)m0 * 3 : nullptr};
        for (int64_t p0 = 0; p0 < n_p; p0 += chunk) {
            const int64_t np = std::min<int64_t>(chunk, n_p - p0);
            DepShape sh;
            sh.n_particles = np;
            sh.n_samples = ns;
            sh.n_pix = npx;
            sh.n_obs = n_obs;
            sh.n_tiles = (npx + kTilePix - 1) / kTilePix;
            const int step = f64 ? SweepCfg<double>::H : SweepCfg<float>::H;
            SweepShape sw;
            sw.n_steps = (int)((ns - 1 + step - 1) / step);
            const int64_t seg_len = f64 ? kSegIntervals64 : kSegIntervals;
            const int64_t units = np * sh.n_tiles, least = (ns + seg_len - 1) / seg_len;
            const int64_t want = std::max<int64_t>({1, least, std::min<int64_t>(sw.n_steps, (kFillBlocks + units - 1) / units)});
            sw.per_seg = (int)((sw.n_steps + want - 1) / want);
            sw.n_seg = sw.per_seg > 0 ? (sw.n_steps + sw.per_seg - 1) / sw.per_seg : 1;
            const int64_t target = sw.n_steps > 1 ? kTargetBlocks : kTargetBlocksShort;
            sh.parts_per_group = std::max<int64_t>(1, std::min<int64_t>(kMaxPartsPerGroup, units * sw.n_seg / target));
            sh.n_groups = (np + sh.parts_per_group - 1) / sh.parts_per_group;
            sh.fmask = fmask;
            sh.C = C;
            const int64_t blocks = (sh.n_groups * sw.n_seg + 7) / 8 * 8 * sh.n_tiles;
            DepShape shc = sh;
            shc.parts_per_group = std::max<int64_t>(1, std::min<int64_t>(kMaxPartsCareful, units / kTargetBlocks));
            shc.n_groups = (np + shc.parts_per_group - 1) / shc.parts_per_group;
            const int64_t blocks_careful = (shc.n_groups + 7) / 8 * 8 * sh.n_tiles;
            if (std::max(blocks, blocks_careful) > 0x7fffffff)
                return fail(LW_E_SHAPE, "lw_deposit_td: problem too large for one launch");
            const DepWs w = carve(ws, np);
            su.n_p = prepassed ? 0 : np;
            su.n_pix = npx;
            su.n_rows = p0 == 0 ? sh.n_tiles * kTilePix : 0;  // <= kPixTabMax
            setup(&w, xd);
            const double *r = t->r + (size_t)p0 * ns * 3, *b = t->beta + (size_t)p0 * ns * 3,
                         *bd = t->beta_dot + (size_t)p0 * ns * 3;
            const double *charge = t->charge ? t->charge + p0 : nullptr;
            const double *rb2 = rbound2 ? rbound2 + p0 : nullptr;
            int pchunk = kPrepassChunk;
            while (pchunk > 256 && np * ((ns + pchunk - 1) / pchunk) < kPrepassBlocks) pchunk /= 2;
            dim3 pgrid((unsigned)np, (unsigned)((ns + pchunk - 1) / pchunk));
            // (the pixel table's padding is zero for the first launch of a pixel pass only)
            bool gather = !prepassed && chunk == n_p && gather_allowed(ns, !pre || pre->whole, n_obs, acc_mode);
            GatherRule rule{};
            rule.n_p = np;
            if (gather) {
                rule.window = f64 ? GatherCfg<double>::W : GatherCfg<float>::W;
                rule.n_win = (n_obs + rule.window - 1) / rule.window;
                rule.bin = rule.window * ((rule.n_win + kGatherBins - 1) / kGatherBins);
                rule.x_mid = xd + 3 * (npx / 2);
                rule.n_obs = (double)n_obs;
                rule.fixed = 5.0f + ((float)rule.n_win * (float)npx) * (6e-3f + 5e-6f * (float)np);
                rule.per_most = 2.2f;
                rule.per_window = 4.1f / 1536.0f * (float)npx;
                rule.per_point = (f64 ? 20e-6f : 13e-6f) * (float)npx;
                rule.per_particle = 0.01f * (float)sh.n_tiles;
                const int at_once = f64 ? SweepCfg<double>::kDensePix : SweepCfg<float>::kDensePix;
                rule.per_pass = (float)((std::min<int64_t>(npx, kTilePix) + at_once - 1) / at_once) * (float)sh.parts_per_group;
                rule.per_mean = 1.7e-3f * rule.per_pass / (float)std::max(1, sw.n_seg);
                // a call too small for it, were all particles' points in one window or over all of the grid
                gather = rule.gathered(1.0f, (float)np, (float)np * (float)n_obs, (float)np);
            }
            if (gather) pgrid.x += (unsigned)std::min<int64_t>((np + 255) / 256, kRuleBlocks);
            if (!prepassed)
                k_prepass<<<pgrid, 256, 0, s>>>(r, b, bd, ns, pchunk, sample0, t->t_start, t->dt, gr->t0, gr->dt_obs, C, w.d,
                                                w.pflag, w.rmax2, geom, rule, w.pt);
            unsigned long long *dg = (unsigned long long *)diag;
            const dim3 grid((unsigned)blocks), grid_careful((unsigned)blocks_careful);
            if (acc_mode != kAccFloat) {
#define LW_DET_LAUNCH(G, A)                                                                                          \
    do {                                                                                                             \
        k_sweep<double, G, A><<<grid, SweepCfg<double>::kThreads, 0, s>>>(r, b, bd, charge, xd, w.d, w.pt, w.pflag, w.rmax2, rb2, (double *)Ep,   \
                                                     dg, sh, sw, dp);                                                \
        k_careful<double, G, A><<<grid_careful, kBlockThreads, 0, s>>>(r, b, bd, charge, xd, w.d, w.pt, w.pflag, w.rmax2, rb2,        \
                                                       (double *)Ep, dg, shc, dp);                                   \
    } while (0)
                if (geom == LW_GEOM_EXACT) {
                    if (acc_mode == kAccMaxAbs) LW_DET_LAUNCH(LW_GEOM_EXACT, kAccMaxAbs); else LW_DET_LAUNCH(LW_GEOM_EXACT, kAccFixed);
                } else {
                    if (acc_mode == kAccMaxAbs) LW_DET_LAUNCH(LW_GEOM_FARFIELD, kAccMaxAbs); else LW_DET_LAUNCH(LW_GEOM_FARFIELD, kAccFixed);
                }
#undef LW_DET_LAUNCH
                const lw_status st = check_launch("lw_deposit_td_det");
                if (st != LW_OK) return st;
                continue;
            }
            // the fast path (timed as the deposit kernel), then the careful path
#define LW_SWEEP_LAUNCH(T, G)                                                                                    \
    k_sweep<T, G, kAccFloat><<<grid, SweepCfg<T>::kThreads, 0, s>>>(r, b, bd, charge, xd, w.d, w.pt, w.pflag, w.rmax2, rb2, (T *)Ep, dg, \
                                                    sh, sw, DetAcc{nullptr, nullptr})
#define LW_CAREFUL_LAUNCH(T, G)                                                                                   \
    k_careful<T, G, kAccFloat><<<grid_careful, kBlockThreads, 0, s>>>(r, b, bd, charge, xd, w.d, w.pt, w.pflag, w.rmax2, rb2,         \
                                                      (T *)Ep, dg, shc, DetAcc{nullptr, nullptr})
            hipEvent_t ev = timing_begin(LW_KERNEL_DEPOSIT, s);
            if (f64) {
                if (geom == LW_GEOM_EXACT) LW_SWEEP_LAUNCH(double, LW_GEOM_EXACT); else LW_SWEEP_LAUNCH(double, LW_GEOM_FARFIELD);
            } else {
                if (geom == LW_GEOM_EXACT) LW_SWEEP_LAUNCH(float, LW_GEOM_EXACT); else LW_SWEEP_LAUNCH(float, LW_GEOM_FARFIELD);
            }
            if (gather) {
                auto go = [&](auto *k, auto *e) {
                    k<<<dim3((unsigned)std::min(rule.n_win * npx, kGatherBlocks)), 256, 0, s>>>(r, b, bd, charge, xd, w.d, w.pt, w.pflag, w.rmax2, rb2, e,
                                                                           dg, sh);
                };
                if (f64)
                    go(geom == LW_GEOM_EXACT ? k_gather<double, LW_GEOM_EXACT> : k_gather<double, LW_GEOM_FARFIELD>, (double *)Ep);
                else
                    go(geom == LW_GEOM_EXACT ? k_gather<float, LW_GEOM_EXACT> : k_gather<float, LW_GEOM_FARFIELD>, (float *)Ep);
            }
            timing_end(LW_KERNEL_DEPOSIT, ev, s);
            if (f64) {
                if (geom == LW_GEOM_EXACT) LW_CAREFUL_LAUNCH(double, LW_GEOM_EXACT); else LW_CAREFUL_LAUNCH(double, LW_GEOM_FARFIELD);
            } else {
                if (geom == LW_GEOM_EXACT) LW_CAREFUL_LAUNCH(float, LW_GEOM_EXACT); else LW_CAREFUL_LAUNCH(float, LW_GEOM_FARFIELD);
            }
#undef LW_SWEEP_LAUNCH
#undef LW_CAREFUL_LAUNCH
            const lw_status st = check_launch("lw_deposit_td");
            if (st != LW_OK) return st;
        }
    }
    return LW_OK;
}

}  // namespace lw
