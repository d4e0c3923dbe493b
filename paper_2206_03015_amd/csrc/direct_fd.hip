// Direct frequency-domain sum (Eq. inty_dft, Algorithm 1), the comparison path.
//
// A block of threads owns one pixel, a tile of frequencies and a range of chunks of samples.  Per chunk every
// thread evaluates one sample (arrival time t_a - t0 and E*kappa, the integrand of Eq. const_phase_drop) into
// LDS; then the block sums the chunk for its frequencies.
//
// FP64 (k_direct_fd): the phase w (t_a - t0) is formed in double and reduced to one revolution before
// sin/cos; for equally spaced frequencies the sums are matrix products, otherwise one sin/cos pair per term.
//
// Mixed (k_direct_fd_mixed): lane l owns K consecutive frequencies (8, or fewer for short frequency lists).
// Per 64 samples and lane the phase of the lane's first frequency at a reference arrival time is
// formed in double (reduced to one revolution); per sample one float FMA adds nu*(t_a -
// t_ref), a few revolutions at most, and the hardware sin/cos (arguments in revolutions)
// give the first phasor.  When the wavefront's frequencies are equally spaced by dw (checked
// once per wavefront), the others follow by a recurrence over frequency: with the step
// phasor e^{i dw t_a} formed once per sample at staging (phase in double, reduced, then
// float sin/cos), p_1 = p_0 e^{i dw t} and p_{j+1} = 2 cos(dw t) p_j - p_{j-1}, two FMAs per
// further frequency instead of a sin/cos pair.  Otherwise every phasor gets its own sin/cos.
// Terms are summed in float over 64 samples, those sums in double.
//
// Partial sums of a block go to a double workspace with atomics; a final kernel forms
// S = (dt^2/2pi) sum_c |F_c|^2.
#include "lw_internal.h"

#include <algorithm>

namespace lw {
namespace {

// value of lane src (wavefront-uniform src) of a double register
__device__ __forceinline__ double readlane_f64(double v, int src)
{
    const uint64_t b = (uint64_t)__double_as_longlong(v);
    const uint32_t lo = __builtin_amdgcn_readlane((uint32_t)b, src);
    const uint32_t hi = __builtin_amdgcn_readlane((uint32_t)(b >> 32), src);
    return __longlong_as_double((long long)(((uint64_t)hi << 32) | lo));
}

struct FdShape {
    int64_t n_particles, n_samples, n_pix, n_omega;
    int64_t n_wblocks;               // frequency tiles
    int64_t n_groups, parts_per_group;  // groups of chunks of samples, chunks per group
    double t_start, dt, t0, inv_cdt, cdt;
    int fmask;
    int flat;  // FP64 sums: chunks of several particles' samples
};

// how equal the spacing of a mixed wavefront's frequencies must be (relative) for the recurrence over
// frequency
constexpr double kFdEqualTol = 1e-13;

// Arrival time relative to t0 (s) and E*kappa of sample i of particle k at pixel g; zeros for
// samples past the end, unusable samples and non-finite results.
template <typename T, int GEOM>
__device__ __forceinline__ void stage_sample(const double *__restrict__ r, const double *__restrict__ beta,
                                             const double *__restrict__ beta_dot, const PixGeo &g, const double *xm,
                                             double q, int64_t k, int64_t i, const FdShape &sh, double &ta, T &ex,
                                             T &ey, T &ez)
{
    ta = 0.0;
    ex = ey = ez = (T)0;
    if (i >= sh.n_samples || !g.ok) return;
    const size_t s = (size_t)(k * sh.n_samples + i) * 3;
    if (!sample_usable(r + s, beta + s, beta_dot + s)) return;
    double kap;
    lw_field<T, GEOM>(g, xm, r[s], r[s + 1], r[s + 2], beta[s], beta[s + 1], beta[s + 2], beta_dot[s], beta_dot[s + 1],
                      beta_dot[s + 2], q, sh.fmask, ex, ey, ez, &kap);
    // arrival time relative to t0 (s), formed in units of u = cdt / c (its compensated base d and
    // the pixel terms, as in the deposit)
    const double u = sh.cdt / kC;
    const double d = arrival_base(sh.t_start, sh.dt, (double)i, sh.t0, u, r[s + 2]);
    ta = arrival_tau<GEOM, kTauSqrt>(pix_const_of(g, sh.inv_cdt), d, r[s], r[s + 1], r[s + 2], 0.0, sh.inv_cdt) * u;
    const T tk = (T)kap;
    ex *= tk;
    ey *= tk;
    ez *= tk;
    if (!(isfinite(ta) && isfinite((double)ex) && isfinite((double)ey) && isfinite((double)ez))) {
        ta = 0.0;
        ex = ey = ez = (T)0;
    }
}

// ---------------------------------------------------------------------------------------------
// FP64 sums
//
// Equally spaced frequencies (kFdBlk of them to a block, block centre w_A, offsets +-h dw with
// h = 1/2, 3/2 ... 31/2): e^{i (w_A +- h dw) t} = e^{i w_A t} (cos h dw t +- i sin h dw t), so the sums are
// one matrix product over the samples,
//   [A_c cos w_A t, A_c sin w_A t] (6 rows per block)  x  [cos h dw t, sin h dw t] (32 columns),
// whose 192 elements per block are 32 frequencies x 3 components x (re, im): six multiply-adds a term, on
// the matrix cores, and 1/32 + 1/64 sine/cosine pairs a term instead of one.  Other lists take one sine/cosine
// pair per term as they come.  The rule is decided per block of threads from the frequencies themselves.
// 20 x 2001 samples, 9 pixels, 1024 frequencies: 997 us with a sine/cosine pair per term -> 156 us (57 us of it
// the matrix product at this card's FP64 rate, the rest the phasors and the exchange through LDS).
constexpr int kFdBlk = 32;
// How far a frequency may lie from its block's line, relative to the larger of it and the block's centre: 4 x 2^-53, what
// the two or three roundings of lists made by linspace, arange or multiples of 2 pi / (N dt) come to
// (3000 lists of each with 2 to 5000 entries: at most 3.99).  The line then stands for the list, so a phase is off by
// up to as much of itself; a sine/cosine pair per term rounds it by 2.4 x 2^-53 (frequency / 2 pi, times t).
constexpr double kFdTol64 = 4.0 * 0x1p-53;
constexpr double kInv2Pi = 0.15915494309189535, kInv2PiLo = -9.839338337591243e-18;
typedef double v4d __attribute__((ext_vector_type(4)));

// centre of frequency block A
__device__ __forceinline__ double fd_centre(const double *__restrict__ omega, int64_t n, int64_t A, double dw)
{
    const int64_t j0 = A * kFdBlk;
    return j0 + kFdBlk <= n ? 0.5 * omega[j0] + 0.5 * omega[j0 + kFdBlk - 1]
                            : fma(0.5 * (kFdBlk - 1), dw, omega[j0]);
}
__device__ __forceinline__ double fd_step(const double *__restrict__ omega, int64_t n)
{
    return n > 1 ? (omega[n - 1] - omega[0]) / (double)(n - 1) : 0.0;
}
// whether the whole list is equally spaced (by the whole block of threads)
__device__ __forceinline__ bool fd_equal(const double *__restrict__ omega, int64_t n, double dw)
{
    bool ok = true;
    for (int64_t j = threadIdx.x; j < n; j += blockDim.x) {
        const double c = fd_centre(omega, n, j / kFdBlk, dw);
        const double pred = fma((double)(j % kFdBlk) - 0.5 * (kFdBlk - 1), dw, c);
        ok &= fabs(omega[j] - pred) <= kFdTol64 * fmax(fabs(omega[j]), fabs(c));
    }
    return __syncthreads_and(ok) != 0;
}
// frequency in cycles per second, as an unevaluated sum
__device__ __forceinline__ double2 fd_cycles(double w)
{
    const double hi = w * kInv2Pi;
    return make_double2(hi, fma(w, kInv2PiLo, fma(w, kInv2Pi, -hi)));
}
// cos and sin of the phase nu t (nu in cycles per second)
__device__ __forceinline__ void fd_phasor(double2 nu, double t, double &c, double &s)
{
    const double x = nu.x * t;
    const double fr = (x - floor(x)) + fma(nu.y, t, fma(nu.x, t, -x));
    sincospi(2.0 * fr, &s, &c);
}

// A block of 256 threads owns one pixel, a tile of 256 W frequencies (W = 1, 2, 4) and a range of chunks of
// kFdChunk samples.  Equal spacing: per kSub samples the two factors are formed in LDS, then wavefront
// v takes the 8 frequency blocks v mod W (48 x 32 accumulators) and every (4 / W)-th group of samples.
// Two blocks per compute unit: one forms phasors on the vector pipe while the other multiplies.
constexpr int kFdChunk = 256;
template <int W>
struct alignas(16) Fd64Lds {
    static constexpr int kSub = W == 1 ? 64 : 32;
    // pitches: a half wavefront's operand read is two rows of 16 doubles, its writes one column of 32 rows; 18 mod 32
    // doubles (16-byte writes) and 49 put nearly all of either in distinct banks (16 mod 32: reads without
    // conflicts but 16 writes on one bank, 202 us instead of 156 at the size above)
    static constexpr int kRows = 48 * W, kPitch = kRows + (kRows % 32 ? 2 : 18);
    static constexpr int kPitchR = 49;
    double ta[kFdChunk], e[3][kFdChunk];
    double2 nu[8 * W];
    union {
        struct {
            double l[kSub][kPitch], r[kSub][kPitchR];
        };
        double sum[4 / W][kRows][kFdBlk];
        double part[4][6][256];  // any frequencies: the wavefronts' sums
    };
};

template <int GEOM, int W>
__global__ __launch_bounds__(256, 2) void k_direct_fd(const double *__restrict__ r, const double *__restrict__ beta,
                                                      const double *__restrict__ beta_dot,
                                                      const double *__restrict__ charge,
                                                      const double *__restrict__ x_det,
                                                      const double *__restrict__ omega, double *__restrict__ acc,
                                                      FdShape sh)
{
    using Lds = Fd64Lds<W>;
    __shared__ Lds s;
    const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
    // equal spacing takes the blocks of blockIdx.y = 0 (which start first); with any other list a block takes 256 of the
    // tile's frequencies
    const int sub = blockIdx.y;
    const int64_t per_pix = sh.n_wblocks * sh.n_groups;
    const int64_t m = blockIdx.x / per_pix, rem = blockIdx.x - m * per_pix;
    const int64_t wb = rem / sh.n_groups, grp = rem - wb * sh.n_groups;
    const int64_t w0 = wb * 256 * W;
    if (w0 + 256 * sub >= sh.n_omega) return;
    // chunks of one particle, or (flat) of the samples of one particle after the other
    const int64_t ns = sh.n_samples, upp = sh.flat ? 1 : (ns + kFdChunk - 1) / kFdChunk, all = sh.n_particles * ns;
    const int64_t u0 = grp * sh.parts_per_group;
    const int64_t u1 = std::min(u0 + sh.parts_per_group, sh.flat ? (all + kFdChunk - 1) / kFdChunk : upp * sh.n_particles);
    const PixGeo g = pix_geo(x_det, m);
    const double *xm = x_det + 3 * m;
    const int64_t left = sh.n_omega - w0;  // frequencies of the tile
    const double dw = fd_step(omega, sh.n_omega);
    // stage chunk u: arrival times and E kappa; returns its number of samples
    auto stage = [&](int64_t u) {
        int64_t k = u / upp, i0 = (u - k * upp) * kFdChunk, i = i0 + tid, end = ns - i0;
        if (sh.flat) {
            end = all - u * kFdChunk;
            const int64_t at = u * kFdChunk + (tid < end ? tid : 0);
            k = at / ns;
            i = tid < end ? at - k * ns : ns;
        }
        double ta, ex, ey, ez;
        stage_sample<double, GEOM>(r, beta, beta_dot, g, xm, charge ? charge[k] : -kQe, k, i, sh, ta, ex, ey, ez);
        s.ta[tid] = ta;
        s.e[0][tid] = ex;
        s.e[1][tid] = ey;
        s.e[2][tid] = ez;
        return (int)std::min<int64_t>(kFdChunk, end);
    };
    if (fd_equal(omega, sh.n_omega, dw)) {
        if (sub > 0) return;
        const int na = (int)std::min<int64_t>(8 * W, (left + kFdBlk - 1) / kFdBlk);
        if (tid < 8 * W) s.nu[tid] = tid < na ? fd_cycles(fd_centre(omega, sh.n_omega, w0 / kFdBlk + tid, dw)) : make_double2(0.0, 0.0);
        const double dnu = dw * kInv2Pi;
        const int fw = wv % W, sw = wv / W;
        const bool mine = 8 * fw < na;
        v4d d[3][2];
#pragma unroll
        for (int i = 0; i < 3; ++i) d[i][0] = d[i][1] = v4d{0.0, 0.0, 0.0, 0.0};
        for (int64_t u = u0; u < u1; ++u) {
            const int n = stage(u);
            __syncthreads();
            for (int q0 = 0; q0 < n; q0 += Lds::kSub) {
                // the factors of samples q0 .. q0 + kSub (past the chunk's end their field is zero)
                for (int it = tid; it < Lds::kSub * 2 * W; it += 256) {
                    const int q = it % Lds::kSub, a0 = it / Lds::kSub * 4;
                    const double t = s.ta[q0 + q], e0 = s.e[0][q0 + q], e1 = s.e[1][q0 + q], e2 = s.e[2][q0 + q];
#pragma unroll
                    for (int a = a0; a < a0 + 4; ++a) {
                        double c = 0.0, sn = 0.0;
                        if (a < na) fd_phasor(s.nu[a], t, c, sn);
                        double2 *o = (double2 *)&s.l[q][6 * a];
                        o[0] = make_double2(e0 * c, e0 * sn);
                        o[1] = make_double2(e1 * c, e1 * sn);
                        o[2] = make_double2(e2 * c, e2 * sn);
                    }
                }
                for (int it = tid; it < Lds::kSub * 16; it += 256) {
                    const int q = it % Lds::kSub, h = it / Lds::kSub;
                    const double x = ((double)h + 0.5) * dnu * s.ta[q0 + q];
                    double c, sn;
                    sincospi(2.0 * (x - floor(x)), &sn, &c);
                    s.r[q][h] = c;
                    s.r[q][16 + h] = sn;
                }
                __syncthreads();
                if (mine) {
#pragma unroll
                    for (int q = 0; q < Lds::kSub / (4 / W); q += 4) {
                        const int k = sw * (Lds::kSub / (4 / W)) + q + (lane >> 4);
                        const double b0 = s.r[k][lane & 15], b1 = s.r[k][16 + (lane & 15)];
#pragma unroll
                        for (int i = 0; i < 3; ++i) {
                            const double a = s.l[k][48 * fw + 16 * i + (lane & 15)];
                            d[i][0] = __builtin_amdgcn_mfma_f64_16x16x4f64(a, b0, d[i][0], 0, 0, 0);
                            d[i][1] = __builtin_amdgcn_mfma_f64_16x16x4f64(a, b1, d[i][1], 0, 0, 0);
                        }
                    }
                }
                __syncthreads();
            }
        }
        // rows (block, component, re / im) x (cos h, sin h), summed over the wavefronts that share them in their order
        if (mine) {
#pragma unroll
            for (int i = 0; i < 3; ++i)
#pragma unroll
                for (int v = 0; v < 4; ++v) {
                    double *o = s.sum[sw][48 * fw + 16 * i + (lane >> 4) + 4 * v] + (lane & 15);
                    o[0] = d[i][0][v];
                    o[16] = d[i][1][v];
                }
        }
        __syncthreads();
        for (int it = tid; it < (int)std::min<int64_t>(left, 256 * W) * 3; it += 256) {
            const int j = it / 3, c = it - 3 * j, b = j % kFdBlk;
            const int row = j / kFdBlk * 6 + 2 * c;
            auto sum = [&](int r, int col) {
                double v = s.sum[0][r][col];
#pragma unroll
                for (int w = 1; w < 4 / W; ++w) v += s.sum[w][r][col];
                return v;
            };
            const int h = b >= 16 ? b - 16 : 15 - b;
            const double sg = b >= 16 ? 1.0 : -1.0;
            double *o = acc + ((size_t)m * sh.n_omega + w0 + j) * 6 + 2 * c;
            atomic_add(o, fma(-sg, sum(row + 1, 16 + h), sum(row, h)));
            atomic_add(o + 1, fma(sg, sum(row, 16 + h), sum(row + 1, h)));
        }
        return;
    }
    // any frequencies, 256 of them: wavefront v takes the v-th quarter of each chunk's samples for all, lanes over
    // frequencies, so that a list of any length keeps the four wavefronts busy.  20 x 2001 samples, 25 pixels, 100
    // frequencies: 547 us with a wavefront per 64 frequencies, 295 now; 1030 frequencies: 4257 us with a tile of
    // W x 256 to a block, 2760 now.
    constexpr int kF = 4;
    const int64_t ws = w0 + 256 * sub;
    double nu[kF], a[kF][6];
#pragma unroll
    for (int f = 0; f < kF; ++f) {
        const int64_t w = ws + 64 * f + lane;
        nu[f] = w < sh.n_omega ? omega[w] / (2.0 * kPi) : 0.0;
#pragma unroll
        for (int c = 0; c < 6; ++c) a[f][c] = 0.0;
    }
    for (int64_t u = u0; u < u1; ++u) {
        const int n = stage(u), share = (n + 3) / 4, qa = share * wv, qb = std::min(qa + share, n);
        __syncthreads();
#pragma unroll
        for (int f = 0; f < kF; ++f) {
            if (ws + 64 * f >= sh.n_omega) break;
            double b0 = 0, b1 = 0, b2 = 0, b3 = 0, b4 = 0, b5 = 0;
            for (int q = qa; q < qb; ++q) {
                const double x = nu[f] * s.ta[q];
                double sn, c;
                sincospi(2.0 * (x - floor(x)), &sn, &c);
                const double e0 = s.e[0][q], e1 = s.e[1][q], e2 = s.e[2][q];
                b0 += e0 * c;
                b1 += e0 * sn;
                b2 += e1 * c;
                b3 += e1 * sn;
                b4 += e2 * c;
                b5 += e2 * sn;
            }
            a[f][0] += b0;
            a[f][1] += b1;
            a[f][2] += b2;
            a[f][3] += b3;
            a[f][4] += b4;
            a[f][5] += b5;
        }
        __syncthreads();
    }
    // the wavefronts' sums in their order
#pragma unroll
    for (int f = 0; f < kF; ++f)
#pragma unroll
        for (int c = 0; c < 6; ++c) s.part[wv][c][64 * f + lane] = a[f][c];
    __syncthreads();
    if (ws + tid < sh.n_omega) {
        double *o = acc + ((size_t)m * sh.n_omega + ws + tid) * 6;
#pragma unroll
        for (int c = 0; c < 6; ++c)
            atomic_add(o + c, ((s.part[0][c][tid] + s.part[1][c][tid]) + s.part[2][c][tid]) + s.part[3][c][tid]);
    }
}

// The mixed sums' place of frequency j of lane l of a wavefront with R of its 64 K frequencies, in a plane per
// component: the wavefront's atomics fall on neighbouring elements (lanes own consecutive frequencies; with a
// frequency's six sums side by side each lane's atomics fell on lines of their own, and 400 groups' adding took
// 1.3 ms of a call)
__host__ __device__ __forceinline__ int64_t fd_place(int64_t R, int K, int j, int64_t l)
{
    return j * (R / K) + (j < R % K ? j : R % K) + l;
}

// ---------------------------------------------------------------------------------------------
// Mixed sums.  A block of W wavefronts owns one pixel, W x 64 K frequencies and a range of chunks of 64 W
// samples.  The samples are staged once for the W wavefronts (the field and the arrival time are ~150 FP64
// instructions a sample); the sums run on the matrix cores: a 4x4x1 product holds 16 blocks of 4 columns, so
// that with the sample's (E_x, E_y, E_z, 0) in every block's rows and the lane's phasor in its column it is
// the three multiply-adds of 64 lanes, each rounded as fmaf rounds, in two passes instead of three.  The vector
// pipe is left with the phasors.  The two kinds of instruction don't overlap (measured: 10.5 cycles a 4x4x1 product,
// 4.4 a vector FMA, ~8 for each change from one to the other), so they come in batches of kFdBatch samples.
// 25 x 20001 samples, 64 pixels, 4096 frequencies: 34.0 ms (six vector FMAs a term, every wavefront staging for
// itself) -> 25.6 ms; a batch of one sample 26.1, four 25.4, instructions mixed by the compiler 31.9.
typedef float v4f __attribute__((ext_vector_type(4)));
constexpr int kFdBatch = 2;

template <int GEOM, int K, int W>
__global__ __launch_bounds__(64 * W, 2) void k_direct_fd_mixed(const double *__restrict__ r,
                                                               const double *__restrict__ beta,
                                                               const double *__restrict__ beta_dot,
                                                               const double *__restrict__ charge,
                                                               const double *__restrict__ x_det,
                                                               const double *__restrict__ omega,
                                                               double *__restrict__ acc, FdShape sh)
{
    constexpr int NS = 64 * W;
    __shared__ float4 s_t[W][NS];  // per wavefront's frequencies: t_a - t_ref (s), e^{i dw t_a}
    __shared__ __align__(16) float s_e[NS][4];  // E kappa
    __shared__ double s_tref[W], s_dnu[W];
    __shared__ int s_eq[W];
    const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
    const int64_t per_pix = sh.n_wblocks * sh.n_groups;
    const int64_t m = blockIdx.x / per_pix, rem = blockIdx.x - m * per_pix;
    const int64_t wb = rem / sh.n_groups, grp = rem - wb * sh.n_groups;
    const int64_t wfirst = (wb * W + wv) * 64 * K, wl = wfirst + (int64_t)lane * K;
    const int64_t ns = sh.n_samples, upp = (ns + NS - 1) / NS;  // chunks per particle
    const int64_t u0 = grp * sh.parts_per_group, u1 = std::min(u0 + sh.parts_per_group, upp * sh.n_particles);
    const bool mine = wfirst < sh.n_omega;
    // frequencies in cycles per second; the wavefront's spacing from its first two
    double nu[K];
#pragma unroll
    for (int j = 0; j < K; ++j) nu[j] = wl + j < sh.n_omega ? omega[wl + j] / (2.0 * kPi) : 0.0;
    const double nu_a = mine ? omega[wfirst] / (2.0 * kPi) : 0.0;
    const double dnu = wfirst + 1 < sh.n_omega ? omega[wfirst + 1] / (2.0 * kPi) - nu_a : 0.0;
    bool lane_eq = true;
#pragma unroll
    for (int j = 0; j < K; ++j) {
        const double pred = nu[0] + (double)j * dnu;
        if (wl + j < sh.n_omega) lane_eq &= fabs(nu[j] - pred) <= kFdEqualTol * fabs(nu[j]);
    }
    const bool equal = __ballot(!lane_eq) == 0;  // wavefront-uniform
    if (lane == 0) {
        s_dnu[wv] = dnu;
        s_eq[wv] = equal && mine;
    }
    __syncthreads();
    const PixGeo g = pix_geo(x_det, m);
    const double *xm = x_det + 3 * m;
    double a[K][6];
#pragma unroll
    for (int j = 0; j < K; ++j)
#pragma unroll
        for (int c = 0; c < 6; ++c) a[j][c] = 0.0;
    for (int64_t u = u0; u < u1; ++u) {
        const int64_t k = u / upp, i0 = (u - k * upp) * NS;
        {
            double ta = 0.0;
            float ex = 0, ey = 0, ez = 0;
            stage_sample<float, GEOM>(r, beta, beta_dot, g, xm, charge ? charge[k] : -kQe, k, i0 + tid, sh, ta, ex, ey, ez);
            const bool live = ex != 0.0f || ey != 0.0f || ez != 0.0f;
            // reference arrival time of 64 samples: the first with a contribution
            const uint64_t lm = __ballot(live);
            const double tref = lm ? readlane_f64(ta, (int)__builtin_ctzll(lm)) : 0.0;
            if (lane == 0) s_tref[wv] = tref;
            const float dt = live ? (float)(ta - tref) : 0.0f;
#pragma unroll
            for (int v = 0; v < W; ++v) {
                float2 st = make_float2(1.0f, 0.0f);
                if (s_eq[v] && live) {
                    const double x = s_dnu[v] * ta;
                    const float fr = (float)(x - floor(x));  // revolutions in [0, 1)
                    st = make_float2(__builtin_amdgcn_cosf(fr), __builtin_amdgcn_sinf(fr));
                }
                s_t[v][tid] = make_float4(dt, st.x, st.y, 0.0f);
            }
            *(float4 *)s_e[tid] = make_float4(ex, ey, ez, 0.0f);
        }
        __syncthreads();
        for (int ch = 0; ch < W && mine; ++ch) {
            // staged samples past the end have a zero field
            const int cnt = ((int)std::min<int64_t>(64, ns - i0 - 64 * ch) + 3) & ~3;
            if (cnt <= 0) break;
            const double tref = s_tref[ch];
            const float4 *st4 = s_t[wv] + 64 * ch;
            const float *ep = &s_e[64 * ch][lane & 3];
            v4f b[K][2];
#pragma unroll
            for (int j = 0; j < K; ++j) b[j][0] = b[j][1] = v4f{0.0f, 0.0f, 0.0f, 0.0f};
            if (equal) {
                const double x = nu[0] * tref;
                const float base = (float)(x - floor(x));  // revolutions in [0, 1)
                const float nuf = (float)nu[0];
                // phasors p_j = e^{i(w_0 + j dw)t}: p_1 = p_0 e^{i dw t}, then the two-term recurrence
                // p_{j+1} = 2 cos(dw t) p_j - p_{j-1} (two FMAs per frequency)
                auto phasors = [&](const float4 q, float *pc, float *ps) {
                    const float ph = fmaf(nuf, q.x, base);
                    pc[0] = __builtin_amdgcn_cosf(ph);
                    ps[0] = __builtin_amdgcn_sinf(ph);
                    const float tc = q.y + q.y;
                    if constexpr (K > 1) {
                        pc[1] = fmaf(pc[0], q.y, -ps[0] * q.z);
                        ps[1] = fmaf(pc[0], q.z, ps[0] * q.y);
                    }
#pragma unroll
                    for (int j = 2; j < K; ++j) {
                        pc[j] = fmaf(tc, pc[j - 1], -pc[j - 2]);
                        ps[j] = fmaf(tc, ps[j - 1], -ps[j - 2]);
                    }
                };
                // matrix and vector instructions in turn cost ~8 cycles a change: batches of kFdBatch samples each
                for (int s = 0; s < cnt; s += 4) {
#pragma unroll
                    for (int v0 = 0; v0 < 4; v0 += kFdBatch) {
                        float pc[kFdBatch][K], ps[kFdBatch][K], e[kFdBatch];
#pragma unroll
                        for (int v = 0; v < kFdBatch; ++v) {
                            e[v] = ep[4 * (s + v0 + v)];
                            phasors(st4[s + v0 + v], pc[v], ps[v]);
                        }
                        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                        for (int v = 0; v < kFdBatch; ++v)
#pragma unroll
                            for (int j = 0; j < K; ++j) {
                                b[j][0] = __builtin_amdgcn_mfma_f32_4x4x1f32(e[v], pc[v][j], b[j][0], 0, 0, 0);
                                b[j][1] = __builtin_amdgcn_mfma_f32_4x4x1f32(e[v], ps[v][j], b[j][1], 0, 0, 0);
                            }
                        __builtin_amdgcn_sched_barrier(0);
                    }
                }
            } else {
                float base[K], nuf[K];
#pragma unroll
                for (int j = 0; j < K; ++j) {
                    const double x = nu[j] * tref;
                    base[j] = (float)(x - floor(x));
                    nuf[j] = (float)nu[j];
                }
                for (int s = 0; s < cnt; ++s) {
                    const float dtf = st4[s].x, e = ep[4 * s];
#pragma unroll
                    for (int j = 0; j < K; ++j) {
                        const float ph = fmaf(nuf[j], dtf, base[j]);
                        b[j][0] = __builtin_amdgcn_mfma_f32_4x4x1f32(e, __builtin_amdgcn_cosf(ph), b[j][0], 0, 0, 0);
                        b[j][1] = __builtin_amdgcn_mfma_f32_4x4x1f32(e, __builtin_amdgcn_sinf(ph), b[j][1], 0, 0, 0);
                    }
                }
            }
#pragma unroll
            for (int j = 0; j < K; ++j)
#pragma unroll
                for (int c = 0; c < 3; ++c) {
                    a[j][2 * c] += (double)b[j][0][c];
                    a[j][2 * c + 1] += (double)b[j][1][c];
                }
        }
        __syncthreads();
    }
#pragma unroll
    for (int j = 0; j < K; ++j) {
        if (wl + j >= sh.n_omega) continue;
        double *o = acc + (size_t)m * 6 * sh.n_omega + wfirst +
                    fd_place(std::min<int64_t>(64 * K, sh.n_omega - wfirst), K, j, lane);
#pragma unroll
        for (int c = 0; c < 6; ++c) atomic_add(o + c * sh.n_omega, a[j][c]);
    }
}

__global__ void k_fd_zero(double *__restrict__ p, int64_t n)
{
    for (int64_t j = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; j < n; j += (int64_t)gridDim.x * blockDim.x)
        p[j] = 0.0;
}

// K = 0: acc [n_pix][n_omega][6]; else [n_pix][6][n_omega], placed by fd_place
__global__ void k_fd_finish(const double *__restrict__ acc, double *__restrict__ S, int64_t n, int64_t n_omega, int K, double f)
{
    for (int64_t j = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; j < n; j += (int64_t)gridDim.x * blockDim.x) {
        double a[6];
        if (K == 0) {
            for (int c = 0; c < 6; ++c) a[c] = acc[6 * j + c];
        } else {
            const int64_t m = j / n_omega, w = j - m * n_omega, w0 = w / (64 * K) * (64 * K);
            const int64_t R = n_omega - w0 < 64 * K ? n_omega - w0 : 64 * K;
            const double *p = acc + m * 6 * n_omega + w0 + fd_place(R, K, (int)((w - w0) % K), (w - w0) / K);
            for (int c = 0; c < 6; ++c) a[c] = p[c * n_omega];
        }
        S[j] = f * (a[0] * a[0] + a[1] * a[1] + a[2] * a[2] + a[3] * a[3] + a[4] * a[4] + a[5] * a[5]);
    }
}

// Adjoint of the direct sum for FP64 inputs: with R_c, I_c the real and imaginary parts of the
// forward sum F_c(w) (recomputed into acc) and A = E kappa, t = t_i + shift - t0 per (sample, pixel),
//   dJ/dA_c = 2f sum_w dS(w) (R_c cos wt + I_c sin wt),
//   dJ/dt   = 2f sum_w dS(w) w sum_c A_c (I_c cos wt - R_c sin wt),       f = dt^2 / 2pi,
// then dJ/dE = kappa dJ/dA, dJ/dkappa = E.dJ/dA through lw_field_vjp, and dt/dr = -n/c.
//
// A block owns 64 consecutive samples of one particle and loops over the pixels, four at a time: wavefront
// v takes the field, arrival time and Jacobian of pixel 4 n + v (lanes over samples), all four the sums of
// each pixel.  With C = dS F (and w dS F for dJ/dt) the sums are the real (imaginary) parts of
// sum_w C(w) e^{-iwt}; for equally spaced frequencies (blocks and offsets as in the forward sums)
//   sum_w C e^{-iwt} = sum_A e^{-i w_A t} sum_h [cos h dw t (C+ + C-) - i sin h dw t (C+ - C-)]_A,
// the inner sum a matrix product over the 32 cosines and sines of a sample, 12 columns (6 quantities, re and
// im) per block of 32 frequencies, four blocks (48 columns) at a time: 12 multiply-adds a term on the matrix
// cores and 1/32 sine/cosine pair.  Where the workspace has room for their partial gradients, the pixels are shared out
// over blocks until there are kFdBwdBlocks of them (a block's chain of pixels and frequency blocks is its time, and two
// fit a compute unit), and k_fd_add sums the partial gradients in their order; otherwise a block takes all pixels.  Within a
// block the parts of a sum go through LDS and are added in a fixed order too: for given sums F_c(w) a call's bits
// are the same on every run.
// 20 x 2001 samples, 9 pixels, 1024 frequencies: 2071 us with a sine/cosine pair per term -> 350 us (112 us of it
// the matrix product).
constexpr int64_t kFdBwdBlocks = 2048;
constexpr int kFdNu = 128;  // frequency blocks whose centres are kept
struct alignas(16) FdBwdLds {
    double2 nua[kFdNu];
    double nu[4][64], ta[4][64];  // any-frequency path: staged frequencies; arrival times of four pixels
    double g[4][6][64];           // G_c, K_c of four pixels
    union {
        struct {
            double w[32][50];    // coefficients of the four blocks (pitch as in Fd64Lds)
            double p[4][64][2];  // cos, sin of w_A t
        };
        double row[4][64][8];   // any-frequency path: dS, w dS, R_x, I_x, R_y, I_y, R_z, I_z
        double part[4][6][64];  // and the wavefronts' sums
        double col[48][65];     // equal spacing: a pixel's 48 columns of sums (odd pitch: writes of 16 columns at a time)
        double red[4][9][64];   // the wavefronts' gradients
    };
};

template <int GEOM>
__global__ __launch_bounds__(256, 2) void k_direct_fd_bwd(const double *__restrict__ r, const double *__restrict__ beta,
                                                          const double *__restrict__ beta_dot,
                                                          const double *__restrict__ charge,
                                                          const double *__restrict__ x_det,
                                                          const double *__restrict__ omega,
                                                          const double *__restrict__ acc, const double *__restrict__ dS,
                                                          double *__restrict__ d_r, double *__restrict__ d_beta,
                                                          double *__restrict__ d_beta_dot, FdShape sh, double two_f,
                                                          int64_t share_stride)
{
    __shared__ FdBwdLds s;
    const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
    const int64_t n_chunks = (sh.n_samples + 63) / 64;
    const int64_t k = blockIdx.x / n_chunks;
    const int64_t i = (blockIdx.x - k * n_chunks) * 64 + lane;
    const bool in = i < sh.n_samples;
    const size_t so = (size_t)(k * sh.n_samples + (in ? i : 0)) * 3;
    double rs[3], bs[3], as[3];
    for (int c = 0; c < 3; ++c) {
        rs[c] = r[so + c];
        bs[c] = beta[so + c];
        as[c] = beta_dot[so + c];
    }
    const bool usable = in && sample_usable(rs, bs, as);
    const double q = charge ? charge[k] : -kQe;
    const double u = sh.cdt / kC;
    const double d = arrival_base(sh.t_start, sh.dt, (double)i, sh.t0, u, rs[2]);
    double gr[3] = {0, 0, 0}, gb[3] = {0, 0, 0}, ga[3] = {0, 0, 0};
    const int64_t n_w = sh.n_omega;
    const double dw = fd_step(omega, n_w), dnu = dw * kInv2Pi;
    const bool equal = fd_equal(omega, n_w, dw);
    const int64_t na = (n_w + kFdBlk - 1) / kFdBlk;
    for (int64_t A = tid; A < std::min<int64_t>(na, kFdNu); A += 256) s.nua[A] = fd_cycles(fd_centre(omega, n_w, A, dw));
    // this block's share of the pixels
    const int64_t mb = std::min<int64_t>((int64_t)blockIdx.y * sh.parts_per_group, sh.n_pix);
    const int64_t me = std::min<int64_t>(mb + sh.parts_per_group, sh.n_pix);
    for (int64_t m0 = mb; m0 < me; m0 += 4) {
        const int64_t m = m0 + wv;
        PixGeo g = pix_geo(x_det, m < me ? m : mb);
        const double *xm = x_det + 3 * (m < me ? m : mb);
        bool ok = usable && g.ok && m < me;
        double ta = 0.0, kap = 0.0, E[3] = {0, 0, 0}, A[3] = {0, 0, 0};
        if (ok) {
            lw_field<double, GEOM>(g, xm, rs[0], rs[1], rs[2], bs[0], bs[1], bs[2], as[0], as[1], as[2], q, sh.fmask,
                                   E[0], E[1], E[2], &kap);
            ta = arrival_tau<GEOM, kTauSqrt>(pix_const_of(g, sh.inv_cdt), d, rs[0], rs[1], rs[2], 0.0, sh.inv_cdt) * u;
            for (int c = 0; c < 3; ++c) A[c] = E[c] * kap;
            ok = isfinite(ta) && isfinite(A[0]) && isfinite(A[1]) && isfinite(A[2]);
        }
        s.ta[wv][lane] = ok ? ta : 0.0;
        __syncthreads();
        const int np = (int)std::min<int64_t>(4, me - m0);
        for (int p = 0; p < np; ++p) {
            const double *fs = acc + (size_t)(m0 + p) * n_w * 6, *ds = dS + (size_t)(m0 + p) * n_w;
            if (equal) {
                // this lane's operand: cos / sin of h dw t of sample 16 wv + lane % 16, h - 1/2 = lane / 16 + 4 j
                const double tl = s.ta[p][16 * wv + (lane & 15)];
                double av[8];
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    const double x = ((double)(4 * j + (lane >> 4)) + 0.5) * dnu * tl;
                    sincospi(2.0 * (x - floor(x)), &av[4 + j], &av[j]);
                }
                double sum[3][4];
#pragma unroll
                for (int t = 0; t < 3; ++t)
#pragma unroll
                    for (int v = 0; v < 4; ++v) sum[t][v] = 0.0;
                // thread -> block a, offset h, component c of four blocks (192 of them); the next four's values are on
                // their way while these multiply
                const int c3 = tid % 3, h16 = tid / 3 % 16, a4 = tid / 48;
                double fp[2], fm[2], dp, dm, wp, wm;
                auto fetch = [&](int64_t w0) {
                    const int64_t jp = w0 + kFdBlk * a4 + 16 + h16, jm = w0 + kFdBlk * a4 + 15 - h16;
                    fp[0] = fp[1] = fm[0] = fm[1] = dp = dm = wp = wm = 0.0;
                    if (tid >= 192) return;
                    if (jp < n_w) {
                        fp[0] = fs[jp * 6 + 2 * c3];
                        fp[1] = fs[jp * 6 + 2 * c3 + 1];
                        dp = ds[jp];
                        wp = omega[jp];
                    }
                    if (jm < n_w) {
                        fm[0] = fs[jm * 6 + 2 * c3];
                        fm[1] = fs[jm * 6 + 2 * c3 + 1];
                        dm = ds[jm];
                        wm = omega[jm];
                    }
                };
                fetch(0);
                for (int64_t w0 = 0; w0 < n_w; w0 += 4 * kFdBlk) {
                    if (tid < 192) {
                        double cp[2] = {dp * fp[0], dp * fp[1]}, cm[2] = {dm * fm[0], dm * fm[1]};
#pragma unroll
                        for (int z = 0; z < 2; ++z) {  // C, then w C
                            double *o = &s.w[h16][12 * a4 + 6 * z + 2 * c3], *o2 = &s.w[16 + h16][12 * a4 + 6 * z + 2 * c3];
                            o[0] = cp[0] + cm[0];
                            o[1] = cp[1] + cm[1];
                            o2[0] = cp[1] - cm[1];
                            o2[1] = cm[0] - cp[0];
#pragma unroll
                            for (int e = 0; e < 2; ++e) {
                                cp[e] *= wp;
                                cm[e] *= wm;
                            }
                        }
                    }
                    {  // block wv's phase at sample `lane`
                        double cs = 0.0, sn = 0.0;
                        const int64_t A = w0 / kFdBlk + wv;
                        if (A < na)
                            fd_phasor(A < kFdNu ? s.nua[A] : fd_cycles(fd_centre(omega, n_w, A, dw)), s.ta[p][lane], cs, sn);
                        *(double2 *)s.p[wv][lane] = make_double2(cs, sn);
                    }
                    __syncthreads();
                    fetch(w0 + 4 * kFdBlk);
                    v4d t3[3];
#pragma unroll
                    for (int t = 0; t < 3; ++t) t3[t] = v4d{0.0, 0.0, 0.0, 0.0};
#pragma unroll
                    for (int j = 0; j < 8; ++j)
#pragma unroll
                        for (int t = 0; t < 3; ++t)
                            t3[t] = __builtin_amdgcn_mfma_f64_16x16x4f64(av[j], s.w[4 * j + (lane >> 4)][16 * t + (lane & 15)],
                                                                         t3[t], 0, 0, 0);
                    // column -> block a, quantity z (< 3: real part wanted, else imaginary), re / im: the part of
                    // (cos - i sin) (re + i im) it feeds (the sign of K's -sin re is applied at the end)
#pragma unroll
                    for (int t = 0; t < 3; ++t) {
                        const int col = 16 * t + (lane & 15), a = col / 12, z = col % 12 / 2, ri = col & 1;
                        const double *pp = &s.p[a][16 * wv + (lane >> 4)][z < 3 ? ri : 1 - ri];
#pragma unroll
                        for (int v = 0; v < 4; ++v) sum[t][v] = fma(t3[t][v], pp[8 * v], sum[t][v]);
                    }
                    __syncthreads();
                }
#pragma unroll
                for (int t = 0; t < 3; ++t) {
#pragma unroll
                    for (int v = 0; v < 4; ++v) s.col[16 * t + (lane & 15)][16 * wv + (lane >> 4) + 4 * v] = sum[t][v];
                }
                __syncthreads();
                for (int it = tid; it < 6 * 64; it += 256) {
                    const int z = it >> 6, q = it & 63;
                    double v = 0.0;
#pragma unroll
                    for (int a = 0; a < 4; ++a) {
                        const double re = s.col[12 * a + 2 * z][q], im = s.col[12 * a + 2 * z + 1][q];
                        v += z >= 3 ? im - re : re + im;
                    }
                    s.g[p][z][q] = v;
                }
                __syncthreads();
            } else {
                // any frequencies: lanes over samples, wavefront v takes every fourth 64 frequencies
                const double tl = s.ta[p][lane];
                double G[3] = {0, 0, 0}, K[3] = {0, 0, 0};
                for (int64_t w0 = 64 * wv; w0 < n_w; w0 += 256) {
                    const int64_t w = w0 + lane;
                    double *row = s.row[wv][lane];
                    const double dv = w < n_w ? ds[w] : 0.0, ov = w < n_w ? omega[w] : 0.0;
                    s.nu[wv][lane] = ov / (2.0 * kPi);
                    row[0] = dv;
                    row[1] = dv * ov;
                    for (int c = 0; c < 6; ++c) row[2 + c] = w < n_w ? fs[w * 6 + c] : 0.0;
                    __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
                    __builtin_amdgcn_wave_barrier();
                    const int cnt = (int)std::min<int64_t>(64, n_w - w0);
                    for (int j = 0; j < cnt; ++j) {
                        const double x = s.nu[wv][j] * tl;
                        double sn, cs;
                        sincospi(2.0 * (x - floor(x)), &sn, &cs);
                        const double *rj = s.row[wv][j];
                        for (int c = 0; c < 3; ++c) {
                            const double Rc = rj[2 + 2 * c], Ic = rj[3 + 2 * c];
                            G[c] = fma(rj[0], fma(Rc, cs, Ic * sn), G[c]);
                            K[c] = fma(rj[1], fma(Ic, cs, -Rc * sn), K[c]);
                        }
                    }
                    __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
                    __builtin_amdgcn_wave_barrier();
                }
                __syncthreads();  // the rows are read
                for (int c = 0; c < 3; ++c) {
                    s.part[wv][c][lane] = G[c];
                    s.part[wv][3 + c][lane] = K[c];
                }
                __syncthreads();
                for (int it = tid; it < 6 * 64; it += 256) {
                    const int z = it >> 6, q = it & 63;
                    s.g[p][z][q] = ((s.part[0][z][q] + s.part[1][z][q]) + s.part[2][z][q]) + s.part[3][z][q];
                }
                __syncthreads();
            }
        }
        __syncthreads();
        if (ok) {
            double G[3], gE[3], gk = 0.0, H = 0.0;
            for (int c = 0; c < 3; ++c) {
                G[c] = two_f * s.g[wv][c][lane];
                gE[c] = kap * G[c];
                gk = fma(E[c], G[c], gk);
                H = fma(A[c], two_f * s.g[wv][3 + c][lane], H);
            }
            lw_field_vjp<GEOM>(g, xm, rs, bs, as, q, sh.fmask, gE, gr, gb, ga, gk);
            // t = t_i + (|x - r| - |x|)/c - t0 (exact) or t_i - n.r/c - t0 (far field): dt/dr = -n/c
            double n[3] = {g.nx, g.ny, g.nz};
            if (GEOM == LW_GEOM_EXACT) {
                const double d0 = xm[0] - rs[0], d1 = xm[1] - rs[1], d2 = xm[2] - rs[2];
                const double R = sqrt(d0 * d0 + d1 * d1 + d2 * d2);
                n[0] = d0 / R;
                n[1] = d1 / R;
                n[2] = d2 / R;
            }
            for (int c = 0; c < 3; ++c) gr[c] -= H * n[c] / kC;
        }
    }
    // the wavefronts' gradients, summed in their order
    __syncthreads();
    for (int c = 0; c < 3; ++c) {
        s.red[wv][c][lane] = gr[c];
        s.red[wv][3 + c][lane] = gb[c];
        s.red[wv][6 + c][lane] = ga[c];
    }
    __syncthreads();
    if (in && wv < 3) {
        double *out = wv == 0 ? d_r : wv == 1 ? d_beta : d_beta_dot;
        for (int c = 0; c < 3; ++c) {
            double v = s.red[0][3 * wv + c][lane];
            for (int w = 1; w < 4; ++w) v += s.red[w][3 * wv + c][lane];
            if (share_stride)  // a share of the pixels: partial gradients
                out[(size_t)blockIdx.y * share_stride + so + c] = v;
            else
                out[so + c] += v;
        }
    }
}

// d_r, d_beta, d_beta_dot (n elements each) += their partial gradients [n_shares][3][n], in order
__global__ void k_fd_add(const double *__restrict__ part, int n_shares, int64_t n, double *__restrict__ d_r,
                         double *__restrict__ d_beta, double *__restrict__ d_beta_dot)
{
    for (int64_t j = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; j < n; j += (int64_t)gridDim.x * blockDim.x) {
        double v[3] = {0.0, 0.0, 0.0};
        for (int y = 0; y < n_shares; ++y)
            for (int a = 0; a < 3; ++a) v[a] += part[((size_t)y * 3 + a) * n + j];
        d_r[j] += v[0];
        d_beta[j] += v[1];
        d_beta_dot[j] += v[2];
    }
}

}  // namespace

size_t direct_fd_ws_bytes(int64_t n_pix, int64_t n_omega)
{
    return (size_t)std::max<int64_t>(n_pix * n_omega, 1) * 6 * sizeof(double);
}

namespace {

FdShape fd_shape(const lw_traj_t *t, const lw_grid_t *gr, int64_t n_omega, int fmask)
{
    FdShape sh;
    sh.n_particles = t->n_particles;
    sh.n_samples = t->n_samples;
    sh.n_pix = gr->n_pix;
    sh.n_omega = n_omega;
    sh.n_wblocks = sh.n_groups = sh.parts_per_group = 0;
    sh.t_start = t->t_start;
    sh.dt = t->dt;
    sh.t0 = gr->t0;
    // any positive grid step gives the same arrival times; use dt (the grid of this call is irrelevant)
    sh.cdt = kC * t->dt;
    sh.inv_cdt = 1.0 / sh.cdt;
    sh.fmask = fmask;
    sh.flat = 0;
    return sh;
}

// most (pixel, frequency tile) pairs, resp. chunks of 64 samples, of a launch: a grid's threads count in 32 bits (at
// most 2^24 blocks of 256); more of them take several launches, a range of pixels resp. particles each
constexpr int64_t kFdLaunch = int64_t(1) << 22;

// chunks of samples (`units` of them) per group, so that about `rounds` times `resident` blocks run; returns the blocks
int64_t fd_groups(FdShape &sh, int64_t units, int64_t resident, int64_t rounds)
{
    const int64_t base = sh.n_pix * sh.n_wblocks;
    const int64_t groups = std::max<int64_t>(1, std::min(units, resident * rounds / base));
    sh.parts_per_group = (units + groups - 1) / groups;
    sh.n_groups = (units + sh.parts_per_group - 1) / sh.parts_per_group;
    return base * sh.n_groups;
}

// launch(n_pix, x_det, acc) for ranges of pixels (a pixel's sums: 6 n_omega doubles in either layout of acc)
template <typename F>
void fd_launches(const FdShape &sh, const double *x_det, double *acc, F launch)
{
    const int64_t most = std::max<int64_t>(1, kFdLaunch / sh.n_wblocks);
    for (int64_t m0 = 0; m0 < sh.n_pix; m0 += most)
        launch(std::min(most, sh.n_pix - m0), x_det + 3 * m0, acc + m0 * 6 * sh.n_omega);
}

// FP64 sums F_c(w), added into acc
void launch_sums64(const lw_traj_t *t, const lw_grid_t *gr, const double *omega, FdShape sh, int geom, double *acc,
                   hipStream_t s)
{
    // frequencies per block: one tile of 256, 512 or 1024
    const int W = sh.n_omega > 512 ? 4 : sh.n_omega > 256 ? 2 : 1;
    sh.n_wblocks = (sh.n_omega + 256 * W - 1) / (256 * W);
    // two blocks per compute unit; more rounds of them, of some eight chunks each (every block adds its sums
    // with 6 atomics per frequency)
    // Chunks hold the samples of several particles where one fills less than half of them and there are blocks enough:
    // 50 x 61 samples, 16 pixels, 600 uneven frequencies 145 -> 102 us; 3 x 101 samples, 2 pixels 24 -> 30 us
    sh.flat = 2 * sh.n_samples <= kFdChunk && sh.n_pix * sh.n_wblocks * sh.n_particles >= 512;
    const int64_t units = sh.flat ? (sh.n_particles * sh.n_samples + kFdChunk - 1) / kFdChunk
                                  : sh.n_particles * ((sh.n_samples + kFdChunk - 1) / kFdChunk);
    const int64_t rounds = std::clamp<int64_t>((units * sh.n_pix * sh.n_wblocks + 512 * 8 - 1) / (512 * 8), 1, 4);
    auto go = [&](auto *k) {
        fd_launches(sh, gr->x_det, acc, [&](int64_t n_pix, const double *x_det, double *a) {
            FdShape part = sh;
            part.n_pix = n_pix;
            const int64_t blocks = fd_groups(part, units, 512, rounds);
            k<<<dim3((unsigned)blocks, W), 256, 0, s>>>(t->r, t->beta, t->beta_dot, t->charge, x_det, omega, a, part);
        });
    };
    if (geom == LW_GEOM_EXACT)
        W == 4 ? go(k_direct_fd<LW_GEOM_EXACT, 4>) : W == 2 ? go(k_direct_fd<LW_GEOM_EXACT, 2>) : go(k_direct_fd<LW_GEOM_EXACT, 1>);
    else
        W == 4 ? go(k_direct_fd<LW_GEOM_FARFIELD, 4>) : W == 2 ? go(k_direct_fd<LW_GEOM_FARFIELD, 2>) : go(k_direct_fd<LW_GEOM_FARFIELD, 1>);
}

template <int GEOM, int K>
void launch_mixed(const lw_traj_t *t, const lw_grid_t *gr, const double *omega, FdShape sh, double *acc, hipStream_t s)
{
    // wavefronts per block: four where they all have frequencies (or nearly), else two or one
    const int64_t waves = (sh.n_omega + 64 * K - 1) / (64 * K);
    const int W = waves >= 8 || waves % 4 == 0 ? 4 : waves % 2 == 0 ? 2 : 1;
    sh.n_wblocks = (waves + W - 1) / W;
    // up to eight rounds of the resident blocks (two wavefronts per SIMD), of at least eight chunks each
    const int64_t units = sh.n_particles * ((sh.n_samples + 64 * W - 1) / (64 * W)), resident = 2048 / W;
    const int64_t rounds = std::max<int64_t>(1, std::min<int64_t>(8, units * sh.n_pix * sh.n_wblocks / (resident * 8)));
    auto go = [&](auto *k) {
        fd_launches(sh, gr->x_det, acc, [&](int64_t n_pix, const double *x_det, double *a) {
            FdShape part = sh;
            part.n_pix = n_pix;
            const int64_t blocks = fd_groups(part, units, resident, rounds);
            k<<<(unsigned)blocks, 64 * W, 0, s>>>(t->r, t->beta, t->beta_dot, t->charge, x_det, omega, a, part);
        });
    };
    W == 4 ? go(k_direct_fd_mixed<GEOM, K, 4>) : W == 2 ? go(k_direct_fd_mixed<GEOM, K, 2>) : go(k_direct_fd_mixed<GEOM, K, 1>);
}

// frequencies per lane: the largest power of two <= 8 that still fills a wavefront
int fd_per_lane(int64_t n_omega) { return n_omega >= 64 * 8 ? 8 : n_omega >= 64 * 4 ? 4 : n_omega >= 64 * 2 ? 2 : 1; }

template <int GEOM>
void launch_mixed(const lw_traj_t *t, const lw_grid_t *gr, const double *omega, const FdShape &sh, double *acc,
                  hipStream_t s)
{
    switch (fd_per_lane(sh.n_omega)) {
    case 8: launch_mixed<GEOM, 8>(t, gr, omega, sh, acc, s); break;
    case 4: launch_mixed<GEOM, 4>(t, gr, omega, sh, acc, s); break;
    case 2: launch_mixed<GEOM, 2>(t, gr, omega, sh, acc, s); break;
    default: launch_mixed<GEOM, 1>(t, gr, omega, sh, acc, s);
    }
}

}  // namespace

lw_status launch_direct_fd(const lw_traj_t *t, const lw_grid_t *gr, const double *omega, int64_t n_omega, int prec,
                           int fmask, int geom, double *S, void *ws, size_t ws_bytes, hipStream_t s)
{
    const int64_t nS = gr->n_pix * n_omega;
    if (nS == 0) return LW_OK;
    double *acc = (double *)ws;
    k_fd_zero<<<(int)std::min<int64_t>((6 * nS + 255) / 256, 65536), 256, 0, s>>>(acc, 6 * nS);
    if (t->n_particles > 0 && t->n_samples > 0) {
        const FdShape sh = fd_shape(t, gr, n_omega, fmask);
        if (prec == LW_PREC_FP64)
            launch_sums64(t, gr, omega, sh, geom, acc, s);
        else if (geom == LW_GEOM_EXACT)
            launch_mixed<LW_GEOM_EXACT>(t, gr, omega, sh, acc, s);
        else
            launch_mixed<LW_GEOM_FARFIELD>(t, gr, omega, sh, acc, s);
    }
    const double f = t->dt * t->dt / (2.0 * kPi);
    k_fd_finish<<<(int)std::min<int64_t>((nS + 255) / 256, 65536), 256, 0, s>>>(acc, S, nS, n_omega,
                                                                              prec == LW_PREC_FP64 ? 0 : fd_per_lane(n_omega), f);
    return check_launch("lw_direct_fd");
}

lw_status launch_direct_fd_bwd(const lw_traj_t *t, const lw_grid_t *gr, const double *omega, int64_t n_omega,
                               int fmask, int geom, const double *dS, double *d_r, double *d_beta, double *d_beta_dot,
                               void *ws, size_t ws_bytes, hipStream_t s)
{
    if (gr->n_pix == 0 || n_omega == 0 || t->n_particles == 0 || t->n_samples == 0) return LW_OK;
    // forward sums F_c(w) in FP64 into the workspace (the |F|^2 pass is not needed)
    double *acc = (double *)ws;
    const int64_t nS = gr->n_pix * n_omega;
    k_fd_zero<<<(int)std::min<int64_t>((6 * nS + 255) / 256, 65536), 256, 0, s>>>(acc, 6 * nS);
    const FdShape sh = fd_shape(t, gr, n_omega, fmask);
    const int64_t chunks = (t->n_samples + 63) / 64, blocks = t->n_particles * chunks;
    launch_sums64(t, gr, omega, sh, geom, acc, s);
    const double two_f = 2.0 * t->dt * t->dt / (2.0 * kPi);
    // pixels per block: a multiple of four (a wavefront each); shares of them as far as the workspace has room
    const int64_t n = t->n_particles * t->n_samples * 3, quads = (gr->n_pix + 3) / 4;
    const size_t room = ws_bytes - direct_fd_ws_bytes(gr->n_pix, n_omega), per_share = (size_t)n * 3 * sizeof(double);
    int64_t share = std::min({quads, (kFdBwdBlocks + blocks - 1) / blocks, (int64_t)(room / per_share)});
    if (share < 2) share = 1;
    FdShape sb = sh;
    sb.parts_per_group = (quads + share - 1) / share * 4;
    const int64_t ny = (gr->n_pix + sb.parts_per_group - 1) / sb.parts_per_group;
    double *part = acc + 6 * nS;
    double *const out[3] = {ny > 1 ? part : d_r, ny > 1 ? part + n : d_beta, ny > 1 ? part + 2 * n : d_beta_dot};
    auto *k = geom == LW_GEOM_EXACT ? k_direct_fd_bwd<LW_GEOM_EXACT> : k_direct_fd_bwd<LW_GEOM_FARFIELD>;
    const int64_t most = std::max<int64_t>(1, kFdLaunch / chunks);
    for (int64_t k0 = 0; k0 < t->n_particles; k0 += most) {
        const size_t o = (size_t)k0 * t->n_samples * 3;
        k<<<dim3((unsigned)(std::min(most, t->n_particles - k0) * chunks), (unsigned)ny), 256, 0, s>>>(
            t->r + o, t->beta + o, t->beta_dot + o, t->charge ? t->charge + k0 : nullptr, gr->x_det, omega, acc, dS, out[0] + o,
            out[1] + o, out[2] + o, sb, two_f, ny > 1 ? 3 * n : 0);
    }
    if (ny > 1)
        k_fd_add<<<(unsigned)std::min<int64_t>((n + 255) / 256, 65536), 256, 0, s>>>(part, (int)ny, n, d_r, d_beta, d_beta_dot);
    return check_launch("lw_direct_fd_bwd");
}

}  // namespace lw
