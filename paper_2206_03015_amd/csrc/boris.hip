// FP64 Boris trajectories of electrons in the laser pulse (the trajectory source of
// the time-domain method; the paper integrates the equations of motion with the
// Boris method), and their forward-mode tangents with respect to the initial phase
// space and the laser amplitude a0.  Samples are r, beta, beta_dot [n_particles][n_samples][3].
#include "lw_internal.h"

#include <algorithm>

namespace lw {
namespace {

// ---- dual numbers: value and ND directional derivatives --------------------------------------
template <int ND>
struct Dual {
    double v;
    double d[ND];
    Dual() = default;
    __device__ __forceinline__ Dual(double x) : v(x)
    {
#pragma unroll
        for (int j = 0; j < ND; ++j) d[j] = 0.0;
    }
};
template <int ND>
__device__ __forceinline__ Dual<ND> operator+(Dual<ND> a, Dual<ND> b)
{
    Dual<ND> r;
    r.v = a.v + b.v;
#pragma unroll
    for (int j = 0; j < ND; ++j) r.d[j] = a.d[j] + b.d[j];
    return r;
}
template <int ND>
__device__ __forceinline__ Dual<ND> operator-(Dual<ND> a, Dual<ND> b)
{
    Dual<ND> r;
    r.v = a.v - b.v;
#pragma unroll
    for (int j = 0; j < ND; ++j) r.d[j] = a.d[j] - b.d[j];
    return r;
}
template <int ND>
__device__ __forceinline__ Dual<ND> operator-(Dual<ND> a)
{
    Dual<ND> r;
    r.v = -a.v;
#pragma unroll
    for (int j = 0; j < ND; ++j) r.d[j] = -a.d[j];
    return r;
}
template <int ND>
__device__ __forceinline__ Dual<ND> operator*(Dual<ND> a, Dual<ND> b)
{
    Dual<ND> r;
    r.v = a.v * b.v;
#pragma unroll
    for (int j = 0; j < ND; ++j) r.d[j] = a.d[j] * b.v + a.v * b.d[j];
    return r;
}
template <int ND>
__device__ __forceinline__ Dual<ND> operator/(Dual<ND> a, Dual<ND> b)
{
    Dual<ND> r;
    r.v = a.v / b.v;
#pragma unroll
    for (int j = 0; j < ND; ++j) r.d[j] = (a.d[j] - r.v * b.d[j]) / b.v;
    return r;
}
template <int ND>
__device__ __forceinline__ Dual<ND> operator*(double a, Dual<ND> b)
{
    Dual<ND> r;
    r.v = a * b.v;
#pragma unroll
    for (int j = 0; j < ND; ++j) r.d[j] = a * b.d[j];
    return r;
}
template <int ND>
__device__ __forceinline__ Dual<ND> operator*(Dual<ND> b, double a)
{
    return a * b;
}
template <int ND>
__device__ __forceinline__ Dual<ND> operator/(Dual<ND> b, double a)
{
    Dual<ND> r;
    r.v = b.v / a;
#pragma unroll
    for (int j = 0; j < ND; ++j) r.d[j] = b.d[j] / a;
    return r;
}
template <int ND>
__device__ __forceinline__ Dual<ND> operator/(double a, Dual<ND> b)
{
    Dual<ND> r;
    r.v = a / b.v;
#pragma unroll
    for (int j = 0; j < ND; ++j) r.d[j] = -r.v * b.d[j] / b.v;
    return r;
}
template <int ND>
__device__ __forceinline__ Dual<ND> operator+(Dual<ND> a, double b)
{
    a.v += b;
    return a;
}
template <int ND>
__device__ __forceinline__ Dual<ND> operator+(double b, Dual<ND> a)
{
    a.v += b;
    return a;
}
template <int ND>
__device__ __forceinline__ Dual<ND> operator-(double b, Dual<ND> a)
{
    return b + (-a);
}
using ::exp;  // the double overloads stay visible beside the dual ones
using ::sincos;
using ::sqrt;
template <int ND>
__device__ __forceinline__ Dual<ND> sqrt(Dual<ND> a)
{
    Dual<ND> r;
    r.v = ::sqrt(a.v);
#pragma unroll
    for (int j = 0; j < ND; ++j) r.d[j] = a.d[j] / (2.0 * r.v);
    return r;
}
template <int ND>
__device__ __forceinline__ Dual<ND> exp(Dual<ND> a)
{
    Dual<ND> r;
    r.v = ::exp(a.v);
#pragma unroll
    for (int j = 0; j < ND; ++j) r.d[j] = a.d[j] * r.v;
    return r;
}
template <int ND>
__device__ __forceinline__ void sincos(Dual<ND> a, Dual<ND> *s, Dual<ND> *c)
{
    double sv, cv;
    ::sincos(a.v, &sv, &cv);
    s->v = sv;
    c->v = cv;
#pragma unroll
    for (int j = 0; j < ND; ++j) {
        s->d[j] = a.d[j] * cv;
        c->d[j] = -a.d[j] * sv;
    }
}
__device__ __forceinline__ double val(double a) { return a; }
template <int ND>
__device__ __forceinline__ double val(const Dual<ND> &a)
{
    return a.v;
}

// ---- the laser pulse and the pusher, written once for double and for dual numbers -----------
struct LaserDev {
    double a0, wl, w0, nc, e0_per_a0;  // wl = 2 pi c / lambda, E0 = a0 e0_per_a0, e0_per_a0 = m_e c wl / e
};

// Pulse written through its normalised vector potential a_x = a0 g(phi) sin(phi),
// g = cos^2(phi/(2 nc)) on |phi| < pi nc, phi = wl (t + z/c):
// E_x = -E0 T(rho) d(g sin)/dphi, B_y = -E_x / c, T = exp(-rho^2/w0^2) (w0 > 0).
template <typename R>
__device__ __forceinline__ void laser_eb(const LaserDev &L, R a0, R x, R y, R z, double t, R &Ex, R &By)
{
    const R phi = L.wl * (t + z / kC);
    Ex = 0.0;
    By = 0.0;
    if (!(fabs(val(phi)) < kPi * L.nc)) return;
    R sh, ch, sp, cp;
    sincos(phi / (2.0 * L.nc), &sh, &ch);
    sincos(phi, &sp, &cp);
    const R g = ch * ch;
    // g' = -sin(phi/nc)/(2 nc) = -sh ch / nc (double angle: one sin/cos pair fewer per step)
    const R gp = -((sh * ch) / L.nc);
    const R dS = gp * sp + g * cp;
    R T = 1.0;
    if (L.w0 > 0.0) T = exp(-((x * x + y * y) / (L.w0 * L.w0)));
    Ex = -(L.e0_per_a0 * (a0 * T * dS));
    By = -(Ex / kC);
}

// Boris update of u = gamma beta over time h for an electron, with E = (Ex,0,0), B = (0,By,0).
template <typename R>
__device__ __forceinline__ void kick(R &ux, R &uy, R &uz, R Ex, R By, double h)
{
    const double q = -kQe, m = kMe;
    const double a = q * h / (2.0 * m * kC);
    const R mx = ux + a * Ex, my = uy, mz = uz;
    const R gm = sqrt(1.0 + (mx * mx + my * my + mz * mz));
    const R ty = (q * h / (2.0 * m)) * By / gm;  // rotation vector (0, ty, 0)
    const R sy = 2.0 * ty / (1.0 + ty * ty);
    // u' = u- + u- x t ;  u+ = u- + u' x s
    const R px = mx - mz * ty, pz = mz + mx * ty;
    const R nx = mx - pz * sy, nz = mz + px * sy;
    ux = nx + a * Ex;
    uy = my;
    uz = nz;
}

// State of one particle's pusher at sample i: position, u = gamma beta at the sample time, u
// half a step later, and the field at (r_i, t_i).  The field is a function of the position and
// the time only, so a state saved without it and resumed at sample i recomputes it bit for bit.
template <typename R>
struct PushState {
    R x, y, z, usx, usy, usz, uhx, uhy, uhz, Ex, By;
};

template <typename R>
__device__ __forceinline__ void push_start(const LaserDev &L, R a0, const R *init, double t_start, double dt,
                                           PushState<R> &S)
{
    S.x = init[0];
    S.y = init[1];
    S.z = init[2];
    S.usx = init[3];
    S.usy = init[4];
    S.usz = init[5];
    S.uhx = S.usx;
    S.uhy = S.usy;
    S.uhz = S.usz;
    laser_eb(L, a0, S.x, S.y, S.z, t_start, S.Ex, S.By);
    kick(S.uhx, S.uhy, S.uhz, S.Ex, S.By, 0.5 * dt);
}

// r, beta and beta_dot of the sample the state stands at; ig: 1/gamma there
template <typename R>
__device__ __forceinline__ void push_sample(const PushState<R> &S, R ig, R *rr, R *bb, R *aa)
{
    const double q = -kQe, m = kMe;
    const R bx = S.usx * ig, by = S.usy * ig, bz = S.usz * ig;
    // d beta/dt = q/(gamma m c) [E + c beta x B - beta (beta.E)],  E = (Ex,0,0), B = (0,By,0)
    const R f = (q / (m * kC)) * ig;
    const R be = bx * S.Ex;
    rr[0] = S.x;
    rr[1] = S.y;
    rr[2] = S.z;
    bb[0] = bx;
    bb[1] = by;
    bb[2] = bz;
    aa[0] = f * (S.Ex - kC * (bz * S.By) - bx * be);
    aa[1] = f * (-(by * be));
    aa[2] = f * (kC * (bx * S.By) - bz * be);
}
template <typename R>
__device__ __forceinline__ void push_sample(const PushState<R> &S, R *rr, R *bb, R *aa)
{
    const R g = sqrt(1.0 + (S.usx * S.usx + S.usy * S.usy + S.usz * S.usz));
    push_sample(S, 1.0 / g, rr, bb, aa);  // one division for the four quotients by gamma
}

// one Boris step from sample i to sample i + 1 (t_next = t_start + (i + 1) dt)
template <typename R>
__device__ __forceinline__ void push_step(const LaserDev &L, R a0, double t_next, double dt, PushState<R> &S)
{
    const R gh = sqrt(1.0 + (S.uhx * S.uhx + S.uhy * S.uhy + S.uhz * S.uhz));
    const R cg = (kC * dt) / gh;  // c dt / gamma at the half step
    S.x = S.x + cg * S.uhx;
    S.y = S.y + cg * S.uhy;
    S.z = S.z + cg * S.uhz;
    R nx = S.uhx, ny = S.uhy, nz = S.uhz;
    // the field at (r_{i+1}, t_{i+1}) drives the kick and is the next sample's field
    laser_eb(L, a0, S.x, S.y, S.z, t_next, S.Ex, S.By);
    kick(nx, ny, nz, S.Ex, S.By, dt);
    S.usx = 0.5 * (S.uhx + nx);
    S.usy = 0.5 * (S.uhy + ny);
    S.usz = 0.5 * (S.uhz + nz);
    S.uhx = nx;
    S.uhy = ny;
    S.uhz = nz;
}

constexpr int kStateDoubles = 9;  // of the pusher, carried between spans

// ---------------------------------------------------------------------------------------------
// The pusher.  A particle's steps are one serial chain, so its time is one wavefront's instructions per step and
// their dependent latency until there are enough wavefronts for every SIMD: 4000 particles x 20001
// samples took 17.3 ms with one lane per particle and everything in the chain (~440 VALU instructions per
// step).  The chain here carries only what the next step needs:
//   * the samples' beta, beta_dot and the stores are other wavefronts' work: a block is one wavefront
//     of the chain and two or four that turn its states, handed over through LDS kPushSteps steps at a
//     time, into samples (lanes over particles and steps, so that a particle's steps are stored
//     next to each other);
//   * a particle has two lanes, which take the pulse's two sine/cosine pairs (carrier and envelope) in
//     one call and exchange them; everything else both lanes do alike.  Only worth it while the
//     wavefronts of paired particles find a SIMD each (kPairParticles);
//   * where no particle of the wavefront can reach the pulse within a batch of steps, the kick changes nothing and
//     the batch is three multiply-adds a step; a particle of the bunch workload is inside the pulse for a third of
//     its steps, and blocks take the particles in the order in which they meet the pulse, so that this
//     holds for most of a block's steps (67 % of them had some of 32 particles inside in the given order);
//   * inside the pulse a step has no branches (push_fast), so that its dependent sequences overlap;
//   * quotients by constants are a product with the rounded reciprocal and one residual correction
//     (Markstein: the correctly rounded quotient), the other quotients and the square roots
//     Newton/Goldschmidt iterations without the range scaling that arguments of this size do not
//     need, and a root's reciprocal comes from the root's own iteration (batches that leave the range of these forms
//     take plain roots and quotients).
// All of these round as the plain expressions do, so the samples keep their bits.  A step takes 0.47 us
// inside the pulse and 0.08 us outside: 17.3 ms at first, 10.4 with the second wavefront and the paired
// lanes, 5.0 now for 4000 particles x 20001 samples.  What is left is the latency of the dependent chain.
constexpr int kPushSteps = 8;                  // steps per hand-over of a paired block (32 particles)
constexpr int64_t kPairParticles = 32 * 1024;  // 1024 SIMDs

// x / c for a constant c with rc = 1/c rounded
__device__ __forceinline__ double div_const(double x, double c, double rc)
{
    const double q = x * rc;
    return __builtin_amdgcn_div_fixup(fma(fma(-q, c, x), rc, q), c, x);
}
// a / b for b of moderate size
__device__ __forceinline__ double div_plain(double a, double b)
{
    double y = __builtin_amdgcn_rcp(b);
    y = fma(fma(-b, y, 1.0), y, y);
    y = fma(fma(-b, y, 1.0), y, y);
    const double q = a * y;
    return __builtin_amdgcn_div_fixup(fma(fma(-b, q, a), y, q), b, a);
}
// sqrt(x) for 1e-200 < x < 1e300
__device__ __forceinline__ double sqrt_plain(double x)
{
    const double y = __builtin_amdgcn_rsq(x);
    double g = x * y, h = 0.5 * y;
    const double r = fma(-h, g, 0.5);
    g = fma(g, r, g);
    h = fma(h, r, h);
    g = fma(fma(-g, g, x), h, g);
    return fma(fma(-g, g, x), h, g);
}

// the quotients' constants; tame: the beam radius's square and its reciprocal are of moderate size
struct PushConst {
    double rc_c, nc2, rnc2, rnc, w02, rw02;
    bool tame;
};
__device__ __forceinline__ PushConst push_const(const LaserDev &L)
{
    PushConst K;
    K.rc_c = 1.0 / kC;
    K.nc2 = 2.0 * L.nc;
    K.rnc2 = 1.0 / K.nc2;
    K.rnc = 1.0 / L.nc;
    K.w02 = L.w0 > 0.0 ? L.w0 * L.w0 : 1.0;
    K.rw02 = 1.0 / K.w02;
    K.tame = K.w02 > 1e-100 && K.w02 < 1e100;
    return K;
}

// value of the pair's even (ODD = 0) or odd lane
template <int ODD>
__device__ __forceinline__ double pair_lane(double v)
{
    constexpr int kCtrl = ODD ? 0xf5 /* quad_perm 1,1,3,3 */ : 0xa0 /* quad_perm 0,0,2,2 */;
    const int lo = __builtin_amdgcn_mov_dpp(__double2loint(v), kCtrl, 0xf, 0xf, true);
    const int hi = __builtin_amdgcn_mov_dpp(__double2hiint(v), kCtrl, 0xf, 0xf, true);
    return __hiloint2double(hi, lo);
}

// the pulse's phase at (z, t)
__device__ __forceinline__ double laser_phase(const LaserDev &L, const PushConst &K, double z, double t)
{
    return L.wl * (t + div_const(z, kC, K.rc_c));
}

// laser_eb's field E_x (B_y = -E_x / c), for any parameters
template <bool PAIR>
__device__ __forceinline__ double laser_ex(const LaserDev &L, const PushConst &K, double x, double y, double z, double t,
                                           bool odd)
{
    const double phi = laser_phase(L, K, z, t);
    if (!(fabs(phi) < kPi * L.nc)) return 0.0;
    const double half = phi / K.nc2;
    double sh, ch, sp, cp;
    if constexpr (PAIR) {
        double sn, cs;
        ::sincos(odd ? phi : half, &sn, &cs);
        sh = pair_lane<0>(sn);
        ch = pair_lane<0>(cs);
        sp = pair_lane<1>(sn);
        cp = pair_lane<1>(cs);
    } else {
        ::sincos(half, &sh, &ch);
        ::sincos(phi, &sp, &cp);
    }
    const double g = ch * ch;
    const double gp = -(sh * ch / L.nc);
    const double dS = gp * sp + g * cp;
    double T = 1.0;
    if (L.w0 > 0.0) T = ::exp(-((x * x + y * y) / (L.w0 * L.w0)));
    return -(L.e0_per_a0 * (L.a0 * T * dS));
}

// sqrt(x) for x >= 1 and finite, as sqrt_plain, and 1/sqrt(x) from the same iteration
__device__ __forceinline__ void sqrt_rcp(double x, double &g, double &y)
{
    const double y0 = __builtin_amdgcn_rsq(x);
    double h = 0.5 * y0;
    g = x * y0;
    const double r = fma(-h, g, 0.5);
    g = fma(g, r, g);
    h = fma(h, r, h);
    g = fma(fma(-g, g, x), h, g);
    g = fma(fma(-g, g, x), h, g);
    y = h + h;
    y = fma(fma(-g, y, 1.0), y, y);
}
// a / b with y = 1/b; a / c for a constant c: without the fix-up of quotients that are not finite numbers
__device__ __forceinline__ double div_by(double a, double b, double y)
{
    const double q = a * y;
    return fma(fma(-b, q, a), y, q);
}

// The phases that push_fast and tangent_step take: below 2^30 in carrier and envelope (phi / (2 n_cycles), the larger one
// for less than half a cycle), with room for the rounding of a bound's sum.
__device__ __forceinline__ double phase_bound(const PushConst &K) { return 0x1p29 * fmin(1.0, K.nc2); }

// One step of the pusher (push_step's arithmetic and rounding) where u, the phase (phase_bound), the beam radius and the
// field are of moderate size: nothing here branches, so that the chain's dependent sequences (the field's sines, cosines and
// exponential, the roots and quotients) overlap as far as they can.  Returns u at the sample.
template <bool PAIR>
__device__ __forceinline__ void push_fast(const LaserDev &L, const PushConst &K, double t_next, double dt, bool odd, double &x,
                                          double &y, double &z, double &uhx, double &uhy, double &uhz, double &Ex,
                                          double &usx, double &usy, double &usz)
{
    double gh, ig;
    sqrt_rcp(1.0 + (uhx * uhx + uhy * uhy + uhz * uhz), gh, ig);
    const double cg = div_by(kC * dt, gh, ig);
    x = x + cg * uhx;
    y = y + cg * uhy;
    z = z + cg * uhz;
    const double phi = L.wl * (t_next + div_by(z, kC, K.rc_c));
    const double half = div_by(phi, K.nc2, K.rnc2);
    const double rho2 = L.w0 > 0.0 ? x * x + y * y : 0.0;
    const double T = ::exp(-div_by(rho2, K.w02, K.rw02));
    double sh, ch, sp, cp;
    // below 2^30 sincos needs no reduction of large arguments (the bound in its own terms: that branch goes)
    if constexpr (PAIR) {
        const double arg = odd ? phi : half;
        if (!(fabs(arg) < 0x1p30)) __builtin_unreachable();
        double sn, cs;
        ::sincos(arg, &sn, &cs);
        sh = pair_lane<0>(sn);
        ch = pair_lane<0>(cs);
        sp = pair_lane<1>(sn);
        cp = pair_lane<1>(cs);
    } else {
        if (!(fabs(phi) < 0x1p30) || !(fabs(half) < 0x1p30)) __builtin_unreachable();
        ::sincos(half, &sh, &ch);
        ::sincos(phi, &sp, &cp);
    }
    const double gp = -div_by(sh * ch, L.nc, K.rnc);
    const double g = ch * ch, dS = gp * sp + g * cp;
    Ex = fabs(phi) < kPi * L.nc ? -(L.e0_per_a0 * (L.a0 * T * dS)) : 0.0;
    const double By = -div_by(Ex, kC, K.rc_c);
    const double q = -kQe, m = kMe, a = q * dt / (2.0 * m * kC);
    const double mx = uhx + a * Ex, mz = uhz;
    double gm, igm;
    sqrt_rcp(1.0 + (mx * mx + uhy * uhy + mz * mz), gm, igm);
    const double ty = div_by((q * dt / (2.0 * m)) * By, gm, igm);
    const double d = 1.0 + ty * ty;
    double yd = __builtin_amdgcn_rcp(d);
    yd = fma(fma(-d, yd, 1.0), yd, yd);
    yd = fma(fma(-d, yd, 1.0), yd, yd);
    const double sy = div_by(2.0 * ty, d, yd);
    const double px = mx - mz * ty, pz = mz + mx * ty;
    const double nx = (mx - pz * sy) + a * Ex, nz = mz + px * sy;
    usx = 0.5 * (uhx + nx);
    usy = 0.5 * (uhy + uhy);
    usz = 0.5 * (uhz + nz);
    uhx = nx;
    uhz = nz;
}

// push_sample, with sqrt_rcp where u is of moderate size
__device__ __forceinline__ void push_sample_fast(const PushState<double> &S, double *rr, double *bb, double *aa)
{
    const double g2 = 1.0 + (S.usx * S.usx + S.usy * S.usy + S.usz * S.usz);
    double g, ig;
    sqrt_rcp(g2, g, ig);
    ig = div_by(1.0, g, ig);
    if (!(g2 < 1e200)) ig = 1.0 / sqrt(g2);
    push_sample(S, ig, rr, bb, aa);
}

// v of the lane that CTRL names, 0 where there is none
template <int CTRL>
__device__ __forceinline__ double dpp_double(double v)
{
    const uint64_t b = (uint64_t)__double_as_longlong(v);
    const uint32_t lo = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)(uint32_t)b, CTRL, 0xf, 0xf, false);
    const uint32_t hi = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)(uint32_t)(b >> 32), CTRL, 0xf, 0xf, false);
    return __longlong_as_double((long long)(((uint64_t)hi << 32) | lo));
}

// The hand-over buffer: x, y, z, E_x, u of S samples of P particles (an odd pitch: the particles' entries start in
// different banks)
template <int P, int S>
struct PushLds {
    static constexpr int kPitch = 8 * S + 1;
    double st[2][P * kPitch];
};

// Which particles a block pushes: those of ranks kb .. kb + P - 1 by the time at which they meet the pulse, so
// that a block's particles are inside it together.  Every block ranks all particles for itself: a histogram of
// kPushBins bins over the keys, then the candidates of its bins by (bin, index).  Keys that crowd into one bin
// (particles that meet the pulse together, or an outlier that stretches the range) are left in their
// order, by the same rule in every block.
constexpr int kPushBins = 2048, kPushCand = 512, kPushMaxBin = 240;
struct PushSort {
    int hist[kPushBins];
    int cand[kPushCand], bin[kPushCand];
    int part[4], n_cand, max_bin;
    float lo[8], hi[8];
};

__device__ __forceinline__ float pulse_time(const double *__restrict__ init, int64_t k, float early)
{
    const double *p = init + 6 * k;
    const float ux = (float)p[3], uy = (float)p[4], uz = (float)p[5];
    const float t = (early - (float)(p[2] * (1.0 / kC))) / (1.0f + uz / sqrtf(1.0f + ux * ux + uy * uy + uz * uz));
    return t > -1e30f ? fminf(t, 1e30f) : -1e30f;  // NaN among the earliest
}

// idx[p], p < P: the block's particles (-1: none).  All threads of the block; ends with a barrier.
template <int P, int NT>
__device__ void push_select(const double *__restrict__ init, int64_t n_particles, int64_t kb, float early, PushSort &q, int *idx)
{
    const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6, n = (int)n_particles;
    float lo = 3e38f, hi = -3e38f;
#pragma unroll 4
    for (int k = tid; k < n; k += NT) {
        const float t = pulse_time(init, k, early);
        lo = fminf(lo, t);
        hi = fmaxf(hi, t);
    }
    for (int off = 32; off > 0; off >>= 1) {
        lo = fminf(lo, __shfl_xor(lo, off));
        hi = fmaxf(hi, __shfl_xor(hi, off));
    }
    if (lane == 0) {
        q.lo[wv] = lo;
        q.hi[wv] = hi;
    }
    for (int j = tid; j < kPushBins; j += NT) q.hist[j] = 0;
    if (tid == 0) q.n_cand = q.max_bin = 0;
    __syncthreads();
    for (int v = 0; v < NT / 64; ++v) {
        lo = fminf(lo, q.lo[v]);
        hi = fmaxf(hi, q.hi[v]);
    }
    const float scale = hi > lo ? ((float)kPushBins - 0.5f) / (hi - lo) : 0.0f;
    auto bin_of = [&](int k) { return min((int)((pulse_time(init, k, early) - lo) * scale), kPushBins - 1); };
#pragma unroll 4
    for (int k = tid; k < n; k += NT) atomicAdd(&q.hist[bin_of(k)], 1);
    __syncthreads();
    // exclusive ranks of the bins' first particles (the first 128 threads, 16 bins each)
    constexpr int kPer = kPushBins / 128;
    int sum = 0, before = 0;
    if (tid < 128) {
        int mx = 0;
        for (int j = 0; j < kPer; ++j) {
            const int h = q.hist[kPer * tid + j];
            sum += h;
            mx = max(mx, h);
        }
        atomicMax(&q.max_bin, mx);
        before = sum;
        for (int off = 1; off < 64; off <<= 1) {
            const int o = __shfl_up(before, off);
            if (lane >= off) before += o;
        }
        if (lane == 63) q.part[wv] = before;
        before -= sum;
    }
    __syncthreads();
    if (tid < 128) {
        if (wv == 1) before += q.part[0];
        for (int j = 0; j < kPer; ++j) {
            const int h = q.hist[kPer * tid + j];
            q.hist[kPer * tid + j] = before;
            before += h;
        }
    }
    __syncthreads();
    const int r0 = (int)kb, r1 = min(r0 + P, n);
    if (q.max_bin > kPushMaxBin) {
        if (tid < P) idx[tid] = r0 + tid < n ? r0 + tid : -1;
        __syncthreads();
        return;
    }
    // candidates: bins that hold some of the ranks r0 .. r1 - 1 (fewer than P + 2 kPushMaxBin particles)
    static_assert(P + 2 * kPushMaxBin <= kPushCand, "candidates fit");
    for (int k = tid; k < n; k += NT) {
        const int b = bin_of(k), f = q.hist[b], e = b + 1 < kPushBins ? q.hist[b + 1] : n;
        if (f < r1 && e > r0) {
            const int c = atomicAdd(&q.n_cand, 1);
            if (c < kPushCand) {
                q.cand[c] = k;
                q.bin[c] = b;
            }
        }
    }
    if (tid < P) idx[tid] = -1;
    __syncthreads();
    const int nc = min(q.n_cand, kPushCand);
    for (int c = tid; c < nc; c += NT) {
        const int k = q.cand[c], b = q.bin[c];
        int rank = q.hist[b];
        for (int o = 0; o < nc; ++o) rank += q.bin[o] == b && q.cand[o] < k ? 1 : 0;
        if (rank >= r0 && rank < r1) idx[rank - r0] = k;
    }
    __syncthreads();
}

// Samples s0 .. s0 + n_span - 1 of each particle: stored in r, beta, beta_dot [n_particles][n_span][3] (OUT),
// and their max |r|^2 in rmax2 if given (fma order z^2 + (y^2 + x^2), that of the deposit's pre-pass).
// The pusher starts from init (s0 = 0) or from the state [n_particles][9] that the span ending at
// sample s0 left (spans share their boundary sample): x, y, z, u at the sample and u half a step
// later.  The field at sample s0 is that of the step that reached it (same arguments, same bits).
// The state at the last sample is left in `state` if given, and x, y, z and u half a step later of the samples
// seg - 1, 2 seg - 1 ... (seg a multiple of kPushSteps) in ck [n_particles][ck_stride] if given.
// PRE: the deposit's arrival bases and flags of the samples as well (the rules of its pre-pass, whose reading of the
// samples, 72 bytes each, was 3.8 of 29.1 ms for 10000 x 20001 samples; the launch here takes 2.4 ms more for them).
template <bool PAIR, bool OUT, bool PRE, int NC>
__global__ __launch_bounds__(64 * (1 + NC)) void k_push(const double *__restrict__ init, int64_t n_particles, int64_t s0,
                                                       int64_t n_span, double t_start, double dt, LaserDev L, int sorted,
                                                       double *__restrict__ state, double *__restrict__ r,
                                                       double *__restrict__ beta, double *__restrict__ beta_dot,
                                                       double *__restrict__ rmax2, double *__restrict__ ck,
                                                       int64_t ck_stride, int64_t seg, DepositPre pre)
{
    constexpr int P = PAIR ? 32 : 64, S = PAIR ? kPushSteps : kPushSteps / 2;
    using Lds = PushLds<P, S>;
    __shared__ union {
        Lds b;
        PushSort q;
    } lds;
    __shared__ int idx[P];
    const int lane = threadIdx.x & 63, wv = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const int64_t kb = (int64_t)blockIdx.x * P;
    bool ranked = false;
    if constexpr (PAIR) {
        ranked = sorted != 0;
        if (ranked)
            push_select<P, 64 * (1 + NC)>(init, n_particles, kb, (float)(-kPi * L.nc / L.wl - t_start), lds.q, idx);
    }
    if (!ranked) {
        if (threadIdx.x < P) idx[threadIdx.x] = kb + threadIdx.x < n_particles ? (int)(kb + threadIdx.x) : -1;
        __syncthreads();
    }
    const PushConst K = push_const(L);
    const int64_t nb = (n_span + S - 1) / S;
    if (wv == 0) {
        const int p = PAIR ? lane >> 1 : lane;
        const bool odd = PAIR && (lane & 1);
        const bool in = idx[p] >= 0;
        const int64_t k = in ? idx[p] : idx[0];
        double x, y, z, usx, usy, usz, uhx, uhy, uhz, Ex;
        double *st = state ? state + kStateDoubles * k : nullptr;
        if (s0 == 0) {
            const double *in0 = init + 6 * k;
            x = in0[0];
            y = in0[1];
            z = in0[2];
            uhx = usx = in0[3];
            uhy = usy = in0[4];
            uhz = usz = in0[5];
            Ex = laser_ex<PAIR>(L, K, x, y, z, t_start, odd);
            kick<double>(uhx, uhy, uhz, Ex, -(Ex / kC), 0.5 * dt);
        } else {
            x = st[0];
            y = st[1];
            z = st[2];
            usx = st[3];
            usy = st[4];
            usz = st[5];
            uhx = st[6];
            uhy = st[7];
            uhz = st[8];
            Ex = laser_ex<PAIR>(L, K, x, y, z, t_start + (double)s0 * dt, odd);
        }
        double *row = lds.b.st[0] + p * Lds::kPitch;
        // both lanes of a pair write the same values
        auto put = [&](double ux, double uy, double uz, double e) {
            row[0] = x;
            row[1] = y;
            row[2] = z;
            row[3] = e;
            if constexpr (OUT) {
                row[4] = ux;
                row[5] = uy;
                row[6] = uz;
            }
        };
        put(usx, usy, usz, Ex);
        double at = (double)s0;  // index of the sample the state stands at
        double cg = 0.0;         // c dt / gamma at the half step, where known
        bool have_cg = false;
        // the pulse, and how far a batch of steps can take the phase (|dz| <= c dt)
        const double lim = kPi * L.nc, far = lim + 2.01 * S * fabs(L.wl * dt) + 1e-6;
        double *ck_at = ck ? ck + k * ck_stride : nullptr;
        int64_t ck_next = seg / S - 1;  // the batch after which the next checkpoint falls
        // a step's fast form needs the phases of the whole batch within its bound: far more than covers the batch's change
        const double most = phase_bound(K) - far;
        const bool moderate = K.tame && fabs(L.e0_per_a0 * L.a0) < 1e100;
        for (int64_t b = 0; b < nb; ++b) {
            const int n = (int)std::min<int64_t>(S, n_span - b * S);
            row = lds.b.st[b & 1] + p * Lds::kPitch - (b == 0 ? 0 : 8);
            const int j0 = b == 0 ? 1 : 0;
            // one kind of step for the whole batch and wavefront
            const double phi0 = fabs(L.wl * fma(z, K.rc_c, t_start + at * dt));
            const double u2 = uhx * uhx + uhy * uhy + uhz * uhz, rho2 = x * x + y * y;
            if (__builtin_amdgcn_ballot_w64(!(phi0 > far) || !(have_cg || u2 < 1e200)) == 0) {
                // no field on the way: the kick changes nothing, u at the sample is u half a step later
                if (!have_cg) cg = div_plain(kC * dt, sqrt_plain(1.0 + u2));
                have_cg = true;
                auto coast = [&] {
                    x = x + cg * uhx;
                    y = y + cg * uhy;
                    z = z + cg * uhz;
                    row += 8;
                    put(uhx, uhy, uhz, 0.0);
                };
                at += (double)(n - j0);
                if (n - j0 == S) {
#pragma unroll
                    for (int j = 0; j < S; ++j) coast();
                } else {
                    for (int j = j0; j < n; ++j) coast();
                }
            } else if (moderate && __builtin_amdgcn_ballot_w64(!(phi0 < most) || !(u2 + rho2 < 1e200)) == 0) {
                have_cg = false;
                for (int j = j0; j < n; ++j) {
                    at += 1.0;
                    push_fast<PAIR>(L, K, t_start + at * dt, dt, odd, x, y, z, uhx, uhy, uhz, Ex, usx, usy, usz);
                    row += 8;
                    put(usx, usy, usz, Ex);
                }
            } else {
                have_cg = false;
                for (int j = j0; j < n; ++j) {
                    at += 1.0;
                    cg = (kC * dt) / sqrt(1.0 + (uhx * uhx + uhy * uhy + uhz * uhz));
                    x = x + cg * uhx;
                    y = y + cg * uhy;
                    z = z + cg * uhz;
                    double nx = uhx, ny = uhy, nz = uhz;
                    Ex = laser_ex<PAIR>(L, K, x, y, z, t_start + at * dt, odd);
                    kick<double>(nx, ny, nz, Ex, -(Ex / kC), dt);
                    row += 8;
                    put(0.5 * (uhx + nx), 0.5 * (uhy + ny), 0.5 * (uhz + nz), Ex);
                    uhx = nx;
                    uhy = ny;
                    uhz = nz;
                }
            }
            if (OUT && ck && b == ck_next && b + 1 < nb) {
                if (in && !odd) {
                    const double v[6] = {x, y, z, uhx, uhy, uhz};
#pragma unroll
                    for (int c = 0; c < 6; ++c) ck_at[c] = v[c];
                }
                ck_at += 6;
                ck_next += seg / S;
            }
            __syncthreads();  // batch b is written, batch b - 1 read
        }
        if (OUT && st && in && !odd) {
            st[0] = x;
            st[1] = y;
            st[2] = z;
            st[3] = row[4];
            st[4] = row[5];
            st[5] = row[6];
            st[6] = uhx;
            st[7] = uhy;
            st[8] = uhz;
        }
    } else {
        // lane -> (particle of a group of 64 / S, step): a particle's S steps on neighbouring lanes; the
        // P S / 64 groups are split between the NC wavefronts
        constexpr int G = 64 / S, NG = P / G / NC;
        const int j = lane & (S - 1), p0 = (wv - 1) * NG * G + lane / S;
        double mx[NG];
#pragma unroll
        for (int g = 0; g < NG; ++g) mx[g] = 0.0;
        // PRE: the lanes' samples of the batch before, and flags
        constexpr int NK = PRE ? NG : 1;
        double last[NK][3];
        bool bad[NK];
#pragma unroll
        for (int g = 0; g < NK; ++g) {
            bad[g] = false;
            last[g][0] = last[g][1] = last[g][2] = 0.0;
        }
        const double cdt = kC * dt, rc_o = PRE ? 1.0 / pre.dt_obs : 0.0;
        auto qc = [&](double v) { return div_const(v, kC, K.rc_c); };
        auto qo = [&](double v) { return div_const(v, pre.dt_obs, rc_o); };
        for (int64_t b = 0; b < nb; ++b) {
            __syncthreads();  // batch b is written
            const int64_t i = b * S + j;
            ArrivalTime tm;
            if constexpr (PRE) tm = arrival_time(t_start, dt, (double)(s0 + i), pre.t0);
            if constexpr (!PRE)
                if (i >= n_span) continue;  // PRE: every lane hands its sample on
#pragma unroll
            for (int g = 0; g < NG; ++g) {
                const int p = p0 + g * G;
                const double *row = lds.b.st[b & 1] + p * Lds::kPitch + 8 * j;
                PushState<double> Q;
                Q.x = row[0];
                Q.y = row[1];
                Q.z = row[2];
                if (!PRE || i < n_span) mx[g] = fmax(mx[g], fma(Q.z, Q.z, fma(Q.y, Q.y, Q.x * Q.x)));
                if constexpr (OUT) {
                    const int k = idx[p];
                    if constexpr (!PRE)
                        if (k < 0) continue;
                    Q.Ex = row[3];
                    Q.By = -div_const(Q.Ex, kC, K.rc_c);
                    Q.usx = row[4];
                    Q.usy = row[5];
                    Q.usz = row[6];
                    double rr[3], bb[3], aa[3];
                    push_sample_fast(Q, rr, bb, aa);
                    if constexpr (PRE) {
                        // the sample before: the neighbouring lane's, at a batch's first sample the last one's of
                        // the batch before
                        double dr[3];
#pragma unroll
                        for (int c = 0; c < 3; ++c) {
                            const double a = dpp_double<0x111>(rr[c]), f = dpp_double<0x100 + S - 1>(last[g][c]);
                            dr[c] = rr[c] - (j == 0 ? f : a);
                            last[g][c] = rr[c];
                        }
                        if (k < 0 || i >= n_span) continue;
                        const double d = arrival_base(tm, rr[2], pre.dt_obs, qc, qo);
                        pre.base[(size_t)k * n_span + i] = d;
                        const double s2 = dr[0] * dr[0] + dr[1] * dr[1] + dr[2] * dr[2];
                        const double step = s2 > 1e-200 && s2 < 1e200 ? sqrt_plain(s2) : sqrt(s2);
                        bad[g] = bad[g] || !sample_usable(rr, bb, aa) ||
                                 (i > 0 && interval_slow(d, rr[0], rr[1], rr[2], step, cdt, pre.C));
                    }
                    const size_t o = ((size_t)k * n_span + i) * 3;
#pragma unroll
                    for (int c = 0; c < 3; ++c) {
                        r[o + c] = rr[c];
                        beta[o + c] = bb[c];
                        beta_dot[o + c] = aa[c];
                    }
                }
            }
        }
        if (rmax2) {
#pragma unroll
            for (int g = 0; g < NG; ++g) {
                double m = mx[g];
                for (int off = S / 2; off > 0; off >>= 1) m = fmax(m, __shfl_xor(m, off));
                const int k = idx[p0 + g * G];
                if (j == 0 && k >= 0) rmax2[k] = m;
            }
        }
        if constexpr (PRE) {
#pragma unroll
            for (int g = 0; g < NG; ++g) {
                const uint64_t m = __builtin_amdgcn_ballot_w64(bad[g]) >> (lane & ~(S - 1));
                const int k = idx[p0 + g * G];
                if (j == 0 && k >= 0) pre.pflag[k] = (m & ((1ull << S) - 1)) != 0 ? 1 : 0;
            }
        }
    }
}

// Gradient through the pusher by forward-mode tangents: lane l handles particle k = l / 7
// and parameter p = l % 7 (init[k][0..5], then a0), runs the pusher in dual numbers seeded
// with d/dp = 1 and accumulates sum_i g_r.dr_i/dp + g_beta.dbeta_i/dp + g_bd.dbeta_dot_i/dp.
// Every trajectory depends only on its own initial condition and on a0, so these seven
// tangents per particle are the whole gradient.
constexpr int kParams = 7;

// ---------------------------------------------------------------------------------------------
// The tangents over samples s0 .. s0 + n_span - 1, in segments.  A lane's chain of steps is serial (1000 particles x
// 10001 samples: 110 wavefronts, 13.0 ms), but the tangents are linear: a segment that starts from the
// state the pusher left on its way takes the unit tangents of that state (x, y, z, u half a step later)
// and that of a0, seven lanes again, and k_tangent_join puts the segments together,
//   d(state)/dp after a segment = sum_j [d(state)/d(start_j)] d(start_j)/dp (+ the a0 lane's for p = a0),
// and likewise the segment's sums g.d(samples).  The first segment of a span starts from the parameters' own
// tangents, those of the initial conditions or those the previous span left.  The number of segments fills
// one wavefront per SIMD (1024), which is where the chains stop being latency-bound: 1000 x 10001 in 9 segments,
// 13.0 -> 1.1 ms (with the step of push_fast).  28086 particles (three wavefronts per SIMD) keep one segment.
// Two or four tangents per lane measured slower on the large workload's adjoint (444 and 448 against 326 ms): their
// registers leave fewer wavefronts.
// Workspace per particle (tstate): the state's nine values, their derivatives [7][9], the checkpoints.
constexpr int kTanCk = 9 * (1 + kParams);                // offset of the checkpoints
constexpr int kTanStateDoubles = 7 * 18;                 // per particle
constexpr int kTanSegments = 1 + (kTanStateDoubles - kTanCk) / 6;
constexpr int kTanRes = 10;                              // results per lane: nine derivatives, the sum
struct TanSegments {
    int64_t n, len;
};
TanSegments tangent_segments(int64_t n_particles, int64_t n_span)
{
    const int64_t waves = (n_particles * kParams + 63) / 64;
    const int64_t want = std::max<int64_t>(1, std::min<int64_t>({kTanSegments, 1024 / waves, n_span / 64}));
    TanSegments g;
    g.len = ((n_span + want - 1) / want + kPushSteps - 1) / kPushSteps * kPushSteps;
    g.n = (n_span + g.len - 1) / g.len;
    return g;
}

// push_fast in dual numbers (values as there; derivatives through the reciprocals at hand); da0: derivative of a0
__device__ __forceinline__ void tangent_step(const LaserDev &L, const PushConst &K, double da0, double t_next, double dt,
                                             PushState<Dual<1>> &S)
{
    using D = Dual<1>;
    const D ux = S.uhx, uy = S.uhy, uz = S.uhz;
    double gh, ig;
    sqrt_rcp(1.0 + (ux.v * ux.v + uy.v * uy.v + uz.v * uz.v), gh, ig);
    const double cg = div_by(kC * dt, gh, ig);
    const double dcg = -cg * (ux.v * ux.d[0] + uy.v * uy.d[0] + uz.v * uz.d[0]) * (ig * ig);
    S.x.v = S.x.v + cg * ux.v;
    S.y.v = S.y.v + cg * uy.v;
    S.z.v = S.z.v + cg * uz.v;
    S.x.d[0] += fma(cg, ux.d[0], dcg * ux.v);
    S.y.d[0] += fma(cg, uy.d[0], dcg * uy.v);
    S.z.d[0] += fma(cg, uz.d[0], dcg * uz.v);
    const double x = S.x.v, y = S.y.v;
    const double phi = L.wl * (t_next + div_by(S.z.v, kC, K.rc_c)), dphi = (L.wl * K.rc_c) * S.z.d[0];
    const double half = div_by(phi, K.nc2, K.rnc2);
    const bool wide = L.w0 > 0.0;
    const double T = ::exp(-div_by(wide ? x * x + y * y : 0.0, K.w02, K.rw02));
    const double dT = wide ? -2.0 * (x * S.x.d[0] + y * S.y.d[0]) * K.rw02 * T : 0.0;
    double sh, ch, sp, cp;
    if (!(fabs(phi) < 0x1p30) || !(fabs(half) < 0x1p30)) __builtin_unreachable();
    ::sincos(half, &sh, &ch);
    ::sincos(phi, &sp, &cp);
    const double gp = -div_by(sh * ch, L.nc, K.rnc);
    const double g = ch * ch, dS = gp * sp + g * cp;
    // d(dS)/dphi: g' = gp, gp' = -(ch^2 - sh^2) / (2 nc^2)
    const double dSp = fma(2.0 * gp, cp, -sp * fma(ch * ch - sh * sh, K.rnc * K.rnc2, g));
    const bool inside = fabs(phi) < kPi * L.nc;
    S.Ex.v = inside ? -(L.e0_per_a0 * (L.a0 * T * dS)) : 0.0;
    S.Ex.d[0] = inside ? -(L.e0_per_a0 * (fma(da0, T, L.a0 * dT) * dS + L.a0 * T * dSp * dphi)) : 0.0;
    S.By.v = -div_by(S.Ex.v, kC, K.rc_c);
    S.By.d[0] = -S.Ex.d[0] * K.rc_c;
    const double q = -kQe, m = kMe, a = q * dt / (2.0 * m * kC), b = q * dt / (2.0 * m);
    const double mx = ux.v + a * S.Ex.v, dmx = fma(a, S.Ex.d[0], ux.d[0]), mz = uz.v, dmz = uz.d[0];
    double gm, igm;
    sqrt_rcp(1.0 + (mx * mx + uy.v * uy.v + mz * mz), gm, igm);
    const double dgm = (mx * dmx + uy.v * uy.d[0] + mz * dmz) * igm;
    const double ty = div_by(b * S.By.v, gm, igm), dty = (b * S.By.d[0] - ty * dgm) * igm;
    const double d = 1.0 + ty * ty;
    double yd = __builtin_amdgcn_rcp(d);
    yd = fma(fma(-d, yd, 1.0), yd, yd);
    yd = fma(fma(-d, yd, 1.0), yd, yd);
    const double sy = div_by(2.0 * ty, d, yd), dsy = 2.0 * dty * fma(-sy, ty, 1.0) * yd;
    const double px = mx - mz * ty, pz = mz + mx * ty;
    const double dpx = dmx - (dmz * ty + mz * dty), dpz = dmz + (dmx * ty + mx * dty);
    D nx, nz;
    nx.v = (mx - pz * sy) + a * S.Ex.v;
    nx.d[0] = dmx - (dpz * sy + pz * dsy) + a * S.Ex.d[0];
    nz.v = mz + px * sy;
    nz.d[0] = dmz + (dpx * sy + px * dsy);
    S.usx = 0.5 * (ux + nx);
    S.usy = uy;
    S.usz = 0.5 * (uz + nz);
    S.uhx = nx;
    S.uhz = nz;
}

// g.d(sample) of the sample the state stands at (push_sample in dual numbers)
__device__ __forceinline__ double tangent_sample(const PushState<Dual<1>> &S, const double *g_r, const double *g_b,
                                                 const double *g_a, double acc)
{
    const double q = -kQe, m = kMe;
    const double ux = S.usx.v, uy = S.usy.v, uz = S.usz.v, Ex = S.Ex.v, By = S.By.v, dEx = S.Ex.d[0], dBy = S.By.d[0];
    double g, ig;
    sqrt_rcp(1.0 + (ux * ux + uy * uy + uz * uz), g, ig);
    const double dig = -(ux * S.usx.d[0] + uy * S.usy.d[0] + uz * S.usz.d[0]) * (ig * ig * ig);
    const double bx = ux * ig, by = uy * ig, bz = uz * ig;
    const double dbx = fma(S.usx.d[0], ig, ux * dig), dby = fma(S.usy.d[0], ig, uy * dig), dbz = fma(S.usz.d[0], ig, uz * dig);
    const double f = (q / (m * kC)) * ig, df = (q / (m * kC)) * dig;
    const double be = bx * Ex, dbe = fma(dbx, Ex, bx * dEx);
    const double ax = Ex - kC * (bz * By) - bx * be, ay = -(by * be), az = kC * (bx * By) - bz * be;
    const double dax = dEx - kC * fma(dbz, By, bz * dBy) - fma(dbx, be, bx * dbe);
    const double day = -fma(dby, be, by * dbe);
    const double daz = kC * fma(dbx, By, bx * dBy) - fma(dbz, be, bz * dbe);
    acc += g_r[0] * S.x.d[0] + g_b[0] * dbx + g_a[0] * fma(df, ax, f * dax);
    acc += g_r[1] * S.y.d[0] + g_b[1] * dby + g_a[1] * fma(df, ay, f * day);
    acc += g_r[2] * S.z.d[0] + g_b[2] * dbz + g_a[2] * fma(df, az, f * daz);
    return acc;
}

// sum of g.d(sample) over samples i0 .. i1 - 1 (of the span whose first sample is sample s0 of the trajectory): from
// the state at sample i0 (`at`), or from that at sample i0 - 1
__device__ __forceinline__ double tangent_run(const LaserDev &L, const PushConst &K, Dual<1> a0, int64_t s0, int64_t i0,
                                              int64_t i1, bool at, double t_start, double dt, PushState<Dual<1>> &S,
                                              const double *__restrict__ g_r, const double *__restrict__ g_b,
                                              const double *__restrict__ g_a)
{
    using D = Dual<1>;
    double acc = 0.0;
    const bool tame = S.x.v * S.x.v + S.y.v * S.y.v < 1e200 && S.uhx.v * S.uhx.v + S.uhy.v * S.uhy.v + S.uhz.v * S.uhz.v < 1e200 &&
                      S.usx.v * S.usx.v + S.usy.v * S.usy.v + S.usz.v * S.usz.v < 1e200 &&
                      fabs(laser_phase(L, K, S.z.v, t_start + (double)(s0 + i0) * dt)) +
                              2.01 * fabs(L.wl * dt) * (double)(i1 - i0) < phase_bound(K) &&
                      K.tame && fabs(L.e0_per_a0 * L.a0) < 1e100;
    if (__ballot(!tame) == 0) {
        // the gradients of kAhead samples are on their way while the kAhead before them are used: a step takes
        // less than a miss of their lines
        constexpr int kAhead = 4;
        double g[2][kAhead][9];
        auto load = [&](double (*o)[9], int64_t from) {
#pragma unroll
            for (int v = 0; v < kAhead; ++v) {
                const int64_t j = 3 * std::min(from + v, i1 - 1);
#pragma unroll
                for (int c = 0; c < 3; ++c) {
                    o[v][c] = g_r[j + c];
                    o[v][3 + c] = g_b[j + c];
                    o[v][6 + c] = g_a[j + c];
                }
            }
        };
        int64_t i = i0;
        if (at) {
            acc = tangent_sample(S, g_r + 3 * i, g_b + 3 * i, g_a + 3 * i, acc);
            ++i;
        }
        if (i >= i1) return acc;
        load(g[0], i);
        for (; i < i1; i += kAhead) {
            load(g[1], i + kAhead);
#pragma unroll
            for (int v = 0; v < kAhead; ++v) {
                if (i + v >= i1) break;
                tangent_step(L, K, a0.d[0], t_start + (double)(s0 + i + v) * dt, dt, S);
                acc = tangent_sample(S, g[0][v], g[0][v] + 3, g[0][v] + 6, acc);
            }
#pragma unroll
            for (int v = 0; v < kAhead; ++v)
#pragma unroll
                for (int c = 0; c < 9; ++c) g[0][v][c] = g[1][v][c];
        }
        return acc;
    }
    for (int64_t i = i0; i < i1; ++i) {
        if (i > i0 || !at) push_step(L, a0, t_start + (double)(s0 + i) * dt, dt, S);
        D rr[3], bb[3], aa[3];
        push_sample(S, rr, bb, aa);
        for (int c = 0; c < 3; ++c)
            acc += g_r[3 * i + c] * rr[c].d[0] + g_b[3 * i + c] * bb[c].d[0] + g_a[3 * i + c] * aa[c].d[0];
    }
    return acc;
}

// lane -> (segment, particle, seed): results [segment][kTanRes][n_particles][7] in res.  Gradients g_* [n_particles][n_span][3].  Spans share their boundary sample; the
// gradients of a boundary sample are split between the two spans' deposit adjoints (each gathers its own
// intervals), so the two contractions add up to the whole.
__global__ __launch_bounds__(64) void k_tangent_segment(const double *__restrict__ init, int64_t n_particles, int64_t s0,
                                                        int64_t n_span, int64_t n_seg, int64_t seg_len, double t_start,
                                                        double dt, LaserDev L, double *tstate,
                                                        const double *__restrict__ g_r, const double *__restrict__ g_b,
                                                        const double *__restrict__ g_a, double *__restrict__ res)
{
    using D = Dual<1>;
    const int64_t l = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    const int64_t per = n_particles * kParams, seg = l / per;
    const int64_t i0 = seg * seg_len, i1 = std::min(i0 + seg_len, n_span);
    if (i0 >= n_span) return;
    const int64_t kp = l - seg * per, k = kp / kParams;
    const int p = (int)(kp - k * kParams);
    const PushConst K = push_const(L);
    D a0(L.a0);
    a0.d[0] = p == 6 ? 1.0 : 0.0;
    PushState<D> S;
    double *st = tstate + kTanStateDoubles * k;
    if (seg > 0) {
        const double *c = st + kTanCk + 6 * (seg - 1);
        D *f[6] = {&S.x, &S.y, &S.z, &S.uhx, &S.uhy, &S.uhz};
        for (int j = 0; j < 6; ++j) {
            f[j]->v = c[j];
            f[j]->d[0] = j == p ? 1.0 : 0.0;
        }
        S.usx = S.uhx;
        S.usy = S.uhy;
        S.usz = S.uhz;
        S.Ex = S.By = 0.0;
    } else if (s0 == 0) {
        D in[6];
        for (int c = 0; c < 6; ++c) {
            in[c] = D(init[6 * k + c]);
            in[c].d[0] = c == p ? 1.0 : 0.0;
        }
        push_start(L, a0, in, t_start, dt, S);
    } else {
        D *f[9] = {&S.x, &S.y, &S.z, &S.usx, &S.usy, &S.usz, &S.uhx, &S.uhy, &S.uhz};
        for (int c = 0; c < 9; ++c) {
            f[c]->v = st[c];
            f[c]->d[0] = st[9 + 9 * p + c];
        }
        // the same arguments as the step that reached sample s0: the same field and derivative
        laser_eb(L, a0, S.x, S.y, S.z, t_start + (double)s0 * dt, S.Ex, S.By);
    }
    const size_t o = (size_t)(k * n_span) * 3;
    const double acc = tangent_run(L, K, a0, s0, i0, i1, seg == 0, t_start, dt, S, g_r + o, g_b + o, g_a + o);
    const D *f[9] = {&S.x, &S.y, &S.z, &S.uhx, &S.uhy, &S.uhz, &S.usx, &S.usy, &S.usz};
    // one segment: straight to the state (each lane has read its own), the sum to the checkpoints' place
    double *out = n_seg > 1 ? res + seg * kTanRes * per + kp : st + 9 + 9 * p;
    const int64_t step = n_seg > 1 ? per : 1;
    for (int c = 0; c < 9; ++c) out[(n_seg > 1 || c < 3 ? c : c < 6 ? c + 3 : c - 3) * step] = f[c]->d[0];
    *(n_seg > 1 ? out + 9 * per : st + kTanCk + p) = acc;
}

// thread -> (particle, parameter): the segments in order; the first span (s0 = 0) writes grad_init, grad_a0,
// later ones add to them; the pusher's state at the span's last sample and its derivatives go to tstate
__global__ __launch_bounds__(256) void k_tangent_join(int64_t n_particles, int64_t n_seg, const double *__restrict__ res,
                                                      const double *__restrict__ state, double *__restrict__ tstate, bool first,
                                                      double *__restrict__ grad_init, double *__restrict__ grad_a0)
{
    const int64_t per = n_particles * kParams, l = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (l >= per) return;
    const int64_t k = l / kParams;
    const int p = (int)(l - k * kParams);
    double *st = tstate + kTanStateDoubles * k;
    double cur[9];  // d(x, y, z, u half a step later, u)/dp
    double acc = n_seg > 1 ? res[9 * per + l] : st[kTanCk + p];
    for (int c = 0; c < 9 && n_seg > 1; ++c) cur[c] = res[c * per + l];
    for (int64_t s = 1; s < n_seg; ++s) {
        const double *q = res + s * kTanRes * per + k * kParams;
        double nxt[kTanRes];
        for (int c = 0; c < kTanRes; ++c) {
            nxt[c] = p == 6 ? q[c * per + 6] : 0.0;
            for (int j = 0; j < 6; ++j) nxt[c] = fma(q[c * per + j], cur[j], nxt[c]);
        }
        for (int c = 0; c < 9; ++c) cur[c] = nxt[c];
        acc += nxt[9];
    }
    double *d = st + 9 + 9 * p;  // x, y, z, u, u half a step later
    for (int c = 0; c < 3 && n_seg > 1; ++c) {
        d[c] = cur[c];
        d[3 + c] = cur[6 + c];
        d[6 + c] = cur[3 + c];
    }
    if (p == 0)
        for (int c = 0; c < 9; ++c) st[c] = state[kStateDoubles * k + c];
    double *out = p < 6 ? grad_init + 6 * k + p : grad_a0 + k;
    *out = first ? acc : *out + acc;
}

// whole trajectories in one segment, without a workspace
__global__ __launch_bounds__(64) void k_boris_tangent(const double *__restrict__ init, int64_t n_particles,
                                                      int64_t n_samples, double t_start, double dt, LaserDev L,
                                                      const double *__restrict__ g_r, const double *__restrict__ g_b,
                                                      const double *__restrict__ g_a, double *__restrict__ grad_init,
                                                      double *__restrict__ grad_a0)
{
    using D = Dual<1>;
    const int64_t l = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (l >= n_particles * kParams) return;
    const int64_t k = l / kParams;
    const int p = (int)(l - k * kParams);
    D in[6];
    for (int c = 0; c < 6; ++c) {
        in[c] = D(init[6 * k + c]);
        in[c].d[0] = c == p ? 1.0 : 0.0;
    }
    D a0(L.a0);
    a0.d[0] = p == 6 ? 1.0 : 0.0;
    PushState<D> S;
    push_start(L, a0, in, t_start, dt, S);
    const size_t o = (size_t)(k * n_samples) * 3;
    const double acc = tangent_run(L, push_const(L), a0, 0, 0, n_samples, true, t_start, dt, S, g_r + o, g_b + o, g_a + o);
    if (p < 6)
        grad_init[6 * k + p] = acc;
    else
        grad_a0[k] = acc;
}

LaserDev laser_dev(const lw_laser_t &l)
{
    LaserDev L;
    L.a0 = l.a0;
    L.wl = 2.0 * kPi * kC / l.lambda;
    L.w0 = l.w0;
    L.nc = l.n_cycles;
    L.e0_per_a0 = kMe * kC * L.wl / kQe;
    return L;
}

}  // namespace

// samples s0 .. s0 + n_span - 1 (r given) and / or max |r|^2 over them (rmax2 given)
static lw_status launch_push(const lw_traj_t *t, int64_t s0, int64_t n_span, double *state, double *r, double *beta,
                             double *beta_dot, double *rmax2, hipStream_t s, const char *what, double *ck = nullptr,
                             int64_t seg = kPushSteps, const DepositPre &pre = DepositPre{})
{
    if (t->n_particles == 0 || n_span == 0) return LW_OK;
    const LaserDev L = laser_dev(t->laser);
    const bool pair = t->n_particles <= kPairParticles;
    const unsigned blocks = (unsigned)((t->n_particles + (pair ? 31 : 63)) / (pair ? 32 : 64));
    // ranking costs a block three passes over the initial conditions (~1 us per 128 particles, L2), a step inside
    // the pulse ~0.4 us more than one outside
    const int sorted = pair && t->n_particles > 32 && n_span >= 256 && n_span * 16 >= t->n_particles;
    // wavefronts that form and store samples: four per block where every block has a compute unit for itself,
    // else two (10000 particles, 313 blocks: 7.6 ms with four, whose chains share SIMDs, 4.6 with two)
    auto go = [&](auto *k, int nc) {
        k<<<blocks, 64 * (1 + nc), 0, s>>>(t->init, t->n_particles, s0, n_span, t->t_start, t->dt, L, sorted, state, r, beta,
                                          beta_dot, rmax2, ck, kTanStateDoubles, seg, pre);
    };
    if (pair && blocks <= 256)
        pre.base ? go(k_push<true, true, true, 4>, 4) : r ? go(k_push<true, true, false, 4>, 4) : go(k_push<true, false, false, 4>, 4);
    else if (pair)
        pre.base ? go(k_push<true, true, true, 2>, 2) : r ? go(k_push<true, true, false, 2>, 2) : go(k_push<true, false, false, 2>, 2);
    else
        pre.base ? go(k_push<false, true, true, 2>, 2) : r ? go(k_push<false, true, false, 2>, 2) : go(k_push<false, false, false, 2>, 2);
    return check_launch(what);
}

lw_status launch_boris(const lw_traj_t *t, double *r, double *beta, double *beta_dot, hipStream_t s)
{
    // a grid counts its threads in 32 bits (three per particle), and a block's indices are 32 bits: more particles take
    // several launches
    constexpr int64_t kMost = int64_t(1) << 28;
    lw_traj_t part = *t;
    for (int64_t k0 = 0; k0 < t->n_particles; k0 += kMost) {
        part.n_particles = std::min(kMost, t->n_particles - k0);
        part.init = t->init + 6 * k0;
        const size_t o = (size_t)k0 * t->n_samples * 3;
        const lw_status st = launch_push(&part, 0, t->n_samples, nullptr, r + o, beta + o, beta_dot + o, nullptr, s,
                                         "lw_trajectory_boris");
        if (st != LW_OK) return st;
    }
    return LW_OK;
}

lw_status launch_boris_rmax2(const lw_traj_t *t, double *rmax2, hipStream_t s)
{
    return launch_push(t, 0, t->n_samples, nullptr, nullptr, nullptr, nullptr, rmax2, s,
                       "max |r|^2 of the pushed trajectories");
}

lw_status launch_boris_span(const lw_traj_t *t, int64_t s0, int64_t n_span, double *state, double *r, double *beta,
                            double *beta_dot, double *rmax2, hipStream_t s, double *tstate, const DepositPre &pre)
{
    const TanSegments g = tangent_segments(t->n_particles, n_span);
    return launch_push(t, s0, n_span, state, r, beta, beta_dot, rmax2, s, "lw_deposit_td (pusher span)",
                       tstate && g.n > 1 ? tstate + kTanCk : nullptr, g.len, pre);
}

lw_status launch_boris_bwd_span(const lw_traj_t *t, int64_t s0, int64_t n_span, const double *state, double *tstate,
                                double *res, const double *g_r, const double *g_beta, const double *g_beta_dot,
                                double *grad_init, double *grad_a0, hipStream_t s)
{
    if (t->n_particles == 0 || n_span == 0) return LW_OK;
    const LaserDev L = laser_dev(t->laser);
    const TanSegments g = tangent_segments(t->n_particles, n_span);
    const int64_t lanes = t->n_particles * kParams;
    hipEvent_t ev = timing_begin(LW_KERNEL_BORIS_TANGENT, s);
    k_tangent_segment<<<(unsigned)((lanes * g.n + 63) / 64), 64, 0, s>>>(t->init, t->n_particles, s0, n_span, g.n, g.len,
                                                                        t->t_start, t->dt, L, tstate, g_r, g_beta, g_beta_dot, res);
    timing_end(LW_KERNEL_BORIS_TANGENT, ev, s);
    k_tangent_join<<<(unsigned)((lanes + 255) / 256), 256, 0, s>>>(t->n_particles, g.n, res, state, tstate, s0 == 0, grad_init,
                                                                   grad_a0);
    return check_launch("lw_deposit_td_bwd_boris (tangent span)");
}

lw_status launch_boris_bwd(const lw_traj_t *t, const double *g_r, const double *g_beta, const double *g_beta_dot,
                           double *grad_init, double *grad_a0, hipStream_t s)
{
    if (t->n_particles == 0) return LW_OK;
    const LaserDev L = laser_dev(t->laser);
    const int64_t lanes = t->n_particles * kParams;
    const int64_t blocks = (lanes + 63) / 64;
    k_boris_tangent<<<(unsigned)blocks, 64, 0, s>>>(t->init, t->n_particles, t->n_samples, t->t_start, t->dt, L, g_r,
                                                   g_beta, g_beta_dot, grad_init, grad_a0);
    return check_launch("lw_trajectory_boris_bwd");
}

}  // namespace lw
