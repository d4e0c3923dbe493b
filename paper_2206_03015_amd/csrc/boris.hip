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

// r, beta and beta_dot of the sample the state stands at
template <typename R>
__device__ __forceinline__ void push_sample(const PushState<R> &S, R *rr, R *bb, R *aa)
{
    const double q = -kQe, m = kMe;
    const R g = sqrt(1.0 + (S.usx * S.usx + S.usy * S.usy + S.usz * S.usz));
    const R ig = 1.0 / g;  // one division for the four quotients by gamma
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

// Runs the pusher of one particle and calls emit(i, r[3], beta[3], beta_dot[3]) per sample.
template <typename R, typename Emit>
__device__ __forceinline__ void push_particle(const LaserDev &L, R a0, const R *init, int64_t n_samples,
                                              double t_start, double dt, Emit emit)
{
    PushState<R> S;
    push_start(L, a0, init, t_start, dt, S);
    for (int64_t i = 0; i < n_samples; ++i) {
        R rr[3], bb[3], aa[3];
        push_sample(S, rr, bb, aa);
        emit(i, rr, bb, aa);
        if (i + 1 == n_samples) break;
        push_step(L, a0, t_start + (double)(i + 1) * dt, dt, S);
    }
}

constexpr int kStateDoubles = 9;  // of the pusher, carried between spans

// ---------------------------------------------------------------------------------------------
// The pusher.  A particle's steps are one serial chain, and a wavefront of it issues one FP64
// instruction in four cycles whether the chip is full or not, so its time is the instructions per
// step of one wavefront until there are enough wavefronts for every SIMD: 4000 particles x 20001
// samples took 17.3 ms with one lane per particle and everything in the chain (~440 VALU
// instructions per step).  The chain here carries only what the next step needs:
//   * the samples' beta, beta_dot and the stores are another wavefront's work: a block is one wavefront
//     of the chain and one that turns its states, handed over through LDS kPushSteps steps at a
//     time, into samples (lanes over particles and steps, so that a particle's steps are stored
//     next to each other);
//   * a particle has two lanes, which take the pulse's two sine/cosine pairs (carrier and envelope) in
//     one call and exchange them; everything else both lanes do alike.  Only worth it while the
//     wavefronts of paired particles find a SIMD each (kPairParticles);
//   * quotients by constants are a product with the rounded reciprocal and one residual correction
//     (Markstein: the correctly rounded quotient), the other quotients and the square roots
//     Newton/Goldschmidt iterations without the range scaling that arguments of this size do not
//     need.
// All of these round as the plain expressions do, so the samples keep their bits.  ~250 instructions
// per step inside the pulse, 0.51 us: 17.0 -> 10.3 ms for 4000 particles x 20001 samples.  What
// is left is the latency of that dependent chain.
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
// sqrt(x) for x >= 1
__device__ __forceinline__ double sqrt_plain(double x)
{
    const double y = __builtin_amdgcn_rsq(x);
    double g = x * y, h = 0.5 * y;
    const double r = fma(-h, g, 0.5);
    g = fma(g, r, g);
    h = fma(h, r, h);
    g = fma(fma(-g, g, x), h, g);
    g = fma(fma(-g, g, x), h, g);
    return x < 1e300 ? g : x;  // infinite (or not a number)
}

// the quotients' constants
struct PushConst {
    double rc_c, nc2, rnc2, rnc, w02, rw02;
};
__device__ __forceinline__ PushConst push_const(const LaserDev &L)
{
    PushConst K;
    K.rc_c = 1.0 / kC;
    K.nc2 = 2.0 * L.nc;
    K.rnc2 = 1.0 / K.nc2;
    K.rnc = 1.0 / L.nc;
    K.w02 = L.w0 * L.w0;
    K.rw02 = 1.0 / K.w02;
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

// laser_eb's field E_x (B_y = -E_x / c)
template <bool PAIR>
__device__ __forceinline__ double laser_ex(const LaserDev &L, const PushConst &K, double x, double y, double z, double t,
                                           bool odd)
{
    const double phi = L.wl * (t + div_const(z, kC, K.rc_c));
    if (!(fabs(phi) < kPi * L.nc)) return 0.0;
    const double half = div_const(phi, K.nc2, K.rnc2);
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
    const double gp = -div_const(sh * ch, L.nc, K.rnc);
    const double dS = gp * sp + g * cp;
    double T = 1.0;
    if (L.w0 > 0.0) T = ::exp(-div_const(x * x + y * y, K.w02, K.rw02));
    return -(L.e0_per_a0 * (L.a0 * T * dS));
}

// kick, with the quotients and the square root of this kernel
__device__ __forceinline__ void kick_plain(double &ux, double &uy, double &uz, double Ex, double By, double h)
{
    const double q = -kQe, m = kMe;
    const double a = q * h / (2.0 * m * kC);
    const double mx = ux + a * Ex, my = uy, mz = uz;
    const double gm = sqrt_plain(1.0 + (mx * mx + my * my + mz * mz));
    const double ty = div_plain((q * h / (2.0 * m)) * By, gm);
    const double sy = div_plain(2.0 * ty, 1.0 + ty * ty);
    const double px = mx - mz * ty, pz = mz + mx * ty;
    const double nx = mx - pz * sy, nz = mz + px * sy;
    ux = nx + a * Ex;
    uy = my;
    uz = nz;
}

// state of one sample in the hand-over buffer: x, y, z, E_x, u (4 doubles with padding)
template <int P, int S>
struct PushLds {
    double2 st[2][P][4 * S + 1];  // one pad entry: the particles' entries start in different banks
};

// Samples s0 .. s0 + n_span - 1 of each particle: stored in r, beta, beta_dot [n_particles][n_span][3] (OUT),
// and their max |r|^2 in rmax2 if given (fma order z^2 + (y^2 + x^2), that of the deposit's pre-pass).
// The pusher starts from init (s0 = 0) or from the state [n_particles][9] that the span ending at
// sample s0 left (spans share their boundary sample): x, y, z, u at the sample and u half a step
// later.  The field at sample s0 is that of the step that reached it (same arguments, same bits).
// The state at the last sample is left in `state` if given.
template <bool PAIR, bool OUT>
__global__ __launch_bounds__(128) void k_push(const double *__restrict__ init, int64_t n_particles, int64_t s0,
                                              int64_t n_span, double t_start, double dt, LaserDev L,
                                              double *__restrict__ state, double *__restrict__ r,
                                              double *__restrict__ beta, double *__restrict__ beta_dot,
                                              double *__restrict__ rmax2)
{
    constexpr int P = PAIR ? 32 : 64, S = PAIR ? kPushSteps : kPushSteps / 2;
    __shared__ PushLds<P, S> lds;
    const int lane = threadIdx.x & 63;
    // the chain is the first wavefront of a block, or the second in every other 512 blocks: where
    // several blocks share a compute unit their chains then sit on different SIMDs
    const bool chain = (__builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6)) ^ (int)((blockIdx.x >> 9) & 1)) == 0;
    const int64_t kb = (int64_t)blockIdx.x * P;
    const PushConst K = push_const(L);
    const int64_t nb = (n_span + S - 1) / S;
    if (chain) {
        const int p = PAIR ? lane >> 1 : lane;
        const bool odd = PAIR && (lane & 1);
        const bool in = kb + p < n_particles;
        const int64_t k = in ? kb + p : n_particles - 1;
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
            kick_plain(uhx, uhy, uhz, Ex, -div_const(Ex, kC, K.rc_c), 0.5 * dt);
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
        double at = (double)s0;  // index of the sample the state stands at
        for (int64_t b = 0; b < nb; ++b) {
            const int n = (int)std::min<int64_t>(S, n_span - b * S);
            const bool last = b + 1 == nb;
            double2 *row = lds.st[b & 1][p];
            for (int j = 0; j < n; ++j) {
                if constexpr (PAIR) {
                    row[4 * j + (odd ? 2 : 0)] = odd ? make_double2(usx, usy) : make_double2(x, y);
                    row[4 * j + (odd ? 3 : 1)] = odd ? make_double2(usz, 0.0) : make_double2(z, Ex);
                } else {
                    row[4 * j] = make_double2(x, y);
                    row[4 * j + 1] = make_double2(z, Ex);
                    row[4 * j + 2] = make_double2(usx, usy);
                    row[4 * j + 3] = make_double2(usz, 0.0);
                }
                if (last && j + 1 == n) break;
                at += 1.0;
                const double gh = sqrt_plain(1.0 + (uhx * uhx + uhy * uhy + uhz * uhz));
                const double cg = div_plain(kC * dt, gh);
                x = x + cg * uhx;
                y = y + cg * uhy;
                z = z + cg * uhz;
                double nx = uhx, ny = uhy, nz = uhz;
                Ex = laser_ex<PAIR>(L, K, x, y, z, t_start + at * dt, odd);
                kick_plain(nx, ny, nz, Ex, -div_const(Ex, kC, K.rc_c), dt);
                usx = 0.5 * (uhx + nx);
                usy = 0.5 * (uhy + ny);
                usz = 0.5 * (uhz + nz);
                uhx = nx;
                uhy = ny;
                uhz = nz;
            }
            __syncthreads();  // batch b is written, batch b - 1 read
        }
        if (st && in && !odd) {
            st[0] = x;
            st[1] = y;
            st[2] = z;
            st[3] = usx;
            st[4] = usy;
            st[5] = usz;
            st[6] = uhx;
            st[7] = uhy;
            st[8] = uhz;
        }
    } else {
        // lane -> (particle of a group of 64 / S, step): a particle's S steps on neighbouring lanes
        constexpr int G = 64 / S;
        const int j = lane & (S - 1), pg = lane / S;
        double mx[P / G];
#pragma unroll
        for (int g = 0; g < P / G; ++g) mx[g] = 0.0;
        for (int64_t b = 0; b < nb; ++b) {
            __syncthreads();  // batch b is written
            const int64_t i = b * S + j;
            if (i >= n_span) continue;
#pragma unroll
            for (int g = 0; g < P / G; ++g) {
                const int p = g * G + pg;
                const double2 *row = lds.st[b & 1][p] + 4 * j;
                const double2 xy = row[0], ze = row[1];
                mx[g] = fmax(mx[g], fma(ze.x, ze.x, fma(xy.y, xy.y, xy.x * xy.x)));
                if constexpr (OUT) {
                    if (kb + p >= n_particles) continue;
                    const double2 uv = row[2], w0 = row[3];
                    PushState<double> Q;
                    Q.x = xy.x;
                    Q.y = xy.y;
                    Q.z = ze.x;
                    Q.Ex = ze.y;
                    Q.By = -div_const(ze.y, kC, K.rc_c);
                    Q.usx = uv.x;
                    Q.usy = uv.y;
                    Q.usz = w0.x;
                    double rr[3], bb[3], aa[3];
                    push_sample(Q, rr, bb, aa);
                    const size_t o = (size_t)((kb + p) * n_span + i) * 3;
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
            for (int g = 0; g < P / G; ++g) {
                double m = mx[g];
                for (int off = S / 2; off > 0; off >>= 1) m = fmax(m, __shfl_xor(m, off));
                const int64_t k = kb + g * G + pg;
                if (j == 0 && k < n_particles) rmax2[k] = m;
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
        in[c].d[0] = (c == p) ? 1.0 : 0.0;
    }
    D a0(L.a0);
    a0.d[0] = (p == 6) ? 1.0 : 0.0;
    double acc = 0.0;
    push_particle<D>(L, a0, in, n_samples, t_start, dt, [&](int64_t i, const D *rr, const D *bb, const D *aa) {
        const size_t o = (size_t)(k * n_samples + i) * 3;
        for (int c = 0; c < 3; ++c) acc += g_r[o + c] * rr[c].d[0] + g_b[o + c] * bb[c].d[0] + g_a[o + c] * aa[c].d[0];
    });
    if (p < 6)
        grad_init[6 * k + p] = acc;
    else
        grad_a0[k] = acc;
}

// The tangents over samples s0 .. s0 + n_span - 1 only, kTanND of the seven per lane: lane l
// takes particle k = l / G and parameters p = kTanND (l % G) + j (j < kTanND, p < 7), G =
// ceil(7 / kTanND) lanes per particle, so each lane runs the pusher's values once for kTanND
// tangents (the laser's sin, cos and exp serve them all).  Each lane starts from its seeded
// initial state (s0 = 0) or from the dual-number state the previous span left at sample s0
// ([lane][9 (1 + kTanND)]: the 9 state values, then their derivatives), contracts the span's
// gradients g_* [n_particles][n_span][3], saves its state at the span's last sample, and writes
// (s0 = 0) or adds its sums.  Spans share their boundary sample; the gradients of a boundary
// sample are split between the two spans' deposit adjoints (each gathers its own intervals), so
// the two contractions add up to the whole.
// One tangent per lane: two or four per lane (values computed once for them) measured slower on
// the large workload's adjoint (444 and 448 against 326 ms): their registers (221, 324) leave
// fewer wavefronts to hide the pusher's serial chain of steps.
constexpr int kTanND = 1;
constexpr int kTanLanes = (kParams + kTanND - 1) / kTanND;          // lanes per particle
constexpr int kTanStateDoubles = 9 * (1 + kTanND);                  // per lane
static_assert(kTanLanes * kTanStateDoubles <= 7 * 18, "the workspace holds 126 doubles of state per particle");

__global__ __launch_bounds__(64) void k_boris_tangent_span(const double *__restrict__ init, int64_t n_particles,
                                                           int64_t s0, int64_t n_span, double t_start, double dt,
                                                           LaserDev L, double *__restrict__ tstate,
                                                           const double *__restrict__ g_r,
                                                           const double *__restrict__ g_b,
                                                           const double *__restrict__ g_a,
                                                           double *__restrict__ grad_init,
                                                           double *__restrict__ grad_a0)
{
    using D = Dual<kTanND>;
    const int64_t l = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (l >= n_particles * kTanLanes) return;
    const int64_t k = l / kTanLanes;
    const int p0 = (int)(l - k * kTanLanes) * kTanND;  // parameters p0 .. p0 + kTanND - 1
    D a0(L.a0);
#pragma unroll
    for (int j = 0; j < kTanND; ++j) a0.d[j] = (p0 + j == 6) ? 1.0 : 0.0;
    PushState<D> S;
    double *st = tstate + kTanStateDoubles * l;
    if (s0 == 0) {
        D in[6];
        for (int c = 0; c < 6; ++c) {
            in[c] = D(init[6 * k + c]);
#pragma unroll
            for (int j = 0; j < kTanND; ++j) in[c].d[j] = (c == p0 + j) ? 1.0 : 0.0;
        }
        push_start(L, a0, in, t_start, dt, S);
    } else {
        D *f[9] = {&S.x, &S.y, &S.z, &S.usx, &S.usy, &S.usz, &S.uhx, &S.uhy, &S.uhz};
        for (int c = 0; c < 9; ++c) {
            f[c]->v = st[c];
#pragma unroll
            for (int j = 0; j < kTanND; ++j) f[c]->d[j] = st[9 + 9 * j + c];
        }
        // the same arguments as the step that reached sample s0: the same field and derivative
        laser_eb(L, a0, S.x, S.y, S.z, t_start + (double)s0 * dt, S.Ex, S.By);
    }
    double acc[kTanND];
#pragma unroll
    for (int j = 0; j < kTanND; ++j) acc[j] = 0.0;
    for (int64_t i = 0; i < n_span; ++i) {
        D rr[3], bb[3], aa[3];
        push_sample(S, rr, bb, aa);
        const size_t o = (size_t)(k * n_span + i) * 3;
        for (int c = 0; c < 3; ++c) {
            const double gr = g_r[o + c], gb = g_b[o + c], ga = g_a[o + c];
#pragma unroll
            for (int j = 0; j < kTanND; ++j) acc[j] += gr * rr[c].d[j] + gb * bb[c].d[j] + ga * aa[c].d[j];
        }
        if (i + 1 == n_span) break;
        push_step(L, a0, t_start + (double)(s0 + i + 1) * dt, dt, S);
    }
    {
        const D *f[9] = {&S.x, &S.y, &S.z, &S.usx, &S.usy, &S.usz, &S.uhx, &S.uhy, &S.uhz};
        for (int c = 0; c < 9; ++c) {
            st[c] = f[c]->v;
#pragma unroll
            for (int j = 0; j < kTanND; ++j) st[9 + 9 * j + c] = f[c]->d[j];
        }
    }
#pragma unroll
    for (int j = 0; j < kTanND; ++j) {
        const int p = p0 + j;
        if (p >= kParams) break;
        double *out = p < 6 ? grad_init + 6 * k + p : grad_a0 + k;
        *out = s0 == 0 ? acc[j] : *out + acc[j];
    }
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
                             double *beta_dot, double *rmax2, hipStream_t s, const char *what)
{
    if (t->n_particles == 0 || n_span == 0) return LW_OK;
    const LaserDev L = laser_dev(t->laser);
    const bool pair = t->n_particles <= kPairParticles;
    const unsigned blocks = (unsigned)((t->n_particles + (pair ? 31 : 63)) / (pair ? 32 : 64));
    auto *k = pair ? (r ? k_push<true, true> : k_push<true, false>) : (r ? k_push<false, true> : k_push<false, false>);
    k<<<blocks, 128, 0, s>>>(t->init, t->n_particles, s0, n_span, t->t_start, t->dt, L, state, r, beta, beta_dot, rmax2);
    return check_launch(what);
}

lw_status launch_boris(const lw_traj_t *t, double *r, double *beta, double *beta_dot, hipStream_t s)
{
    return launch_push(t, 0, t->n_samples, nullptr, r, beta, beta_dot, nullptr, s, "lw_trajectory_boris");
}

lw_status launch_boris_rmax2(const lw_traj_t *t, double *rmax2, hipStream_t s)
{
    return launch_push(t, 0, t->n_samples, nullptr, nullptr, nullptr, nullptr, rmax2, s,
                       "max |r|^2 of the pushed trajectories");
}

lw_status launch_boris_span(const lw_traj_t *t, int64_t s0, int64_t n_span, double *state, double *r, double *beta,
                            double *beta_dot, double *rmax2, hipStream_t s)
{
    return launch_push(t, s0, n_span, state, r, beta, beta_dot, rmax2, s, "lw_deposit_td (pusher span)");
}

lw_status launch_boris_bwd_span(const lw_traj_t *t, int64_t s0, int64_t n_span, double *tstate, const double *g_r,
                                const double *g_beta, const double *g_beta_dot, double *grad_init, double *grad_a0,
                                hipStream_t s)
{
    if (t->n_particles == 0 || n_span == 0) return LW_OK;
    const LaserDev L = laser_dev(t->laser);
    const int64_t lanes = t->n_particles * kTanLanes;
    const int64_t blocks = (lanes + 63) / 64;
    hipEvent_t ev = timing_begin(LW_KERNEL_BORIS_TANGENT, s);
    k_boris_tangent_span<<<(unsigned)blocks, 64, 0, s>>>(t->init, t->n_particles, s0, n_span, t->t_start, t->dt, L,
                                                        tstate, g_r, g_beta, g_beta_dot, grad_init, grad_a0);
    timing_end(LW_KERNEL_BORIS_TANGENT, ev, s);
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
