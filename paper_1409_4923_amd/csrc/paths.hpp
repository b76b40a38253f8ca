// paths.hpp -- the per-path Monte Carlo step (Algorithms 1-4) as device code.
//
// One lane owns PPL paths; the whole path state lives in registers between the
// load at kernel entry and the store at exit (Sec. 5, Memory optimization).
// Instantiated per (precision, dynamics, potential, noise mask, paths per lane)
// so that each kernel contains only the arithmetic of its model.
#pragma once

#include "common.hpp"

namespace bm {

enum : int { DYN_OVERDAMPED = 0, DYN_INERTIAL = 1 };
enum : int { POT_SIN = 0, POT_RATCHET = 1, POT_TENT = 2, POT_FREE = 3 };
enum : int { NZ_GAUSS = 1, NZ_POISSON = 2, NZ_DICH = 4,
             NZ_NORMAL = 8,     // Gaussian noise with normal increments (non-simplified scheme)
             NZ_JGRID = 16 };   // Poisson kicks at their exact times (jump-adapted grid)

// Poisson kicks drawn ahead into a ring of their own (fixed grid only).
template <int NOISE> constexpr bool queued_kicks()
{
    return (NOISE & NZ_POISSON) != 0 && (NOISE & NZ_JGRID) == 0;
}

template <typename R> struct Path {
    R x;           // folded position
    int32_t w;     // folded periods
    R v;           // velocity
    int32_t sP;    // Poisson countdown
    uint32_t kP;   // Poisson kicks so far
    int32_t sD;    // dichotomous countdown
    uint32_t mD;   // dichotomous flips so far
    int32_t d;     // dichotomous state
    double thP;    // jump-adapted grid: fraction of its step at which the next kick falls
};

// ---------------------------------------------------------------------------
// -V'(x) + A, where A is the constant-within-step forcing of the step (drive,
// tilt, Poisson bias, dichotomous level) plus the potential's constant offset
// pot_offset<POT>() (folded into the drive table on the host).
// ---------------------------------------------------------------------------
// The potential's constant factor of the force: -2 pi (sine) or 2 pi (ratchet).
// In FP32 it is held in a vector register the compiler cannot see through: the
// forcing A is wave-uniform and lives in a scalar register, an FMA may read only
// one scalar operand, and with the factor as a literal (a second one) the compiler
// would copy A into a vector register at every use.  Formed once per kernel.
template <int POT, typename R> __device__ __forceinline__ R pot_factor()
{
    constexpr double TWO_PI = 6.28318530717958647692;
    const R c = (R)(POT == POT_SIN ? -TWO_PI : TWO_PI);
    if constexpr (sizeof(R) == 4) {
        R r;
        asm volatile("; pot_factor" : "=v"(r) : "0"(c));
        return r;
    } else {
        return c;
    }
}

// -V'(x) + A, with kp = pot_factor<POT>().
template <int POT> __device__ __forceinline__ float force_plus(float x, float A, float kp)
{
    if constexpr (POT == POT_SIN) {
        // V = sin(2 pi x): -V' = -2 pi cos(2 pi x); v_cos_f32 takes its argument in turns
        return __builtin_fmaf(kp, __builtin_amdgcn_cosf(x), A);
    } else if constexpr (POT == POT_RATCHET) {
        // V = -sin 2 pi x - sin(4 pi x)/4:  -V' = 2 pi c + pi (2 c^2 - 1) = c (2 pi c + 2 pi) - pi
        const float c = __builtin_amdgcn_cosf(x);
        return __builtin_fmaf(c, __builtin_fmaf(kp, c, kp), A);           // A includes -pi
    } else if constexpr (POT == POT_TENT) {
        // eq. (2), period 2: +1 on [0, 1] (V = 1 - x), -1 on (1, 2) (V = 1 + x shifted)
        const float y = x - 2.0f * floorf(x * 0.5f);
        return (y <= 1.0f ? 1.0f : -1.0f) + A;
    } else {
        return A;
    }
}

// cos 2 pi x and the sine potential's force in FP64, with the argument in turns:
// r = x - rint(x) is exact for every finite x and cos 2 pi x = sin 2 pi s with
// s = 1/4 - |r| in [-1/4, 1/4], so one odd polynomial serves every x -- no reduction by
// pi/2, no second polynomial, no quadrant and no fallback for large arguments.
// sin 2 pi s = s (c0 + z Q(z)), z = s^2, the c_k a relative minimax fit on z <= 1/16
// (Remez exchange in 60 digits: 2.6e-19) rounded to nearest, c0 in two doubles.  The
// largest errors found over 4e7 points are 2.73e-16 (near x = 0.5) and 1.43e-15 in the
// force; the rounding of the argument 2 pi x alone moves a cosine by up to 4.4e-16.
// FP64 VALU issue bounds the FP64 kernels (4.3 cycles per wave instruction and SIMD, and
// nothing issues beside it): 13 - 14 instructions per evaluation, where two polynomials
// behind a three-part reduction by pi/2 took about 45.  Inertial Poisson model, 262147 FP64
// paths x 800 steps: 1400 -> 572 us a call (533 with the jump rings); 1024 paths x 600 steps
// (the latency of one wave's chain): 300 -> 117 us (89 with fewer launches).
__device__ __forceinline__ double turn_quarter(double x) { return 0.25 - fabs(x - rint(x)); }

constexpr double SIN_C0 = 0x1.921fb54442d18p+2, SIN_C0_LO = 0x1.1a62633145c07p-52;
constexpr double SIN_C[8] = {-0x1.4abbce625be52p+5, 0x1.466bc6775aa6ep+6,  -0x1.32d2cce627542p+6,
                             0x1.50783485190c5p+5,  -0x1.e3074ddd1d40dp+3, 0x1.e8f35e9d4c4a0p+1,
                             -0x1.6f79770a5bb06p-1, 0x1.9d1b8657cb612p-4};

__device__ __forceinline__ double cos_turns(double x)
{
    const double s = turn_quarter(x), z = s * s;
    double q = SIN_C[7];
#pragma unroll
    for (int k = 6; k >= 0; --k) q = fma(q, z, SIN_C[k]);
    return fma(s, SIN_C0, s * fma(z, q, SIN_C0_LO));
}

// A - 2 pi cos 2 pi x: the same polynomial times -2 pi, its last multiplication merged
// with the addition of A.
constexpr double FORCE_C0 = -0x1.3bd3cc9be45dep+5, FORCE_C0_LO = -0x1.692b71366cc04p-49;
constexpr double FORCE_C[8] = {0x1.03c1f081b5ac3p+8, -0x1.005ed5ead8fa0p+9, 0x1.e1f5068914938p+8,
                               -0x1.084337a3092afp+8, 0x1.7b5ea6164de3cp+6, -0x1.80055d20f480dp+4,
                               0x1.209d206b45ca0p+2, -0x1.447431e6df8f9p-1};

__device__ __forceinline__ double sine_force_plus(double x, double A)
{
    const double s = turn_quarter(x), z = s * s;
    double q = FORCE_C[7];
#pragma unroll
    for (int k = 6; k >= 0; --k) q = fma(q, z, FORCE_C[k]);
    return fma(s, FORCE_C0, fma(s, fma(z, q, FORCE_C0_LO), A));
}

template <int POT> __device__ __forceinline__ double force_plus(double x, double A, double kp)
{
    if constexpr (POT == POT_SIN) {
        return sine_force_plus(x, A);
    } else if constexpr (POT == POT_RATCHET) {
        const double c = cos_turns(x);
        return fma(c, fma(kp, c, kp), A);                                 // A includes -pi
    } else if constexpr (POT == POT_TENT) {
        const double y = x - 2.0 * floor(x / 2.0);
        return (y <= 1.0 ? 1.0 : -1.0) + A;
    } else {
        return A;
    }
}

// ---------------------------------------------------------------------------
// Normal increments of the non-simplified scheme: the Box-Muller transform of
// two uniform words, r = sqrt(-2 ln(1 - phi1)), (r cos 2 pi phi2, r sin 2 pi phi2)
// with phi = w 2^-32.  1 - phi1 = (2^32 - w1) 2^-32 is formed from the integer,
// so it is exact before the conversion and never 0.
// ---------------------------------------------------------------------------
__device__ __forceinline__ void normal_pair(uint32_t w1, uint32_t w2, float &zc, float &zs)
{
    constexpr float NEG_2LN2 = -1.38629436111989061f;            // -2 ln 2
    const float om = w1 ? (float)(0u - w1) * 0x1p-32f : 1.0f;
    const float r = __builtin_amdgcn_sqrtf(NEG_2LN2 * __builtin_amdgcn_logf(om));   // log2, then scale
    const float t = (float)w2 * 0x1p-32f;                        // turns: v_sin/v_cos take 2 pi t
    zc = r * __builtin_amdgcn_cosf(t);
    zs = r * __builtin_amdgcn_sinf(t);
}

__device__ __forceinline__ void normal_pair(uint32_t w1, uint32_t w2, double &zc, double &zs)
{
    constexpr double PI = 3.14159265358979323846;
    const double om = w1 ? (double)(0u - w1) * 0x1p-32 : 1.0;
    const double r = sqrt(-2.0 * log(om));
    const double t = (double)w2 * 0x1p-32;
    zc = r * cos(2.0 * PI * t);
    zs = r * sin(2.0 * PI * t);
}

// Constant part of -V'(x) moved into the drive table.
template <int POT> constexpr double pot_offset()
{
    return POT == POT_RATCHET ? -3.14159265358979323846 : 0.0;
}

template <int POT> constexpr double period() { return POT == POT_TENT ? 2.0 : 1.0; }

// ---------------------------------------------------------------------------
// Folding of x modulo L (Sec. 5, Instruction optimization).
// ---------------------------------------------------------------------------
template <int POT, typename R> __device__ __forceinline__ void fold(Path<R> &s)
{
    if constexpr (POT == POT_TENT) {
        const R k = floor(s.x / R(2));
        s.x = s.x - k * R(2);
        s.w += (int32_t)k;
    } else {
        const R k = floor(s.x);
        s.x = s.x - k;
        s.w += (int32_t)k;
    }
}

// ---------------------------------------------------------------------------
// Jump processes.  The times and sizes of the jumps do not depend on the path state, so
// each lane draws them ahead (the same draws as in Algorithms 3 / 4 step by step) into a
// ring in LDS and the step loop only compares the step number with the next queued one.
// Before a block of steps the wave draws until every lane's ring covers it; every lane
// with room draws along, so the draws of many blocks happen side by side whichever lane
// asked for them.  (Windows of a fixed number of steps, whose draws took as many turns as
// the lane with the most jumps needed, took 1.6 times the turns at 0.016 kicks per step.)
// Windows -> rings: 500001 paths x 4000 steps on the jump-adapted grid 3.60 -> 3.33 ms,
// 262147 FP64 paths with kicks x 800 steps 558 -> 524 us (rings of 24 KiB per 256 lanes
// instead of queues of 48: four groups per CU, as the registers allow, instead of three),
// 2^20 inertial Poisson paths x 4000 steps 2.80 -> 2.70 ms.
// A ring holds one jump less than its slots: the slot behind the last queued jump is a
// sentinel with the step of the first jump not drawn yet.
// ---------------------------------------------------------------------------

// A kick of the jump-adapted grid, drawn ahead: its step, the fraction of that step at
// which it falls, its amplitude, and the Gaussian increment (times G sqrt(3 dt) or
// G sqrt(dt)) of the piece that follows it.
template <typename R> struct alignas(4 * sizeof(R)) JGKick {
    uint32_t off;
    R th, z, u;
};

// Slots of the rings by the model's fastest rate: busy = 0 up to 0.1 jumps per step, 1 up to
// 0.2, 2 beyond.  A full ring cuts the block short, a larger one costs groups per CU.
// Kicks of the fixed grid and flips: 8 slots, or 16 where a lane expects more
// than 1.6 jumps in 16 steps (500001 FP32 paths with Gaussian noise and kicks, 8 and 16 slots:
// 502 and 515 ns per step at 0.05 kicks per step, 558 and 549 at 0.1, 627 and 568 at 0.15, 768
// and 606 at 0.2; with flips as well 641 and 723 at 0.05, 869 and 883 at 0.12, 982 and 943
// at 0.15).
// Kicks of the jump-adapted grid: 6 in FP64, so that the rings of 256 lanes with flips
// fit in 64 KiB.  In FP32 9, the most that four groups of 256 lanes hold in a CU's LDS, or 12,
// with three groups (500001 paths, us per step with 9 and 12: 1.75 and 1.82 at 0.1 kicks per
// step, 2.22 and 2.22 at 0.15, 3.96 and 3.60 at 0.3, 23.5 and 20.5 at 2).  With flips 9
// beside 16 flips, three groups as well (without the digit tables of three-point increments:
// 2.41 us at 0.15, 20.7 at 2; 12 beside 8 leave two: 2.86 and 20.5); with the tables both
// leave two, and 12 beside 8 is the better (3.22 against 3.36 us at 0.15, 26.5 against 31.3
// at 2).  A step with more kicks than its ring draws the rest at the step.
template <typename R, int NOISE> constexpr RingSizes ring_sizes(uint32_t busy)
{
    constexpr bool JG = sizeof(R) == 4 && (NOISE & NZ_JGRID) != 0, FLIPS = (NOISE & NZ_DICH) != 0;
    if (JG && FLIPS && (NOISE & NZ_GAUSS) != 0) return busy >= 1u ? RingSizes{3, 12} : RingSizes{3, 9};
    return RingSizes{busy >= 1u ? 4u : 3u, sizeof(R) != 4 ? 6u : JG && !FLIPS && busy >= 2u ? 12u : 9u};
}

// A queued kick: its step and amplitude (FP64: 12 bytes, so that LDS does not limit the
// groups of a CU).
template <typename R> struct KickEntry;
template <> struct alignas(8) KickEntry<float> {
    uint32_t off;
    float z;
    __device__ static KickEntry make(uint32_t o, float v) { return KickEntry{o, v}; }
    __device__ float amplitude() const { return z; }
};
template <> struct KickEntry<double> {
    uint32_t off, lo, hi;
    __device__ static KickEntry make(uint32_t o, double v)
    {
        return KickEntry{o, (uint32_t)__double2loint(v), (uint32_t)__double2hiint(v)};
    }
    __device__ double amplitude() const { return __hiloint2double((int)hi, (int)lo); }
};

// LDS at a byte address.  The path kernels address their LDS by numbers: it is all dynamic
// and begins at 0, so ring positions wrap with one AND and no base is added at each
// access.  Static LDS would lie in front of it: the kernels have no __shared__ variable,
// name the dynamic array (use_dynamic_lds: a kernel that uses no LDS the compiler knows of
// has its stack arrays moved there), and their launchers check that none is left
// (dynamic_lds_only).
template <typename T> __device__ __forceinline__ T &lds_at(uint32_t at)
{
    return *(T *)(__attribute__((address_space(3))) T *)(uintptr_t)at;
}
__device__ __forceinline__ void use_dynamic_lds()
{
    extern __shared__ __align__(16) unsigned char smem[];
    asm volatile("" ::"v"((uint32_t)(uintptr_t)(__attribute__((address_space(3))) unsigned char *)smem));
}

// One ring's place in LDS (wave-uniform): the byte offset of its slots, the bytes from one
// slot of a lane's column to the next, and of all slots.  Positions in a ring are byte
// offsets from `base` that include the lane's column.
struct Ring {
    uint32_t base, stride, total;
};
template <typename E> inline constexpr bool ring_masked = true; // 2^k slots of 2^i bytes, 2^j columns
template <> inline constexpr bool ring_masked<KickEntry<double>> = false;
template <typename R> inline constexpr bool ring_masked<JGKick<R>> = false;
template <typename E> __device__ __forceinline__ uint32_t ring_next(const Ring &r, uint32_t at)
{
    const uint32_t n = at + r.stride;
    if constexpr (ring_masked<E>) {
        return n & (r.total - 1u);
    } else {
        const uint32_t m = n - r.total;          // huge unless n is past the last slot
        return n < m ? n : m;
    }
}
// Bytes queued between the current position and the tail.
__device__ __forceinline__ uint32_t ring_queued(const Ring &r, uint32_t at, uint32_t tail)
{
    const uint32_t d = tail - at;
    return (int32_t)d < 0 ? d + r.total : d;
}

// Exponential countdown s = floor(E / (rate dt)), E = -ln(1 - phi), phi = w 2^-32,
// decided exactly as in FP64 (the oracle's expression).  FP32 paths first form
// an FP32 estimate X32 with v_log_f32; its error is below
// 3e-7 / (rate dt) + 4.2e-7 X (rounding of 1 - phi, log2 near 1, the scale), and
// the tolerance tol0 + tol1 X is several times that, so floor(X32) is exact
// unless X32 lies within the tolerance of an integer -- then FP64 decides.  The
// FP64 work sits behind a wave-uniform branch taken only when some lane needs it
// (a few per cent of the draws); as a plain per-lane branch the compiler turns it
// into a select and evaluates the FP64 log and divide for every draw.
// The FP64 decision, out of line: inlined, its log and divide would be repeated at
// every draw site of the unrolled step loop although they rarely run.
__device__ __noinline__ uint32_t countdown_fp64(uint32_t w, double rate_dt)
{
    return (uint32_t)floor(expo64(w) / rate_dt);
}

template <typename R>
__device__ __forceinline__ uint32_t countdown(uint32_t w, double rate_dt, float c, float tol0, float tol1)
{
    if constexpr (sizeof(R) == 4) {
        const float one_minus_phi = ((float)(~w) + 1.0f) * 0x1p-32f;   // (2^32 - w) 2^-32
        const float X = -__builtin_amdgcn_logf(one_minus_phi) * c;
        const float fl = floorf(X);
        const float fr = X - fl;
        const float tol = fmaf(tol1, X, tol0);
        const bool sure = fr > tol && fr < 1.0f - tol;
        uint32_t s = (uint32_t)fl;
        if (__builtin_amdgcn_ballot_w64(!sure) != 0) {
            const uint32_t s64 = countdown_fp64(w, rate_dt);
            if (!sure) s = s64;
        }
        return s;
    }
    return countdown_fp64(w, rate_dt);
}

// Kick amplitude z = zeta E (no decision depends on it: FP32 paths use v_log_f32).
template <typename R> __device__ __forceinline__ R amplitude(const PointConst &a, uint32_t w)
{
    if constexpr (sizeof(R) == 4) {
        const float one_minus_phi = ((float)(~w) + 1.0f) * 0x1p-32f;
        return __builtin_amdgcn_logf(one_minus_phi) * a.zeta_ln2;
    } else {
        return a.zeta * expo64(w);
    }
}

// Algorithm 3 draw for kick number k: next waiting time s (steps) and amplitude z.
// Kick k uses words (2(k%2), 2(k%2)+1) of block k/2.
template <typename R>
__device__ __forceinline__ void kick_from(const PointConst &a, uint32_t ws, uint32_t wz, uint32_t &s, R &z)
{
    s = countdown<R>(ws, a.lam_dt, a.c_lam, a.tol0_lam, a.tol1);
    z = amplitude<R>(a, wz);
}

// Algorithm 4: dwell (steps) in state d_new from the flip's word w.
template <typename R>
__device__ __forceinline__ uint32_t flip_from(const PointConst &a, uint32_t w, int32_t d_new)
{
    return d_new ? countdown<R>(w, a.mub_dt, a.c_mub, a.tol0_mub, a.tol1)
                 : countdown<R>(w, a.mua_dt, a.c_mua, a.tol0_mua, a.tol1);
}

// Algorithm 4 draw for flip number m into state d_new: dwell s (steps).
template <typename R>
__device__ __forceinline__ uint32_t flip_draw(const PointConst &a, uint32_t path, uint32_t m, int32_t d_new)
{
    const U4 q = philox4x32_10(m >> 2, path, a.point, TAG_DICH, a.key0, a.key1);
    return flip_from<R>(a, pick(q, m & 3u), d_new);
}

// ---------------------------------------------------------------------------
// Algorithm 1: one predictor-corrector step.  A0 / A1 are the constant-within-
// step forcing at t_n / t_{n+1} (drive, tilt, Poisson bias, dichotomous level:
// part of the drift in all three evaluations); z is the Poisson kick, added once
// in the corrector; hh = dt / 2.
// ---------------------------------------------------------------------------
template <int DYN, int POT, bool KICK, typename R>
__device__ __forceinline__ void pc_step(Path<R> &s, R h, R hh, R ngam, R kp, R dxi, R z, R A0, R A1)
{
    // The noise increment enters all three stages unchanged, so it is added to the
    // noisy component once (vd / xd) instead of after each stage.  The trapezoid
    // of the predictor and of the corrector share the half-step term of F1:
    // y + (F1 + F) dt/2 is formed as (y + F1 dt/2) + F dt/2, one FMA on a common
    // base instead of an add and an FMA each (the same sums in another rounding
    // order).  Inertial: three cosines, six FMAs in the drifts, nine operations in
    // the stages; overdamped: three cosines and five operations in the stages.
    if constexpr (DYN == DYN_INERTIAL) {
        const R x = s.x, v = s.v, vd = v + dxi;
        const R f1 = fma(ngam, v, force_plus<POT>(x, A0, kp));
        const R xb = fma(v, h, x);                             // Euler
        const R vb = fma(f1, h, vd);
        const R f2 = fma(ngam, vb, force_plus<POT>(xb, A1, kp));
        const R xc = fma(v, hh, x), vc = fma(f1, hh, vd);      // y_n + F1 dt/2
        const R xp = fma(vb, hh, xc);                          // predictor
        const R vpr = fma(f2, hh, vc);
        const R f3 = fma(ngam, vpr, force_plus<POT>(xp, A1, kp));
        s.x = fma(vpr, hh, xc);                                // corrector
        R vn = fma(f3, hh, vc);
        if constexpr (KICK) vn = vn + z;
        s.v = vn;
    } else {
        const R x = s.x, xd = x + dxi;
        const R f1 = force_plus<POT>(x, A0, kp);
        const R xb = fma(f1, h, xd);                           // Euler
        const R f2 = force_plus<POT>(xb, A1, kp);
        const R xc = fma(f1, hh, xd);                          // y_n + F1 dt/2
        const R xp = fma(f2, hh, xc);                          // predictor
        const R f3 = force_plus<POT>(xp, A1, kp);
        R xn = fma(f3, hh, xc);                                // corrector
        if constexpr (KICK) xn = xn + z;
        s.x = xn;
    }
}

// Algorithm 1 as pc_step (no kick), also returning the local error estimate of the
// paragraph after the algorithm: chi = predictor - corrector, as max(|chi_x|, |chi_v|)
// for the inertial state (x, v).
template <int DYN, int POT, typename R>
__device__ __forceinline__ R pc_step_chi(Path<R> &s, R h, R hh, R ngam, R kp, R dxi, R A0, R A1)
{
    if constexpr (DYN == DYN_INERTIAL) {
        const R x = s.x, v = s.v, vd = v + dxi;
        const R f1 = fma(ngam, v, force_plus<POT>(x, A0, kp));
        const R xb = fma(v, h, x);                             // Euler
        const R vb = fma(f1, h, vd);
        const R f2 = fma(ngam, vb, force_plus<POT>(xb, A1, kp));
        const R xc = fma(v, hh, x), vc = fma(f1, hh, vd);      // y_n + F1 dt/2
        const R xp = fma(vb, hh, xc);                          // predictor
        const R vpr = fma(f2, hh, vc);
        const R f3 = fma(ngam, vpr, force_plus<POT>(xp, A1, kp));
        const R xn = fma(vpr, hh, xc);                         // corrector
        const R vn = fma(f3, hh, vc);
        s.x = xn;
        s.v = vn;
        return fmax(fabs(xp - xn), fabs(vpr - vn));
    } else {
        const R x = s.x, xd = x + dxi;
        const R f1 = force_plus<POT>(x, A0, kp);
        const R xb = fma(f1, h, xd);                           // Euler
        const R f2 = force_plus<POT>(xb, A1, kp);
        const R xc = fma(f1, hh, xd);                          // y_n + F1 dt/2
        const R xp = fma(f2, hh, xc);                          // predictor
        const R f3 = force_plus<POT>(xp, A1, kp);
        const R xn = fma(f3, hh, xc);                          // corrector
        s.x = xn;
        return fabs(xp - xn);
    }
}

// u * 6 mod 2^32 with two full-rate shifts (the compiler would otherwise emit a
// quarter-rate 32-bit multiply): the next base-6 digit of the fraction u / 2^32.
__device__ __forceinline__ uint32_t times6(uint32_t u)
{
    uint32_t r;
    asm("v_lshl_add_u32 %0, %1, 1, %1\n\tv_lshlrev_b32 %0, 1, %0" : "=v"(r) : "v"(u));
    return r;
}

} // namespace bm
