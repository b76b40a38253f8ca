// paths_kernels.hpp -- __global__ kernels of the single-ensemble path:
// initial conditions, the hot integration loop, per-path velocity with wave
// partials, and the state export.  Included once per precision/dynamics
// translation unit (paths_f32.hip, paths_f64.hip), which instantiate them.
#pragma once

#include <type_traits>

#include "bmotor.h"
#include "launch.hpp"
#include "paths.hpp"
#include "reduce.hpp"

namespace bm {

template <typename R> __device__ __forceinline__ R *arr(void *p) { return reinterpret_cast<R *>(p); }

template <typename R>
__device__ __forceinline__ R three_point(uint32_t u, R g3)
{
    return u < T_MINUS ? -g3 : (u < T_PLUS ? g3 : R(0));
}

template <typename R, int POT, int NOISE>
__device__ __forceinline__ void load_path(const KArgs &a, uint32_t p, Path<R> &s)
{
    s.x = arr<R>(a.x)[p];
    s.w = a.w[p];
    s.v = arr<R>(a.v)[p];
    if constexpr ((NOISE & NZ_POISSON) != 0) { s.sP = a.sP[p]; s.kP = a.kP[p]; }
    else { s.sP = 0; s.kP = 0u; }
    if constexpr ((NOISE & NZ_JGRID) != 0) s.thP = a.thP[p];
    else s.thP = 0.0;
    if constexpr ((NOISE & NZ_DICH) != 0) { s.sD = a.sD[p]; s.mD = a.mD[p]; s.d = a.d[p]; }
    else { s.sD = 0; s.mD = 0u; s.d = 0; }
}

template <typename R, int POT, int NOISE>
__device__ __forceinline__ void store_path(const KArgs &a, uint32_t p, const Path<R> &s)
{
    arr<R>(a.x)[p] = s.x;
    a.w[p] = s.w;
    arr<R>(a.v)[p] = s.v;
    if constexpr ((NOISE & NZ_POISSON) != 0) { a.sP[p] = s.sP; a.kP[p] = s.kP; }
    if constexpr ((NOISE & NZ_JGRID) != 0) a.thP[p] = s.thP;
    if constexpr ((NOISE & NZ_DICH) != 0) { a.sD[p] = s.sD; a.mD[p] = s.mD; a.d[p] = s.d; }
}

// Constant-within-step forcing at phase k: drive + tilt - Poisson bias + potential
// offset, from the host-built table (period a.spp >= 1, extended by 16 entries so
// that the 17 values of a 16-step block are contiguous).
template <typename R> __device__ __forceinline__ R drive_at(const PointConst &a, uint32_t k)
{
    return reinterpret_cast<const R *>(a.tab)[k];
}

// Per-lane cursors into the rings.  Steps are absolute step numbers modulo 2^32 (a run has
// fewer than 2^32 steps and a countdown fewer than 2^31).  cX: position of the current
// entry, whose contents are in registers; tX: position of the sentinel.
template <typename R> struct JumpCursor {
    uint32_t nP;    // step of the next kick
    R zP;           // its amplitude
    uint32_t cP, tP;
    uint32_t uP;    // step of the first kick not drawn
    uint32_t nD;    // step of the next flip
    uint32_t cD, tD;
    uint32_t uD;    // step of the first flip not drawn
    int32_t dT;     // state after the flips drawn
    R lev;          // dichotomous level of the current state
    // jump-adapted grid
    JGKick<R> g;    // next kick
    uint32_t cG, tG;
    uint32_t poff;  // step of the first kick not drawn
    double pth;     // its fraction of the step (FP64: kick times decide the integer state)
};

// Forcing at the time t_n + theta dt inside a step of drive phase k (jump-adapted
// grid): a cos(2 pi (k + theta) / spp) + tilt - Poisson bias + potential offset.
// The phase k may be passed unreduced (k < spp + 16): cos is periodic in it.
template <typename R> __device__ __forceinline__ R drive_inside(const PointConst &a, uint32_t k, double th)
{
    if constexpr (sizeof(R) == 4) {
        const float turns = ((float)k + (float)th) * a.inv_spp;      // within 2 ulp of the quotient
        return (float)a.drive_a * __builtin_amdgcn_cosf(turns) + (float)a.drive_c;
    } else {
        constexpr double PI = 3.14159265358979323846;
        return a.drive_a * cos(2.0 * PI * ((double)k + th) / (double)a.spp) + a.drive_c;
    }
}

// Gaussian increment (times G sqrt(3 dt) or G sqrt(dt)) of the piece that follows
// kick k on the jump-adapted grid (tag 5, indexed by kick number).
template <typename R, int NOISE>
__device__ __forceinline__ R piece_noise(const PointConst &a, uint32_t path, uint32_t k, R g3)
{
    if constexpr ((NOISE & NZ_GAUSS) != 0) {
        const U4 q = philox4x32_10(k >> 4, path, a.point, TAG_KICK_NOISE, a.key0, a.key1);
        uint32_t u = pick(q, (k >> 2) & 3u);
        for (uint32_t t = 0; t < (k & 3u); ++t) u = times6(u);
        return three_point<R>(u, g3);
    } else if constexpr ((NOISE & NZ_NORMAL) != 0) {
        const U4 q = philox4x32_10(k >> 2, path, a.point, TAG_KICK_NOISE, a.key0, a.key1);
        const bool hi = ((k >> 1) & 1u) != 0;
        R zc, zs;
        normal_pair(hi ? q.z : q.x, hi ? q.w : q.y, zc, zs);
        return g3 * ((k & 1u) ? zs : zc);
    } else {
        return R(0);
    }
}

// sqrt of a piece's fraction of the step: the hardware square root (1 ulp) in FP32,
// the correctly rounded one in FP64.
__device__ __forceinline__ float piece_sqrt(float f) { return __builtin_amdgcn_sqrtf(f); }
__device__ __forceinline__ double piece_sqrt(double f) { return sqrt(f); }

// Most kicks one step of the jump-adapted grid may hold (a Poisson(16) count
// exceeds it with probability below 10^-1000).
constexpr uint32_t JG_MAX_KICKS = 4096;

// Time of the next kick in steps from the start of the current one's step: th + E /
// (lambda dt) in FP64 (out of line: it is needed once per kick, not per step).
__device__ __noinline__ double jg_next_time(double th, uint32_t w, double lam_dt)
{
    return th + expo64(w) / lam_dt;
}

// Draws the kick that falls at (off, th) -- its amplitude, the
// increment of the piece after it -- and the time of the next kick, counted from
// it in FP64: off += floor(T), th = T - floor(T) with T = th + E / (lambda dt).
template <typename R, int NOISE>
__device__ __forceinline__ JGKick<R> jg_draw(const PointConst &a, uint32_t path, uint32_t &kP, uint32_t &off,
                                             double &th)
{
    const U4 b = philox4x32_10(kP >> 1, path, a.point, TAG_POISSON, a.key0, a.key1);
    const bool second = (kP & 1u) != 0u;
    JGKick<R> e;
    e.off = off;
    e.th = (R)th;
    e.z = amplitude<R>(a, second ? b.w : b.y);
    e.u = piece_noise<R, NOISE>(a, path, kP, (R)a.g3);
    const double T = jg_next_time(th, second ? b.z : b.x, a.lam_dt);
    const double Tf = floor(T);
    off += (uint32_t)Tf;                     // Tf < 2^31: validated on the host
    th = T - Tf;
    ++kP;
    return e;
}

// The same draw out of line, for the step that holds more kicks than a ring.  Arguments and
// results go by value, so that the caller's state stays in registers, and are few enough to
// go in registers themselves: the whole PointConst went through scratch memory at every call
// (500001 paths at 8 kicks per step: 172 -> 69 us per step).
template <typename R> struct JGDrawn {
    JGKick<R> e;
    double th;
    uint32_t kP, off;
};
template <typename R, int NOISE>
__device__ __noinline__ JGDrawn<R> jg_draw_call(uint32_t key0, uint32_t key1, uint32_t point, double lam_dt, R zeta,
                                                R g3, uint32_t path, uint32_t kP, uint32_t off, double th)
{
    PointConst a;
    a.key0 = key0;
    a.key1 = key1;
    a.point = point;
    a.lam_dt = lam_dt;
    a.g3 = g3;
    if constexpr (sizeof(R) == 4) a.zeta_ln2 = zeta;
    else a.zeta = zeta;
    JGDrawn<R> d;
    d.e = jg_draw<R, NOISE>(a, path, kP, off, th);
    d.th = th;
    d.kP = kP;
    d.off = off;
    return d;
}
template <typename R, int NOISE>
__device__ __forceinline__ JGDrawn<R> jg_draw_inline(const PointConst &a, uint32_t path, uint32_t kP, uint32_t off,
                                                     double th)
{
    const R zeta = sizeof(R) == 4 ? (R)a.zeta_ln2 : (R)a.zeta;
    return jg_draw_call<R, NOISE>(a.key0, a.key1, a.point, a.lam_dt, zeta, (R)a.g3, path, kP, off, th);
}

// Moves the cursor past the kick just applied.  Every kick of a block is queued; only the
// single-step fallback (INL) draws past its ring, those of its own step `off`.
template <typename R, int NOISE, bool INL>
__device__ __forceinline__ void jg_advance(const PointConst &a, uint32_t path, uint32_t off, uint32_t &kP,
                                           JumpCursor<R> &J, const Ring &gr)
{
    if (!INL || J.cG != J.tG) {
        J.cG = ring_next<JGKick<R>>(gr, J.cG);
        J.g = lds_at<JGKick<R>>(gr.base + J.cG);
    }
    if (INL && J.cG == J.tG) {
        if (J.poff == off) {
            const JGDrawn<R> d = jg_draw_inline<R, NOISE>(a, path, kP, J.poff, J.pth);
            J.g = d.e;
            J.pth = d.th;
            J.poff = d.off;
            kP = d.kP;
        } else {
            J.g.off = J.poff;
        }
    }
}

// One step of the jump-adapted grid.  When no lane of the wave has a kick in this
// step it is a plain Algorithm 1 step.  Otherwise every lane integrates the first
// piece of its step -- the whole step, or up to its first kick at t_n + theta dt --
// with the same instructions; lanes with a kick then integrate the remaining pieces
// (one per further kick in the step, then the rest of the step).  The first piece
// takes the step's own Gaussian increment scaled by sqrt(theta); a piece after
// kick k takes the increment drawn for k.
// The pieces of a kicked lane's step after its first kick (at fraction `from`, drive
// A_from there, u the increment of the next piece): one per further kick in the step,
// then the rest of the step.  The cursor already points past the first kick.
template <typename R, int DYN, int POT, int NOISE, bool INL>
__device__ __forceinline__ void jg_rest(const PointConst &a, uint32_t path, Path<R> &s, JumpCursor<R> &J,
                                        const Ring &gr, uint32_t off,
                                        uint32_t kph, R h, R hh, R ngam, R kp, R A1, R lev, R from, R A_from, R u)
{
    // further kicks in this step (lambda dt <= 16 is enforced on the host; the bound
    // only guarantees that every lane leaves the loop)
    for (uint32_t it = 0; J.g.off == off && it < JG_MAX_KICKS; ++it) {
        const R th = J.g.th;
        const R A_th = drive_inside<R>(a, kph, (double)th) + lev;
        pc_step<DYN, POT, true, R>(s, (th - from) * h, (th - from) * hh, ngam, kp, u * piece_sqrt(th - from), J.g.z,
                                   A_from, A_th);
        from = th;
        A_from = A_th;
        u = J.g.u;
        jg_advance<R, NOISE, INL>(a, path, off, s.kP, J, gr);
    }
    pc_step<DYN, POT, false, R>(s, (R(1) - from) * h, (R(1) - from) * hh, ngam, kp, u * piece_sqrt(R(1) - from), R(0),
                                A_from, A1);
}

template <typename R, int DYN, int POT, int NOISE, bool INL>
__device__ __forceinline__ void jg_step(const PointConst &a, uint32_t path, Path<R> &s, JumpCursor<R> &J,
                                        const Ring &gr, uint32_t off,
                                        uint32_t kph, R dxi, R h, R hh, R ngam, R kp, R A0, R A1, R lev)
{
    const bool kick = J.g.off == off;
    const bool any = __builtin_amdgcn_ballot_w64(kick) != 0;      // some lane of the wave kicks now
    R th1 = R(1), A_e = A1, dxi1 = dxi, z1 = R(0);
    if constexpr (sizeof(R) == 4 && !INL) {
        // FP32: one instance of the first piece for every step.  When a lane of the
        // wave kicks, the kick's length, drive, increment and amplitude are formed in
        // every lane and selected (no divergent branch; the cosine and the square root
        // go to the transcendental unit); otherwise the piece is the whole step
        // (th1 = 1 makes th1 dt exact).
        if (any) {
            const R thk = J.g.th;
            R A_k = drive_inside<R>(a, kph, (double)thk);
            if constexpr ((NOISE & NZ_DICH) != 0) A_k = A_k + lev;
            const R dxk = dxi * piece_sqrt(thk);
            th1 = kick ? thk : R(1);
            A_e = kick ? A_k : A1;
            dxi1 = kick ? dxk : dxi;
            z1 = kick ? J.g.z : R(0);
        }
        pc_step<DYN, POT, true, R>(s, th1 * h, th1 * hh, ngam, kp, dxi1, z1, A0, A_e);
        if (!any) return;
        // the kicked lanes' cursors move on: every lane reads the entry after its
        // cursor, the kicked lanes take it
        const R u_after = J.g.u;                 // increment of the piece after the kick
        const uint32_t nx = ring_next<JGKick<R>>(gr, J.cG);
        const JGKick<R> e = lds_at<JGKick<R>>(gr.base + nx);
        J.cG = kick ? nx : J.cG;
        J.g.off = kick ? e.off : J.g.off;
        J.g.th = kick ? e.th : J.g.th;
        J.g.z = kick ? e.z : J.g.z;
        J.g.u = kick ? e.u : J.g.u;
        if (kick) jg_rest<R, DYN, POT, NOISE, INL>(a, path, s, J, gr, off, kph, h, hh, ngam, kp, A1, lev, th1, A_e,
                                                   u_after);
    } else {
        if (!any) {
            pc_step<DYN, POT, false, R>(s, h, hh, ngam, kp, dxi, R(0), A0, A1);
            return;
        }
        if (kick) {
            th1 = J.g.th;
            A_e = drive_inside<R>(a, kph, (double)th1) + lev;
            dxi1 = dxi * piece_sqrt(th1);
            z1 = J.g.z;
        }
        pc_step<DYN, POT, true, R>(s, th1 * h, th1 * hh, ngam, kp, dxi1, z1, A0, A_e);
        if (kick) {
            const R u_after = J.g.u;
            jg_advance<R, NOISE, INL>(a, path, off, s.kP, J, gr);
            jg_rest<R, DYN, POT, NOISE, INL>(a, path, s, J, gr, off, kph, h, hh, ngam, kp, A1, lev, th1, A_e,
                                             u_after);
        }
    }
}

// One step of one path, step number `off` (drive phase kph): flips due at this
// step, Algorithm 1, and the Poisson kick due at this step, which Algorithm 3 adds
// to the corrector's result.  `dxi` is the Algorithm 2 increment.  (Folding is
// done by the caller.)  QUIET: no lane of the wave has a jump at this step (nothing to
// test).
template <typename R, int DYN, int POT, int NOISE, bool INL = false, bool QUIET = false>
__device__ __forceinline__ void full_step(const PointConst &a, uint32_t path, Path<R> &s, JumpCursor<R> &J,
                                          const Ring &kr, const Ring &gr, const Ring &fr,
                                          uint32_t off, uint32_t kph, R dxi, R h, R hh, R ngam, R kp,
                                          R A0, R A1, R Fa, R Fb)
{
    if constexpr ((NOISE & NZ_DICH) != 0 && !QUIET) {
        const bool flip = J.nD == off;           // Algorithm 4: s <= 0 at this step
        if ((NOISE & NZ_POISSON) != 0 || __builtin_amdgcn_ballot_w64(flip) != 0) {
            if (flip) {
                s.d = 1 - s.d;
                J.lev = s.d ? Fb : -Fa;
                J.cD = ring_next<uint32_t>(fr, J.cD);
                J.nD = lds_at<uint32_t>(fr.base + J.cD);
                // The entry is waited for here, in the rare flip: waited for at the next step's
                // compare, the kick read just before would be waited for as well (20000 FP32
                // paths with kicks and flips: 130 -> 113 ns per step; flips alone, 0.15 per
                // step, and FP64 lose 3% by it).
                if constexpr (sizeof(R) == 4 && queued_kicks<NOISE>()) asm volatile("" : "+v"(J.nD));
            }
        }
    }
    R lev = R(0);
    if constexpr ((NOISE & NZ_DICH) != 0) {
        lev = J.lev;
        A0 = A0 + lev;
        A1 = A1 + lev;
    }
    if constexpr ((NOISE & NZ_JGRID) != 0 && !QUIET) {
        jg_step<R, DYN, POT, NOISE, INL>(a, path, s, J, gr, off, kph, dxi, h, hh, ngam, kp, A0, A1, lev);
    } else {
        pc_step<DYN, POT, false, R>(s, h, hh, ngam, kp, dxi, R(0), A0, A1);
    }
    if constexpr (queued_kicks<NOISE>() && !QUIET) {
        if (J.nP == off) {                       // Algorithm 3: s <= 0 at this step
            if constexpr (DYN == DYN_INERTIAL) s.v = s.v + J.zP;
            else s.x = s.x + J.zP;
            J.cP = ring_next<KickEntry<R>>(kr, J.cP);
            const KickEntry<R> e = lds_at<KickEntry<R>>(kr.base + J.cP);
            J.nP = e.off;
            J.zP = e.amplitude();
        }
    }
}

// Draws for the rings, one turn: every lane with room draws (at most two kicks, the halves
// of one Philox block; at most two flips; one kick of the jump-adapted grid), but only
// jumps before step n + left, the end of the call: nothing is drawn that the call does not
// apply.  Each returns whether this lane still needs a jump before step n + run and has
// room for it.
template <typename R>
__device__ __forceinline__ bool draw_kicks(const PointConst &a, uint32_t path, uint32_t n, uint32_t run, uint32_t left,
                                           uint32_t &kP, JumpCursor<R> &J, const Ring &r)
{
    using E = KickEntry<R>;
    uint32_t room = r.total - r.stride - ring_queued(r, J.cP, J.tP);            // bytes
    if (room != 0u && J.uP - n < left) {
        const U4 b = philox4x32_10(kP >> 1, path, a.point, TAG_POISSON, a.key0, a.key1);
        const bool odd = (kP & 1u) != 0u;
        uint32_t sn;
        R z;
        kick_from<R>(a, odd ? b.z : b.x, odd ? b.w : b.y, sn, z);
        lds_at<E>(r.base + J.tP) = E::make(J.uP, z);
        J.tP = ring_next<E>(r, J.tP);
        J.uP += 1u + sn;
        ++kP;
        room -= r.stride;
        if (!odd && room != 0u && J.uP - n < left) {
            kick_from<R>(a, b.z, b.w, sn, z);
            lds_at<E>(r.base + J.tP) = E::make(J.uP, z);
            J.tP = ring_next<E>(r, J.tP);
            J.uP += 1u + sn;
            ++kP;
            room -= r.stride;
        }
    }
    return room != 0u && J.uP - n < run;
}

template <typename R>
__device__ __forceinline__ bool draw_flips(const PointConst &a, uint32_t path, uint32_t n, uint32_t run, uint32_t left,
                                           uint32_t &mD, JumpCursor<R> &J, const Ring &r)
{
    uint32_t room = r.total - r.stride - ring_queued(r, J.cD, J.tD);
    if (room != 0u && J.uD - n < left) {
        const U4 q = philox4x32_10(mD >> 2, path, a.point, TAG_DICH, a.key0, a.key1);
        const uint32_t w = mD & 3u;
        J.dT = 1 - J.dT;
        const uint32_t s0 = flip_from<R>(a, pick(q, w), J.dT);
        lds_at<uint32_t>(r.base + J.tD) = J.uD;
        J.tD = ring_next<uint32_t>(r, J.tD);
        J.uD += 1u + s0;
        ++mD;
        room -= r.stride;
        if (w != 3u && room != 0u && J.uD - n < left) {
            J.dT = 1 - J.dT;
            const uint32_t s1 = flip_from<R>(a, pick(q, w + 1u), J.dT);
            lds_at<uint32_t>(r.base + J.tD) = J.uD;
            J.tD = ring_next<uint32_t>(r, J.tD);
            J.uD += 1u + s1;
            ++mD;
            room -= r.stride;
        }
    }
    return room != 0u && J.uD - n < run;
}

template <typename R, int NOISE>
__device__ __forceinline__ bool draw_jg(const PointConst &a, uint32_t path, uint32_t n, uint32_t run, uint32_t left,
                                        uint32_t &kP, JumpCursor<R> &J, const Ring &r)
{
    using E = JGKick<R>;
    uint32_t room = r.total - r.stride - ring_queued(r, J.cG, J.tG);
    if (room != 0u && J.poff - n < left) {
        lds_at<E>(r.base + J.tG) = jg_draw<R, NOISE>(a, path, kP, J.poff, J.pth);
        J.tG = ring_next<E>(r, J.tG);
        room -= r.stride;
    }
    return room != 0u && J.poff - n < run;
}

// Three-point increments from a table of digit pairs in LDS, one table per wave (the
// waves of a scan hold different points): entry 6 a + b is the pair (increment of digit
// a, increment of digit b).  The step loop is bound by VALU issue, and compares, selects
// and shifts take the same issue slot as an FMA (4.2 - 4.9 cycles per wave instruction and
// SIMD) while adds and logic issue beside one (2.6): two compares, two selects and a
// multiplication by 6 per step were 20 of its 112 cycles (inertial Poisson, FP32).  The
// pair costs a multiply and a mask, once per two steps.  2^20 paths x 4000 steps: 3.10 ->
// 2.81 ms (inertial Poisson), 2.84 -> 2.64 ms (overdamped dichotomous).
template <typename R> struct alignas(2 * sizeof(R)) Pair { R a, b; };
template <typename R, int NOISE> constexpr uint32_t digit_bytes()
{
    return (NOISE & NZ_GAUSS) != 0 ? 36u * (uint32_t)sizeof(Pair<R>) : 0u;
}
// LDS bytes a work-group of `waves` waves needs for its tables (behind the rings).
template <typename R, int NOISE> __host__ __device__ constexpr uint32_t table_lds(uint32_t waves)
{
    return digit_bytes<R, NOISE>() * waves;
}

template <typename R> __device__ __forceinline__ R digit_increment(uint32_t digit, R g3)
{
    return digit == 0u ? -g3 : (digit == 1u ? g3 : R(0));
}

// Increments of the two leading base-6 digits of u, from the table at LDS offset `tab`
// (a multiple of the entry size S): floor(36 u / 2^32) S = floor(36 S u / 2^32) with the
// low bits cleared, so one multiply and one mask give the address.
template <typename R> __device__ __forceinline__ Pair<R> digit_pair(uint32_t tab, uint32_t u)
{
    constexpr uint32_t S = (uint32_t)sizeof(Pair<R>);
    const uint32_t off = (uint32_t)(((uint64_t)u * (36u * S) + ((uint64_t)tab << 32)) >> 32) & ~(S - 1u);
    return lds_at<Pair<R>>(off);
}

// LDS bytes of the rings per lane and path.
template <typename R, int NOISE> __host__ __device__ constexpr uint32_t ring_bytes(RingSizes n)
{
    return (queued_kicks<NOISE>() ? (uint32_t)sizeof(KickEntry<R>) << n.log2 : 0u) +
           (((NOISE & NZ_JGRID) != 0) ? n.jg * (uint32_t)sizeof(JGKick<R>) : 0u) +
           (((NOISE & NZ_DICH) != 0) ? 4u << n.log2 : 0u);
}
// Sizes that fit: the busy ones while a work-group of `lanes` paths stays within 60 KiB.
template <typename R, int NOISE> __host__ constexpr RingSizes ring_fit(uint32_t busy, uint32_t lanes)
{
    const RingSizes n = ring_sizes<R, NOISE>(busy);
    return ring_bytes<R, NOISE>(n) * lanes <= 61440u ? n : ring_sizes<R, NOISE>(0);
}

// The smallest of the lanes' values, the same in every lane: kept scalar, so that step
// numbers and forcing-table reads stay wave-uniform.
__device__ __forceinline__ uint32_t wave_min(uint32_t v)
{
    auto take = [&](auto ctrl, auto rows) {      // lanes without a source keep their value
        const uint32_t o = (uint32_t)__builtin_amdgcn_update_dpp(-1, (int)v, decltype(ctrl)::value,
                                                                 decltype(rows)::value, 0xF, false);
        v = o < v ? o : v;
    };
    using std::integral_constant;
    take(integral_constant<int, 0x111>{}, integral_constant<int, 0xF>{});      // row_shr 1, 2, 4, 8
    take(integral_constant<int, 0x112>{}, integral_constant<int, 0xF>{});
    take(integral_constant<int, 0x114>{}, integral_constant<int, 0xF>{});
    take(integral_constant<int, 0x118>{}, integral_constant<int, 0xF>{});
    take(integral_constant<int, 0x142>{}, integral_constant<int, 0xA>{});      // last lanes of rows 0, 2
    take(integral_constant<int, 0x143>{}, integral_constant<int, 0xC>{});      // of the lower half
    return (uint32_t)__builtin_amdgcn_readlane((int)v, 63);
}

// ---------------------------------------------------------------------------
// The integration loop: advances PPL paths per lane over steps [n0, n1) in
// blocks of 16 steps (aligned to multiples of 16) sharing one Philox call for
// Algorithm 2 (4 words x 4 base-6 digits; the normal increments of the
// non-simplified scheme take one call per 4 steps) and 17 loads of the
// forcing table; x is folded after every step whose index is a multiple of 16.
// Where the rings do not cover the next block they are filled until they do, and the blocks
// they then cover run without another look; a lane whose full ring does not cover a block
// cuts it short for the wave, and the steps it does cover run one by one, as do the ends of a
// call that are no whole block.
// LDS holds the rings, slot-major with the lanes' columns side by side, and behind them the
// waves' increment tables.  A block ends at a.n_window as well, and snap() runs after that
// step: one launch crosses the start of eq. (31)'s averaging.
// ---------------------------------------------------------------------------
template <typename R, int DYN, int POT, int NOISE, int PPL, typename Snap>
__device__ __forceinline__ void advance_range(const PointConst &a, const uint32_t (&path)[PPL],
                                              Path<R> (&s)[PPL], uint64_t n0, uint64_t n1,
                                              uint32_t qs, uint32_t col0, Snap snap)
{
    constexpr bool KICKS = queued_kicks<NOISE>(), JG = (NOISE & NZ_JGRID) != 0, FLIPS = (NOISE & NZ_DICH) != 0;
    constexpr bool JUMPS = KICKS || JG || FLIPS;
    const uint32_t slots = 1u << a.rings.log2;
    Ring kr{0u, qs * (uint32_t)sizeof(KickEntry<R>), slots * qs * (uint32_t)sizeof(KickEntry<R>)};
    Ring gr{0u, qs * (uint32_t)sizeof(JGKick<R>), a.rings.jg * qs * (uint32_t)sizeof(JGKick<R>)};
    Ring fr{KICKS ? kr.total : (JG ? gr.total : 0u), qs * 4u, slots * qs * 4u};
    const uint32_t dtab = fr.base + (FLIPS ? fr.total : 0u) +
                          digit_bytes<R, NOISE>() * (uint32_t)__builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    if constexpr ((NOISE & NZ_GAUSS) != 0) {
        const uint32_t e = threadIdx.x & 63u;
        if (e < 36u)
            lds_at<Pair<R>>(dtab + e * (uint32_t)sizeof(Pair<R>)) =
                Pair<R>{digit_increment<R>(e / 6u, (R)a.g3), digit_increment<R>(e % 6u, (R)a.g3)};
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
    }
    JumpCursor<R> J[PPL];
    const R h = (R)a.dt, hh = (R)(0.5 * a.dt), ngam = (R)(-a.gamma), g3 = (R)a.g3;
    const R kp = pot_factor<POT, R>();
    const R Fa = (R)a.Fa, Fb = (R)a.Fb;
    const uint32_t wave_cols = qs / PPL;

    uint64_t n = n0;
    uint32_t k = (uint32_t)(n % a.spp);           // drive phase of step n
    const uint32_t k16 = 16u % a.spp;             // its advance in a block
#pragma unroll
    for (int j = 0; j < PPL; ++j) {               // empty rings: the next jump is the first not drawn
        const uint32_t col = (uint32_t)j * wave_cols + col0;
        if constexpr (KICKS) {
            J[j].cP = J[j].tP = col * (uint32_t)sizeof(KickEntry<R>);
            J[j].nP = J[j].uP = (uint32_t)n0 + (uint32_t)s[j].sP;
            J[j].zP = R(0);
        }
        if constexpr (JG) {
            J[j].cG = J[j].tG = col * (uint32_t)sizeof(JGKick<R>);
            J[j].poff = (uint32_t)n0 + (uint32_t)s[j].sP;
            J[j].pth = s[j].thP;
            J[j].g = JGKick<R>{J[j].poff, R(0), R(0), R(0)};
        }
        if constexpr (FLIPS) {
            J[j].cD = J[j].tD = col * 4u;
            J[j].nD = J[j].uD = (uint32_t)n0 + (uint32_t)s[j].sD;
            J[j].dT = s[j].d;
            J[j].lev = s[j].d ? Fb : -Fa;
        }
    }
    // Dichotomous noise alone: the wave looks four steps ahead and runs them without a test
    // when none of its lanes flips in them (70% of the time at 1.4e-3 flips per step), and
    // a step without flips skips the flip's instructions.  Tested and selected step by
    // step, flips cost every step about 10 of 96 cycles (2^20 paths x 4000 steps: 2.65 ->
    // 2.39 ms).  Poisson kicks come often enough (0.016 per step: some lane of the wave
    // kicks in 98% of all four steps) that looking ahead only costs (2.81 -> 2.83 ms).
    constexpr bool AHEAD = FLIPS && (NOISE & NZ_POISSON) == 0;
    const bool busy = a.rings.log2 > 3u;          // some lane flips in most fours
    uint32_t safe = (uint32_t)n0;                 // the jumps before this step are queued, in every lane

    while (n < n1) {
        const uint64_t stop = n < a.n_window && a.n_window < n1 ? a.n_window : n1;
        const uint32_t n32 = (uint32_t)n;
        uint32_t run = 16u - (n32 & 15u);
        if (stop - n < run) run = (uint32_t)(stop - n);
        // A lane whose step holds more kicks than its ring (jump-adapted grid only): that
        // one step runs alone, drawing the kicks past the ring at the step.
        bool single = false;
        if constexpr (JUMPS) {
            auto cover = [&] {                    // steps from n whose jumps are all queued
                uint32_t c = 0xFFFFFFFFu;
#pragma unroll
                for (int j = 0; j < PPL; ++j) {
                    if constexpr (KICKS) c = J[j].uP - n32 < c ? J[j].uP - n32 : c;
                    if constexpr (JG) c = J[j].poff - n32 < c ? J[j].poff - n32 : c;
                    if constexpr (FLIPS) c = J[j].uD - n32 < c ? J[j].uD - n32 : c;
                }
                return c;
            };
            if (safe - n32 < run) {
                // steps left in the call; at most 2^30, so that the jump after the last one
                // drawn (a countdown is below 2^31) lies less than 2^32 steps ahead
                const uint32_t left = n1 - n < 0x40000000u ? (uint32_t)(n1 - n) : 0x40000000u;
                bool more;
                do {
                    more = false;
#pragma unroll
                    for (int j = 0; j < PPL; ++j) {
                        if constexpr (KICKS) more |= draw_kicks<R>(a, path[j], n32, run, left, s[j].kP, J[j], kr);
                        if constexpr (JG) more |= draw_jg<R, NOISE>(a, path[j], n32, run, left, s[j].kP, J[j], gr);
                        if constexpr (FLIPS) more |= draw_flips<R>(a, path[j], n32, run, left, s[j].mD, J[j], fr);
                    }
                } while (__builtin_amdgcn_ballot_w64(more) != 0);
                // full rings cut the block short (on the fixed grid not to nothing: the
                // queued jumps of one lane are at different steps)
                const uint32_t c = wave_min(cover());
                run = c < run ? c : run;
                if constexpr (JG) {
                    single = run == 0u;
                    run = single ? 1u : run;
                }
                safe = n32 + (c > run ? c : run);
#pragma unroll
                for (int j = 0; j < PPL; ++j) {   // sentinels, and the current entries again
                    if constexpr (KICKS) {
                        lds_at<KickEntry<R>>(J[j].tP) = KickEntry<R>::make(J[j].uP, R(0));
                        const KickEntry<R> e = lds_at<KickEntry<R>>(J[j].cP);
                        J[j].nP = e.off;
                        J[j].zP = e.amplitude();
                    }
                    if constexpr (JG) {
                        lds_at<JGKick<R>>(J[j].tG) = JGKick<R>{J[j].poff, R(0), R(0), R(0)};
                        J[j].g = lds_at<JGKick<R>>(J[j].cG);
                    }
                    if constexpr (FLIPS) {
                        lds_at<uint32_t>(fr.base + J[j].tD) = J[j].uD;
                        J[j].nD = lds_at<uint32_t>(fr.base + J[j].cD);
                    }
                }
            }
        }

        // Generic single step (ends of a call, blocks cut short); INL: the single step whose
        // kicks overflow a ring.  q: the Philox block of the 16 steps n lies in, formed once per
        // run of single steps (500001 paths at 2 kicks per step: 2.07 -> 1.63 us per step).
        auto one_step = [&](auto inl, const U4 (&q)[PPL]) {
            constexpr bool INL = decltype(inl)::value;
            const R A0 = drive_at<R>(a, k);
            const R A1 = drive_at<R>(a, k + 1u);
#pragma unroll
            for (int j = 0; j < PPL; ++j) {
                R dxi = R(0);
                if constexpr ((NOISE & NZ_GAUSS) != 0) {
                    uint32_t u = pick(q[j], (uint32_t)(n >> 2) & 3u);
                    for (uint32_t t = 0; t < (uint32_t)(n & 3u); ++t) u = times6(u);
                    dxi = three_point<R>(u, g3);
                }
                if constexpr ((NOISE & NZ_NORMAL) != 0) {
                    // step n: words (2j, 2j+1) of block n/4, j = (n mod 4)/2; cos even, sin odd
                    const U4 qn = philox4x32_10((uint32_t)(n >> 2), path[j], a.point, TAG_GAUSS,
                                               a.key0, a.key1);
                    const bool hi = ((n >> 1) & 1u) != 0;
                    R zc, zs;
                    normal_pair(hi ? qn.z : qn.x, hi ? qn.w : qn.y, zc, zs);
                    dxi = g3 * ((n & 1u) ? zs : zc);
                }
                full_step<R, DYN, POT, NOISE, INL>(a, path[j], s[j], J[j], kr, gr, fr, (uint32_t)n, k, dxi, h, hh,
                                                   ngam, kp, A0, A1, Fa, Fb);
            }
            k = (k + 1u == a.spp) ? 0u : k + 1u;
            ++n;
            if ((n & 15u) == 0u) {                   // fold at absolute multiples of 16 steps
#pragma unroll
                for (int j = 0; j < PPL; ++j) fold<POT, R>(s[j]);
            }
        };

        if (run < 16u) {
            U4 q[PPL] = {};
#pragma unroll
            for (int j = 0; j < PPL; ++j)
                if constexpr ((NOISE & NZ_GAUSS) != 0)
                    q[j] = philox4x32_10((uint32_t)(n >> 4), path[j], a.point, TAG_GAUSS, a.key0, a.key1);
            if (single) {
                if constexpr (JG) one_step(std::true_type{}, q);
            } else {
                for (uint32_t t = 0; t < run; ++t) one_step(std::false_type{}, q);
            }
        } else {
            // whole blocks to the next refill or stop, without another look
            uint32_t blocks = 0;
            if constexpr (JUMPS) {
                blocks = (stop - n < 0x40000000u ? (uint32_t)(stop - n) : 0x40000000u) >> 4;
                blocks = (safe - n32) >> 4 < blocks ? (safe - n32) >> 4 : blocks;
            }
            do {
                uint32_t off = (uint32_t)n;
                U4 q[PPL];
#pragma unroll
                for (int j = 0; j < PPL; ++j) {
                    if constexpr ((NOISE & NZ_GAUSS) != 0)
                        q[j] = philox4x32_10((uint32_t)(n >> 4), path[j], a.point, TAG_GAUSS, a.key0, a.key1);
                    else
                        q[j] = U4{0u, 0u, 0u, 0u};
                }
                R A[17];                                  // forcing at steps n .. n+16
                const R *arow = reinterpret_cast<const R *>(a.tab) + k;   // k + 16 < spp + 16
#pragma unroll
                for (int t = 0; t < 17; ++t) A[t] = arow[t];
#pragma unroll
                for (int wd = 0; wd < 4; ++wd) {
                    R zn[PPL][4];                         // normal increments of steps 4 wd .. 4 wd + 3
                    if constexpr ((NOISE & NZ_NORMAL) != 0) {
#pragma unroll
                        for (int j = 0; j < PPL; ++j) {
                            const U4 qn = philox4x32_10((uint32_t)(n >> 2) + (uint32_t)wd, path[j], a.point,
                                                        TAG_GAUSS, a.key0, a.key1);
                            normal_pair(qn.x, qn.y, zn[j][0], zn[j][1]);
                            normal_pair(qn.z, qn.w, zn[j][2], zn[j][3]);
                        }
                    }
                    R dx[PPL][4];                         // three-point increments of the same steps
                    if constexpr ((NOISE & NZ_GAUSS) != 0) {
#pragma unroll
                        for (int j = 0; j < PPL; ++j) {
                            const uint32_t u = pick(q[j], (uint32_t)wd);
                            const Pair<R> p0 = digit_pair<R>(dtab, u);
                            const Pair<R> p1 = digit_pair<R>(dtab, 36u * u);
                            dx[j][0] = p0.a;
                            dx[j][1] = p0.b;
                            dx[j][2] = p1.a;
                            dx[j][3] = p1.b;
                        }
                    }
                    auto four = [&](auto quiet) {
#pragma unroll
                        for (int dg = 0; dg < 4; ++dg) {
                            const R A0 = A[4 * wd + dg], A1 = A[4 * wd + dg + 1];
#pragma unroll
                            for (int j = 0; j < PPL; ++j) {
                                R dxi = R(0);
                                if constexpr ((NOISE & NZ_GAUSS) != 0) dxi = dx[j][dg];
                                if constexpr ((NOISE & NZ_NORMAL) != 0) dxi = g3 * zn[j][dg];
                                full_step<R, DYN, POT, NOISE, false, decltype(quiet)::value>(
                                    a, path[j], s[j], J[j], kr, gr, fr, off + (uint32_t)dg,
                                    k + (uint32_t)(4 * wd + dg), dxi, h, hh, ngam, kp, A0, A1, Fa, Fb);
                            }
                        }
                    };
                    if constexpr (AHEAD) {
                        bool jump = false;               // within these four steps
#pragma unroll
                        for (int j = 0; j < PPL; ++j) jump = jump || J[j].nD - off < 4u;
                        if (busy || __builtin_amdgcn_ballot_w64(jump) != 0) four(std::false_type{});
                        else four(std::true_type{});
                    } else {
                        four(std::bool_constant<!JUMPS>{});
                    }
                    off += 4u;
                }
                n += 16u;
                k += k16;
                k = k >= a.spp ? k - a.spp : k;
                // without this line the compiler mixes the next block's draws of the normals into
                // this one's end (2^20 paths: 1030 against 1000 ns per step)
                if constexpr ((NOISE & NZ_NORMAL) != 0) __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                for (int j = 0; j < PPL; ++j) fold<POT, R>(s[j]);   // x mod L at the block end
            } while (JUMPS ? --blocks != 0u : n + 16u <= stop);
        }
        if (n == a.n_window) snap();
    }
    // Countdowns at the end: the next jump is the first one not drawn.
#pragma unroll
    for (int j = 0; j < PPL; ++j) {
        if constexpr (KICKS) {
            s[j].sP = (int32_t)(J[j].uP - (uint32_t)n);
        }
        if constexpr (JG) {
            s[j].sP = (int32_t)(J[j].poff - (uint32_t)n);
            s[j].thP = J[j].pth;
        }
        if constexpr (FLIPS) {
            s[j].sD = (int32_t)(J[j].uD - (uint32_t)n);
        }
    }
}

// Ensemble integration kernel: lane layout path = (blockIdx.x * PPL + j) * blockDim.x + tid.
template <typename R, int DYN, int POT, int NOISE, int PPL>
__global__ void __launch_bounds__(512) k_advance(const KArgs a)
{
    use_dynamic_lds();
    const uint64_t base = (uint64_t)blockIdx.x * PPL * blockDim.x + threadIdx.x;
    if ((base & ~(uint64_t)63) >= a.p.n_paths) return;     // the whole wave
    uint32_t path[PPL];
    bool valid[PPL];
    Path<R> s[PPL];
#pragma unroll
    for (int j = 0; j < PPL; ++j) {
        // lanes past the end shadow the last path: the wave's tables and votes take every lane
        const uint64_t p = base + (uint64_t)j * blockDim.x;
        valid[j] = p < a.p.n_paths;
        path[j] = valid[j] ? (uint32_t)p : a.p.n_paths - 1u;
        load_path<R, POT, NOISE>(a, path[j], s[j]);
    }
    advance_range<R, DYN, POT, NOISE, PPL>(a.p, path, s, a.n0, a.n1, PPL * blockDim.x, threadIdx.x, [&] {
#pragma unroll
        for (int j = 0; j < PPL; ++j)
            if (valid[j]) { arr<R>(a.xi)[path[j]] = s[j].x; a.wi[path[j]] = s[j].w; }
    });
#pragma unroll
    for (int j = 0; j < PPL; ++j)
        if (valid[j]) store_path<R, POT, NOISE>(a, path[j], s[j]);
}

// ---------------------------------------------------------------------------
// Initial conditions (tag 2), computed in FP64 and stored in the path precision:
// x ~ U[x0_lo, x0_hi) folded, v ~ U[v0_lo, v0_hi), Poisson countdown
// floor(E / (lambda dt)), dichotomous state opposite to a stationary draw with
// countdown 0 (the first step flips into the stationary state).  The first work-group
// also stores the first tab_words words of the forcing table.
// ---------------------------------------------------------------------------
template <typename R, int DYN, int POT, int NOISE>
__device__ __forceinline__ Path<R> init_path(const PointConst &a, uint32_t p)
{
    const U4 q = philox4x32_10(0u, p, a.point, TAG_INIT, a.key0, a.key1);
    const double L = period<POT>();
    double x = a.x0_lo + a.x0_w * ((double)q.x * 0x1p-32);
    const double kf = floor(x / L);
    x = x - kf * L;
    Path<R> s;
    s.w = (int32_t)kf;
    s.x = (R)x;
    if (s.x >= (R)L) { s.x -= (R)L; s.w += 1; }   // rounding to the path precision may reach L
    s.v = (DYN == DYN_INERTIAL) ? (R)(a.v0_lo + a.v0_w * ((double)q.y * 0x1p-32)) : R(0);
    s.sP = 0; s.kP = 0u; s.sD = 0; s.mD = 0u; s.d = 0; s.thP = 0.0;
    if constexpr ((NOISE & NZ_JGRID) != 0) {
        const double T = expo64(q.z) / a.lam_dt;          // first kick time in steps
        const double Tf = floor(T);
        s.sP = (int32_t)Tf;
        s.thP = T - Tf;
    } else if constexpr ((NOISE & NZ_POISSON) != 0) {
        s.sP = (int32_t)floor(expo64(q.z) / a.lam_dt);
    }
    if constexpr ((NOISE & NZ_DICH) != 0) {
        const int32_t dstar = ((double)q.w * 0x1p-32 < a.p_hi) ? 1 : 0;
        s.d = 1 - dstar;
    }
    return s;
}

template <typename R, int DYN, int POT, int NOISE>
__global__ void __launch_bounds__(256) k_init(const KArgs a, const TableChunk tab, uint32_t tab_words)
{
    if (blockIdx.x == 0) store_chunk(tab, tab_words, (uint32_t *)const_cast<void *>(a.p.tab));
    const uint64_t p64 = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (p64 >= a.p.n_paths) return;
    const uint32_t p = (uint32_t)p64;
    const Path<R> s = init_path<R, DYN, POT, NOISE>(a.p, p);
    arr<R>(a.x)[p] = s.x;
    a.w[p] = s.w;
    arr<R>(a.v)[p] = s.v;
    if constexpr ((NOISE & NZ_POISSON) != 0) { a.sP[p] = s.sP; a.kP[p] = s.kP; }
    if constexpr ((NOISE & NZ_JGRID) != 0) a.thP[p] = s.thP;
    if constexpr ((NOISE & NZ_DICH) != 0) { a.d[p] = s.d; a.sD[p] = s.sD; a.mD[p] = s.mD; }
    if (a.snapshot) { arr<R>(a.xi)[p] = s.x; a.wi[p] = s.w; }
    if (a.lev) { a.lev[p] = (int32_t)a.sc_J; a.kA[p] = 0u; }   // step control starts at the smallest step
}

// ---------------------------------------------------------------------------
// eq. (31) per path in FP64, plus one double-double partial per wave (64 paths).
// Launched with 256-lane work-groups; chunk c covers paths [64c, 64c + 64).
// ---------------------------------------------------------------------------
template <typename R, int POT> __device__ __forceinline__ void velocity_of(const KArgs &a, uint64_t p)
{
    const double L = period<POT>();
    double vp = 0.0;
    bool have = p < a.p.n_paths;
    if (have) {
        const double dx = (double)(a.w[p] - a.wi[p]) * L +
                          ((double)arr<R>(a.x)[p] - (double)arr<R>(a.xi)[p]);
        vp = dx / a.t_window;
        a.vp[p] = vp;
    }
    const Partial part = wave_partial(vp, have);
    const uint64_t chunk = p >> 6;
    if ((threadIdx.x & 63u) == 0u && (chunk << 6) < a.p.n_paths) {
        a.part[chunk] = part;
    }
}

template <typename R, int POT>
__global__ void __launch_bounds__(256) k_velocity(const KArgs a)
{
    velocity_of<R, POT>(a, (uint64_t)blockIdx.x * blockDim.x + threadIdx.x);
}

// The same and the reduction of the partials in one launch of 1024 lanes, for ensembles
// where the second launch costs more than the parallelism of the first gives: at most
// REDUCE_SMALL paths, one pass.
template <typename R, int POT>
__global__ void __launch_bounds__(1024) k_velocity_reduce(const KArgs a, bm_stats *out)
{
    for (uint64_t p = threadIdx.x; (p & ~(uint64_t)63) < a.p.n_paths; p += 1024) velocity_of<R, POT>(a, p);
    __syncthreads();                             // the partials, from the same CU's memory
    reduce_chunks(a.part, ((uint64_t)a.p.n_paths + 63) / 64, a.t_window, out);
}

// ---------------------------------------------------------------------------
// Export of paths [n0, n0 + n1) (n0/n1 reused as first/count) to FP64 arrays and
// to lossless per-path records (every field widened exactly).  flags (launch.hpp):
// READ_VP the per-path velocity exists, READ_SNAP the window snapshot exists
// (before the window start the record's window fields are 0, not the workspace's
// unwritten contents).
// ---------------------------------------------------------------------------

template <typename R, int POT>
__global__ void __launch_bounds__(256) k_read(const KArgs a, double *xo, double *vo, int64_t *no,
                                              double *vpo, int flags, bm_path *so)
{
    const uint64_t i = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= a.n1) return;
    const uint64_t p = a.n0 + i;
    const double L = period<POT>();
    if (xo) xo[i] = (double)a.w[p] * L + (double)arr<R>(a.x)[p];
    if (vo) vo[i] = (double)arr<R>(a.v)[p];
    const int64_t nz[5] = {a.sP ? a.sP[p] : 0, a.kP ? (int64_t)a.kP[p] : 0, a.sD ? a.sD[p] : 0,
                           a.mD ? (int64_t)a.mD[p] : 0, a.d ? a.d[p] : 0};
    if (no) {
        for (int j = 0; j < 5; ++j) no[5 * i + j] = nz[j];
    }
    if (vpo && (flags & READ_VP)) {
        const double dx = (double)(a.w[p] - a.wi[p]) * L +
                          ((double)arr<R>(a.x)[p] - (double)arr<R>(a.xi)[p]);
        vpo[i] = dx / a.t_window;
    }
    if (so) {
        bm_path r;
        r.periods = a.w[p];
        r.x = (double)arr<R>(a.x)[p];
        r.v = (double)arr<R>(a.v)[p];
        const bool snap = (flags & READ_SNAP) != 0;
        r.periods_window = snap ? a.wi[p] : 0;
        r.x_window = snap ? (double)arr<R>(a.xi)[p] : 0.0;
        r.kick_frac = a.thP ? a.thP[p] : 0.0;
        for (int j = 0; j < 5; ++j) r.noise[j] = nz[j];
        r.step_level = a.lev ? a.lev[p] : 0;
        r.steps_taken = a.kA ? (int64_t)a.kA[p] : 0;
        so[i] = r;
    }
}

// ---------------------------------------------------------------------------
// Import of records into paths [n0, n0 + n1): the inverse of k_read's records.
// Out-of-range values are clamped so that the path kernels' assumptions (countdowns
// and counts in range, state 0/1, a kick fraction in [0, 1)) hold whatever the input.
// snap: 0 leave the window snapshot, 1 set it to the written position, 2 take it
// from the record.
// ---------------------------------------------------------------------------
__device__ __forceinline__ int32_t clamp_i32(int64_t v, int64_t lo, int64_t hi)
{
    return (int32_t)(v < lo ? lo : (v > hi ? hi : v));
}

template <typename R, int POT>
__global__ void __launch_bounds__(256) k_write(const KArgs a, const bm_path *si, uint32_t snap)
{
    const uint64_t i = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= a.n1) return;
    const uint64_t p = a.n0 + i;
    const bm_path r = si[i];
    const int32_t w = clamp_i32(r.periods, INT32_MIN, INT32_MAX);
    arr<R>(a.x)[p] = (R)r.x;
    a.w[p] = w;
    arr<R>(a.v)[p] = (R)r.v;
    if (snap == 1u) {
        arr<R>(a.xi)[p] = (R)r.x;
        a.wi[p] = w;
    } else if (snap == 2u) {
        arr<R>(a.xi)[p] = (R)r.x_window;
        a.wi[p] = clamp_i32(r.periods_window, INT32_MIN, INT32_MAX);
    }
    if (a.sP) a.sP[p] = clamp_i32(r.noise[0], 0, INT32_MAX);
    if (a.kP) a.kP[p] = (uint32_t)(r.noise[1] < 0 ? 0 : (r.noise[1] > (int64_t)UINT32_MAX ? UINT32_MAX : r.noise[1]));
    if (a.thP) a.thP[p] = (r.kick_frac >= 0.0 && r.kick_frac < 1.0) ? r.kick_frac : 0.0;
    if (a.sD) a.sD[p] = clamp_i32(r.noise[2], 0, INT32_MAX);
    if (a.mD) a.mD[p] = (uint32_t)(r.noise[3] < 0 ? 0 : (r.noise[3] > (int64_t)UINT32_MAX ? UINT32_MAX : r.noise[3]));
    if (a.d) a.d[p] = r.noise[4] != 0 ? 1 : 0;
    if (a.lev) {
        a.lev[p] = clamp_i32(r.step_level, 0, (int64_t)a.sc_J);
        a.kA[p] = (uint32_t)(r.steps_taken < 0 ? 0 : (r.steps_taken > (int64_t)UINT32_MAX ? UINT32_MAX : r.steps_taken));
    }
}

// ---------------------------------------------------------------------------
// eq. (19): histogram of the folded positions y = x mod L in n_bins equal bins of
// [0, L), bin = floor(y n_bins / L), computed in FP64; counts are added to `hist`
// (integer atomics: the result does not depend on their order).
// ---------------------------------------------------------------------------
template <typename R, int POT>
__global__ void __launch_bounds__(256) k_density(const KArgs a, uint32_t n_bins, unsigned long long *hist)
{
    const uint64_t p = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (p >= a.p.n_paths) return;
    const double L = period<POT>();
    const double x = (double)arr<R>(a.x)[p];
    const double y = x - L * floor(x / L);
    const double t = y * (double)n_bins / L;
    uint32_t b = t >= (double)n_bins ? n_bins - 1u : (uint32_t)t;   // y rounded up to L
    if (!(t >= 0.0)) return;                                          // non-finite position
    atomicAdd(&hist[b], 1ull);
}

} // namespace bm
