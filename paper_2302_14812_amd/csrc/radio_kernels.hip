// HIP kernels of libradio for gfx950 (MI355X).
//
// The deposit evaluates, for every (particle, segment, cell) triple, the
// Lienard-Wiechert field (Eq. 1) of the segment's current state and the
// arrival times of its two end states (Eq. 2), and adds the field held
// between those arrival times to the detector slots with the integrator
// weights of Sec. 3.2 / Alg. 2.  Four kernels run per deposit:
//
// 1. kinematics_kernel (Alg. 1, velocity and acceleration lines): one thread
//    per trajectory state turns (x, u) into a record with x, beta, betadot and
//    1/gamma^2 (80 bytes; 64 for the mixed modes, with (q/c) betadot and
//    1/(2 gamma^2) in single precision),
//    laid out particle-major so that the states of one particle's run are
//    contiguous.
//
// 2. order_kernel: for every tile of kTileCells detector cells, a counting
//    sort of the particles by their light-travel time to the tile's centre at
//    the chunk's middle state.  Processing particles in that order makes the
//    arrival slots a tile's cells see advance nearly monotonically.
//
// 3. ring_choice_kernel: per tile, whether the arrivals a batch touches fit
//    the small LDS ring (slow advance, many segments per slot) or need the
//    large one (a slot crossed every segment or two), with its runs staged whole
//    or in shorter stretches; it samples batches.  Where a second launch for a part
//    of the tiles would cost more than it gains, all tiles take one ring.
//
// 4. deposit_kernel: one workgroup per (tile, range of runs), launched once
//    per ring size; tiles of the other size leave at once.  Lane
//    (cell, group) = (lane % kTileCells, lane / kTileCells): the kTileCells
//    cells of the tile each get kGroups lanes, and the lanes of one group walk
//    the same particle.  Trajectories are cut into runs of kRunL segments; a
//    batch of kGroups particles (consecutive in the tile's order) x
//    (kRunL + 1) states is staged in LDS and each lane walks its particle's
//    run against its cell.  The lane integrates the held field over its
//    current slot with the exact slot-unit overlaps of Alg. 2 and emits
//    a slot's value only when its arrivals move on; emissions go to a
//    per-cell ring of slots in LDS that slides forward as the sorted batches
//    advance, and only slots leaving the ring (or emissions that fall outside
//    it) reach the detector in HBM, through atomic adds.
//
// A chunk of a few particles takes few_kernel alone.
//
// Slot accumulator.  The detector holds, per cell and slot, the sum over
// segments of the held E and B times the segment's overlap with the slot in
// units of dt_det (Alg. 2): the slot's time average, read out as it is.  All
// updates are additive, so the ring, its fallback and the order of the
// particles only change rounding.
#include "radio_internal.h"

#include <algorithm>

#include <atomic>
#include <climits>
#include <type_traits>
#include <utility>

namespace radio {

namespace {

// pointers into LDS keep their address space, so ring updates compile to ds_*
// instructions rather than generic (flat) ones
#define RADIO_LDS __attribute__((address_space(3)))
// likewise for device memory reached through pointers that were loaded from
// memory (the job descriptors of the persistent kernel)
#define RADIO_GLOBAL __attribute__((address_space(1)))

typedef long long v2i64 __attribute__((ext_vector_type(2)));  // a 16-byte piece

template <typename P>
__device__ __forceinline__ RADIO_GLOBAL P* gptr(P* p)
{
    return (RADIO_GLOBAL P*)p;
}

// ---------------------------------------------------------------------------
// Quantities that cancel catastrophically.  Both this library and any
// reference evaluation have to round them the same way, so they are
// evaluated one IEEE operation at a time, in a fixed order, without fused
// multiply-adds.  (The slot coordinate amplifies one ulp of the arrival time
// at t_det ~ 1e5 to ~1e-7 of a slot, and 1 - n.beta ~ 1/(2 gamma^2).)
// ---------------------------------------------------------------------------
__device__ __forceinline__ double canon_norm2(double a, double b, double c)
{
#pragma clang fp contract(off)
    return (a * a + b * b) + c * c;
}

// time of the run's state s (s < 2^53, an integer held exactly as a double)
__device__ __forceinline__ double canon_state_time(double t_first, double s, double dt)
{
#pragma clang fp contract(off)
    return t_first + s * dt;
}

// sqrt(x) correctly rounded for x = 0 and 2^-767 <= x < inf (every distance of
// physical size), with 1/sqrt(x) to an ulp or two beside it.  A hardware
// reciprocal square root seed (about 23 bits) is refined by one coupled
// Goldschmidt step, g ~ sqrt(x) and h ~ 1/(2 sqrt(x)), and g by two residual
// corrections g += (x - g^2) h, each rounded once -- the sequence the compiler
// emits for a correctly rounded double sqrt, without its rescaling of inputs
// below 2^-767 and its special-value checks (0 is handled here; inf and NaN do
// not occur).  The reciprocal is one Newton step on 1/g from 2h; for x = 0 it
// is NaN, as d (1/R) is when d = 0.
__device__ __forceinline__ double canon_sqrt(double x, double* rinv)
{
    const double y = __builtin_amdgcn_rsq(x);
    double g = x * y;
    double h = 0.5 * y;
    const double r = fma(-g, h, 0.5);
    g = fma(g, r, g);
    h = fma(h, r, h);
    double d = fma(-g, g, x);
    g = fma(d, h, g);
    d = fma(-g, g, x);
    g = fma(d, h, g);
    const double q = 2.0 * h;
    *rinv = fma(q, fma(-g, q, 1.0), q);
    return x == 0.0 ? 0.0 : g;
}

__device__ __forceinline__ double canon_sqrt(double x)
{
    double unused;
    return canon_sqrt(x, &unused);
}

__device__ __forceinline__ double canon_arrival(double t, double R, double inv_c)
{
#pragma clang fp contract(off)
    return t + R * inv_c;
}

// The slot coordinate (t_det - t0) / dt_det, correctly rounded, as the one IEEE
// division that defines it, without a division per state.  With the divisor b =
// dt_det, its correctly rounded reciprocal y = RN(1/b) from the host and the
// numerator x = t_det - t0:
//   q0 = RN(x y)                         within 2.5 ulp of z = x/b
//   q1 = RN(q0 + RN(x - b q0) y)         within ulp/2 + 10 u ulp   (u = 2^-53)
//   q2 = RN(q1 + (x - b q1) y)           (x - b q1 is exact here)
// Two corrections in the manner of Markstein's theorem.  q1 + (x - b q1) y =
// z + (z - q1) e with e = b y - 1, and |z - q1| <= (1/2 + 10 u) ulp(z).  A
// quotient of two doubles is never a rounding midpoint, and x - b m for a
// midpoint m is a nonzero multiple of ulp(b) ulp(z)/2, so z lies at least
// ulp(z)/(2 B) from every midpoint, B being b's significand as an integer in
// [2^52, 2^53).  q2 is therefore RN(z) whenever |e| B (1 + 20 u) < 1: true for
// most divisors (|e| <= B 2^-106) and checked for each detector on the host
// (slot_div = 0).  For the divisors where it is not, the kernels divide.
// Valid for normal x and z away from overflow and underflow (|x| >= 2^-900),
// which physical arrival times are; a non-finite x gives NaN (a dropped segment).
__device__ __forceinline__ double canon_slot(double tau, double t0, double dt_det,
                                             double inv_dt_det, bool slot_div)
{
#pragma clang fp contract(off)
    const double x = tau - t0;
    if (slot_div)
        return x / dt_det;
    double q = x * inv_dt_det;
    double r = fma(-q, dt_det, x);
    q = fma(r, inv_dt_det, q);
    r = fma(-q, dt_det, x);
    return fma(r, inv_dt_det, q);
}

// n = d/R as d * (1/R) and w = n - beta
__device__ __forceinline__ void canon_direction(const double d[3], double rinv, const double b[3],
                                                double n[3], double w[3])
{
#pragma clang fp contract(off)
    n[0] = d[0] * rinv;
    n[1] = d[1] * rinv;
    n[2] = d[2] * rinv;
    w[0] = n[0] - b[0];
    w[1] = n[1] - b[1];
    w[2] = n[2] - b[2];
}

// kappa = 1 - n.beta evaluated as (|n - beta|^2 + 1/gamma^2)/2, equal for unit n and
// free of the cancellation 1 - n.beta suffers as beta -> 1
__device__ __forceinline__ double canon_kappa(const double w[3], double inv_g2)
{
#pragma clang fp contract(off)
    return 0.5 * (((w[0] * w[0] + w[1] * w[1]) + w[2] * w[2]) + inv_g2);
}

// beta = u / sqrt(|u|^2 + 1), 1/gamma^2 = 1/(|u|^2 + 1)   (Alg. 1)
__device__ __forceinline__ void canon_kinematics(double u0, double u1, double u2, double b[3],
                                                 double* inv_g2)
{
#pragma clang fp contract(off)
    double g = canon_norm2(u0, u1, u2) + 1.0;
    double sq = __builtin_sqrt(g);
    b[0] = u0 / sq;
    b[1] = u1 / sq;
    b[2] = u2 / sq;
    *inv_g2 = 1.0 / g;
}

// betadot = (beta_s - beta_{s-1}) / dt
__device__ __forceinline__ double canon_betadot(double b, double bp, double dt)
{
#pragma clang fp contract(off)
    return (b - bp) / dt;
}

// ---------------------------------------------------------------------------
// detector updates
// ---------------------------------------------------------------------------

// Where a lane's finished slot values go in HBM.  Double path: one atomic
// add per component.  Mixed path: a compensated single-precision pair (hi, lo)
// per component; the atomic add on hi returns the old value, so the lane knows
// the exact sum the hardware rounded (old + v) and adds that rounding error
// (two-sum) to lo.
__device__ __forceinline__ float two_sum_err(float a, float b, float s)
{
#pragma clang fp contract(off)
    const float bv = s - a;
    return (a - (s - bv)) + (b - bv);
}

__device__ __forceinline__ void global_add(RADIO_GLOBAL double* row, int j, const double a[6])
{
    RADIO_GLOBAL double* q = row + (int64_t)j * 6;
#pragma unroll
    for (int k = 0; k < 6; ++k)
        __hip_atomic_fetch_add(q + k, a[k], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// Compensated single-precision adds into the HBM pair (hi[6], lo[6]) of slot j:
// the six returning adds to hi are issued together, so that their round trips
// overlap, then the lo words take each add's rounding error.  A zero component
// adds exactly nothing (old + 0 is exact, its error 0), so no component is
// skipped: a branch per component would put the round trips in sequence.
__device__ __forceinline__ void global_add(RADIO_GLOBAL float* row, int j, const float a[6])
{
    RADIO_GLOBAL float* q = row + (int64_t)j * 12;
    float old[6];
#pragma unroll
    for (int k = 0; k < 6; ++k)
        old[k] = __hip_atomic_fetch_add(q + k, a[k], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
#pragma unroll
    for (int k = 0; k < 6; ++k)
        __hip_atomic_fetch_add(q + 6 + k, two_sum_err(old[k], a[k], old[k] + a[k]),
                               __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// one component k of slot j
__device__ __forceinline__ void global_add_one(RADIO_GLOBAL double* row, int j, int k, double v)
{
    __hip_atomic_fetch_add(row + (int64_t)j * 6 + k, v, __ATOMIC_RELAXED,
                           __HIP_MEMORY_SCOPE_AGENT);
}

// the same into the compensated pair: v split into hi and lo
__device__ __forceinline__ void global_add_one(RADIO_GLOBAL float* row, int j, int k, double v)
{
    RADIO_GLOBAL float* q = row + (int64_t)j * 12 + k;
    const float hi = (float)v;
    const float lo = (float)(v - (double)hi);
    const float old =
        __hip_atomic_fetch_add(q, hi, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    __hip_atomic_fetch_add(q + 6, two_sum_err(old, hi, old + hi) + lo, __ATOMIC_RELAXED,
                           __HIP_MEMORY_SCOPE_AGENT);
}

// position of slot j >= 0 in a ring of R slots
template <int R>
__device__ __forceinline__ int ring_pos(int j)
{
    if constexpr ((R & (R - 1)) == 0)
        return j & (R - 1);
    else
        return (int)((unsigned)j % (unsigned)R);
}

// One cell's ring of slots in LDS, covering slots [base, base + R); slot j lives
// at position j mod R.  Emissions inside go to the ring (LDS atomic add: the
// kGroups lanes of a cell share it), anything else straight to HBM.  The ring
// holds 6 doubles per slot in every mode; the emission (double or single) is
// widened and added.  Acc is the element of the HBM accumulator: double, or
// for compensated single accumulation (Acc = float) the pair hi[6], lo[6] per
// slot, which a slot leaving the ring reaches as the double split into hi and
// lo, and a bypassing emission as itself (two-sum into the pair).
// The rings of a tile's TC cells lie in LDS as [slot][component][cell]: an
// instruction's lanes hold 16 different cells, which then never share a bank,
// whatever slots they are in (with a cell's slots together and a padded stride a
// plasma-mirror sheet of 1e5 electrons x 16 steps x 128 x 128 cells took 248 ms
// instead of 218, the undulator ensemble 107 instead of 102).
// A ring holds slot values, each the sum of what its own segments deposit.  A ring of
// the held field's jumps, summed along the slots when they leave it, is 8% faster on
// that sheet (177 against 192 ms), but a slot then carries the rounding of every field
// summed before it: slots beside one of 1e16 times their field were 10% off.
template <typename Acc, int R, int TC>
struct CellSink {
    static constexpr int W = 6;  // values per ring slot
    RADIO_LDS double* ring;
    RADIO_GLOBAL Acc* row;  // double, or hi[6], lo[6] per slot
    int base;
    int n_t;
    unsigned* n_bypass;
    // The ring covers [base, base + R) with 0 <= base, so a slot in it is >= 0;
    // slots at or past n_t that it holds (n_t < R) are dropped when it moves.
    template <typename F>
    __device__ __forceinline__ void flush(int j, const F a[6]) const
    {
        if ((unsigned)(j - base) < (unsigned)R) {
            RADIO_LDS double* q = ring + ring_pos<R>(j) * (W * TC);
#pragma unroll
            for (int k = 0; k < 6; ++k)
                __hip_atomic_fetch_add(q + k * TC, (double)a[k], __ATOMIC_RELAXED,
                                       __HIP_MEMORY_SCOPE_WORKGROUP);
        } else if ((unsigned)j < (unsigned)n_t) {
            *n_bypass += 1u;
            Acc v[6];
#pragma unroll
            for (int k = 0; k < 6; ++k)
                v[k] = (Acc)a[k];
            global_add(row, j, v);
        }
    }
};

// ---------------------------------------------------------------------------
// the lane's open slot
// ---------------------------------------------------------------------------

// For the run being processed the lane integrates the held field over its
// current slot J (V); when the run leaves slot J, V is final and is emitted.
// Every overlap is the exact slot-unit overlap of the integrator definition
// (Alg. 2), so each segment contributes the same numbers the definition
// gives; only the order of the additions differs.  Slots outside [0, n_t)
// are dropped by the sink, which is how the window clips (Alg. 1).
//
// The carry keeps J + 1 as a double (J1) and the bound `lim` of the fast path:
// a segment [a, b] with a <= b < lim starts in the open slot (a in [J, J+1)),
// with J >= 0, and ends below n_t, so it lies inside the window.  lim is n_t
// while the next segment's start is known to lie in the open slot, inside the
// window, and -inf otherwise; such a segment takes the general path, which
// also counts the segments that reach outside [0, n_t] (clipped) and those
// that run backward.

template <typename T>
struct Carry {
    double J1;   // open slot + 1; the slot may lie outside [0, n_t), far below 0 when none is open
    double lim;  // fast-path bound of the next segment
    T V[6];      // integral of the held field over the open slot so far
};

template <typename T>
__device__ __forceinline__ void carry_open(Carry<T>& C, double J)
{
    C.J1 = J + 1.0;
#pragma unroll
    for (int k = 0; k < 6; ++k)
        C.V[k] = T(0);
}

// the fast-path bound when the open slot is J and the next segment starts at a
__device__ __forceinline__ double fast_limit(double J, double a, double ntd)
{
    return ((J >= 0.0) & (a >= J) & (a < J + 1.0)) ? ntd : -INFINITY;
}

// a segment between a and b reaches outside the window [0, n_t] (a NaN end is
// not counted as outside)
__device__ __forceinline__ unsigned clipped(double a, double b, double ntd)
{
    return ((a < 0.0) | (b < 0.0) | (a > ntd) | (b > ntd)) ? 1u : 0u;
}

// The ends of the segment between a and b, ordered and clamped to [0, n_t].
// Compares and selects only: min/max instructions would make the compiler
// quiet the operands of every state, general path taken or not.  A NaN end
// gives a NaN bound, which the callers' lo < hi test treats as empty.
__device__ __forceinline__ void clamp_segment(double a, double b, double ntd, double& lo,
                                              double& hi)
{
    const bool back = b < a;
    const double mn = back ? b : a, mx = back ? a : b;
    lo = mn < 0.0 ? 0.0 : (mn > ntd ? ntd : mn);
    hi = mx < 0.0 ? 0.0 : (mx > ntd ? ntd : mx);
}

// General case: hold F over the slot-coordinate interval between a and b,
// clipped to [0, n_t]; any order, any length.  A segment that does not start
// in the open slot closes it first, which is exact because deposits add.
// Backward segments are counted here (the fast path takes none).
template <typename T, typename Sink>
__device__ __forceinline__ void add_segment_general(Carry<T>& C, const Sink& sink, int n_t,
                                                    double a, double b, const T F[6],
                                                    unsigned& n_back, unsigned& n_clip)
{
    const double ntd = (double)n_t;
    n_back += (b < a) ? 1u : 0u;
    n_clip += clipped(a, b, ntd);
    double lo, hi;
    clamp_segment(a, b, ntd, lo, hi);
    if (lo < hi) {  // else empty, entirely outside, or NaN
        const double fl = floor(lo);  // < n_t
        const double fh = floor(hi);  // <= n_t; n_t only when hi reaches the end
        if (fl != C.J1 - 1.0) {
            sink.flush((int)(C.J1 - 1.0), C.V);
            carry_open(C, fl);
        }
        if (fh == fl) {
            const T w = T(hi - lo);
#pragma unroll
            for (int k = 0; k < 6; ++k)
                C.V[k] += F[k] * w;
        } else {
            const T wa = T((fl + 1.0) - lo);
#pragma unroll
            for (int k = 0; k < 6; ++k)
                C.V[k] += F[k] * wa;
            const int jl = (int)fl, jh = (int)fh;
            sink.flush(jl, C.V);
            for (int j = jl + 1; j < jh; ++j)  // whole slots hold F
                sink.flush(j, F);
            const T wb = T(hi - fh);
#pragma unroll
            for (int k = 0; k < 6; ++k)
                C.V[k] = F[k] * wb;
            C.J1 = fh + 1.0;
        }
    }
    C.lim = fast_limit(C.J1 - 1.0, b, ntd);
}

// One segment [a, b] of a lane's run.  Fast path (a <= b < lim): the overlaps
// are b - a (same slot) or J + 1 - a, whole slots, and b - floor(b) -- those
// of the definition -- and the emissions are guarded by the crossing count
// only.  Everything else goes through add_segment_general.
template <typename T, typename Sink>
__device__ __forceinline__ void add_segment(Carry<T>& C, const Sink& sink, int n_t, double a,
                                            double b, const T F[6], unsigned& n_back,
                                            unsigned& n_clip)
{
    if ((b >= a) & (b < C.lim)) {
        const bool leaves = b >= C.J1;  // the segment leaves the open slot
        const T w0 = T((leaves ? C.J1 : b) - a);
#pragma unroll
        for (int k = 0; k < 6; ++k)
            C.V[k] += F[k] * w0;
        if (leaves) {
            const double fb = floor(b);
            sink.flush((int)C.J1 - 1, C.V);
            if (fb > C.J1)  // whole slots J + 1 .. floor(b) - 1 hold F
                for (int j = (int)C.J1; j < (int)fb; ++j)
                    sink.flush(j, F);
            const T wb = T(b - fb);
#pragma unroll
            for (int k = 0; k < 6; ++k)
                C.V[k] = F[k] * wb;
            C.J1 = fb + 1.0;
        }
    } else {
        add_segment_general(C, sink, n_t, a, b, F, n_back, n_clip);
    }
}

// The linear rule: the field runs from Fa at slot coordinate a to Fb at b, and
// each slot receives its overlap with the segment times the interpolant at the
// overlap's midpoint (the exact integral of a linear function).  Same fast and
// general paths as add_segment.
template <typename T>
__device__ __forceinline__ void lerp_field(const T Fa[6], const T dF[6], T f, T out[6])
{
#pragma unroll
    for (int k = 0; k < 6; ++k)
        out[k] = Fa[k] + dF[k] * f;
}

template <typename T, typename Sink>
__device__ __forceinline__ void add_segment_linear_general(Carry<T>& C, const Sink& sink, int n_t,
                                                           double a, double b, const T Fa[6],
                                                           const T dF[6], double inv_len,
                                                           unsigned& n_back, unsigned& n_clip)
{
    const double ntd = (double)n_t;
    n_back += (b < a) ? 1u : 0u;
    n_clip += clipped(a, b, ntd);
    double lo, hi;
    clamp_segment(a, b, ntd, lo, hi);
    if (lo < hi) {
        const double fl = floor(lo);
        const double fh = floor(hi);
        if (fl != C.J1 - 1.0) {
            sink.flush((int)(C.J1 - 1.0), C.V);
            carry_open(C, fl);
        }
        T F[6];
        auto piece = [&](double p, double q) {  // the interpolant times the overlap [p, q]
            lerp_field(Fa, dF, T(0.5 * ((p - a) + (q - a)) * inv_len), F);
            const T w = T(q - p);
#pragma unroll
            for (int k = 0; k < 6; ++k)
                F[k] *= w;
        };
        if (fh == fl) {
            piece(lo, hi);
#pragma unroll
            for (int k = 0; k < 6; ++k)
                C.V[k] += F[k];
        } else {
            const int jl = (int)fl, jh = (int)fh;
            piece(lo, fl + 1.0);
#pragma unroll
            for (int k = 0; k < 6; ++k)
                C.V[k] += F[k];
            sink.flush(jl, C.V);
            for (int j = jl + 1; j < jh; ++j) {
                piece((double)j, (double)(j + 1));
                sink.flush(j, F);
            }
            piece(fh, hi);
#pragma unroll
            for (int k = 0; k < 6; ++k)
                C.V[k] = F[k];
            C.J1 = fh + 1.0;
        }
    }
    C.lim = fast_limit(C.J1 - 1.0, b, ntd);
}

template <typename T, typename Sink>
__device__ __forceinline__ void add_segment_linear(Carry<T>& C, const Sink& sink, int n_t,
                                                   double a, double b, const T Fa[6],
                                                   const T Fb[6], unsigned& n_back,
                                                   unsigned& n_clip)
{
    if (a == b) {  // no length: nothing to hold, and the carry still fits the next start
        n_clip += clipped(a, b, (double)n_t);
        return;
    }
    T dF[6];
#pragma unroll
    for (int k = 0; k < 6; ++k)
        dF[k] = Fb[k] - Fa[k];
    const double inv_len = 1.0 / (b - a);
    if ((b > a) & (b < C.lim)) {
        const double Jd = C.J1 - 1.0;
        const double e0 = b < C.J1 ? b : C.J1;
        T F[6];
        lerp_field(Fa, dF, T(0.5 * (e0 - a) * inv_len), F);
        const T w0 = T(e0 - a);
#pragma unroll
        for (int k = 0; k < 6; ++k)
            C.V[k] += F[k] * w0;
        if (b >= C.J1) {
            const double fb = floor(b);
            const int J = (int)C.J1 - 1;
            const int n = (int)(fb - C.J1) + 1;  // slots crossed
            sink.flush(J, C.V);
            for (int i = 1; i < n; ++i) {  // whole slots: the interpolant at their middle
                lerp_field(Fa, dF, T(0.5 * ((Jd + (double)i - a) + (Jd + (double)(i + 1) - a)) *
                                     inv_len),
                           F);
                sink.flush(J + i, F);
            }
            lerp_field(Fa, dF, T(0.5 * ((fb - a) + (b - a)) * inv_len), F);
            const T wb = T(b - fb);
#pragma unroll
            for (int k = 0; k < 6; ++k)
                C.V[k] = F[k] * wb;
            C.J1 = fb + 1.0;
        }
    } else {
        add_segment_linear_general(C, sink, n_t, a, b, Fa, dF, inv_len, n_back, n_clip);
    }
}

// ---------------------------------------------------------------------------
// field evaluation
// ---------------------------------------------------------------------------

struct Consts {
    double t0, inv_dt_det, inv_c;
    double kR;      // inv_c * inv_dt_det: slots per unit of distance (mixed modes)
    double dt_det;  // the slot width (the divisor of the double slot coordinate)
    bool slot_div;  // the double slot coordinate takes a division (see canon_slot)
};

__device__ __forceinline__ double canon_slot(double tau, const Consts& K)
{
    return canon_slot(tau, K.t0, K.dt_det, K.inv_dt_det, K.slot_div);
}

// E and B of Eq. 1 from the unit vector n to the cell, w = n - beta, 1/kappa,
// 1/R and the state's 1/gamma^2 and betadot, for a charge with qc = q/c and
// qv = q times the weight of the velocity term.  The acceleration term is
// regrouped with the identity n x (w x bd) = w (n.bd) - bd (n.w):
//   E = c1 w - c2 bd,  c1 = (qc n.bd + qv g2i / R) / (kappa^3 R),
//                      c2 = qc (n.w) / (kappa^3 R),
//   B = n x E.
// nwk is (n.w)/kappa.  For a unit n, n.w = 1 - n.beta = kappa and nwk = 1,
// which the single-precision field (lw_fields_mixed) takes: it is the more
// accurate value there.  The double field passes the product of its rounded n
// and w, as the cross products of Eq. 1 would use them (with kappa of order
// 1/gamma^2, the last bits of |n| shift n.w by up to ~1e-12 of itself).
template <typename T>
__device__ __forceinline__ void lw_fields(const T n[3], const T w[3], T kinv, T rinv, T g2i,
                                          const T bd[3], T qc, T qv, T nwk, T F[6])
{
    const T nbd = n[0] * bd[0] + n[1] * bd[1] + n[2] * bd[2];
    const T rk2 = rinv * (kinv * kinv);
    const T c1 = (qc * nbd + qv * g2i * rinv) * (rk2 * kinv);
    const T c2 = qc * rk2 * nwk;
    const T E0 = c1 * w[0] - c2 * bd[0];
    const T E1 = c1 * w[1] - c2 * bd[1];
    const T E2 = c1 * w[2] - c2 * bd[2];
    F[0] = E0;
    F[1] = E1;
    F[2] = E2;
    F[3] = n[1] * E2 - n[2] * E1;
    F[4] = n[2] * E0 - n[0] * E2;
    F[5] = n[0] * E1 - n[1] * E0;
}

// 1/x from the hardware reciprocal refined by two Newton steps (within an ulp
// or two; used where Eq. 1 needs no particular rounding)
__device__ __forceinline__ double recip(double x)
{
    double r = __builtin_amdgcn_rcp(x);
    double e = fma(-x, r, 1.0);
    r = fma(r, e, r);
    e = fma(-x, r, 1.0);
    return fma(r, e, r);
}

// Lienard-Wiechert E, B (Eq. 1) at a cell from one staged state, all in double;
// returns the state's slot coordinate.  Only the arrival time (R and tau) is
// rounded canonically; n, w, kappa and the field, which decide no slot, use
// FMAs, 1/R from canon_sqrt and a Newton reciprocal for 1/kappa (within an ulp
// or two of the correctly rounded values).
__device__ __forceinline__ double field_fp64(const double xc[3], const RecF64& st, double t_s,
                                             double qc, double qv, const Consts& K, double F[6])
{
    double d[3] = {xc[0] - st.x[0], xc[1] - st.x[1], xc[2] - st.x[2]};
    double rinv;
    const double R = canon_sqrt(canon_norm2(d[0], d[1], d[2]), &rinv);
    double tau = canon_arrival(t_s, R, K.inv_c);
    const double n[3] = {d[0] * rinv, d[1] * rinv, d[2] * rinv};
    const double w[3] = {n[0] - st.b[0], n[1] - st.b[1], n[2] - st.b[2]};
    // kappa = (|n - beta|^2 + 1/gamma^2) / 2, as canon_kappa but fused
    const double kinv =
        recip(0.5 * fma(w[0], w[0], fma(w[1], w[1], fma(w[2], w[2], st.g2i))));
    const double nwk = (n[0] * w[0] + n[1] * w[1] + n[2] * w[2]) * kinv;
    lw_fields<double>(n, w, kinv, rinv, st.g2i, st.bd, qc, qv, nwk, F);
    return canon_slot(tau, K);
}

// R = |d| and 1/R from one hardware reciprocal square root (about 23 correct
// bits) refined by a Newton step for 1/R and a residual correction for R,
// both to ~1e-15 relative -- enough for arrival times of 1e5 against slots of
// 1e-4 -- at a third of the cost of a correctly rounded sqrt plus a divide.
__device__ __forceinline__ void fast_norm(double R2, double* R, double* rinv)
{
    double y = __builtin_amdgcn_rsq(R2);
    y = y * fma(-0.5 * R2 * y, y, 1.5);
    double g = R2 * y;
    double r = fma(-g, g, R2);
    *R = fma(r, 0.5 * y, g);
    *rinv = y;
}

// |d|^2 for fast_norm, plus the smallest normal double.  That changes nothing
// for distances above ~1e-146, and a state exactly at a cell (d = 0) then gets
// R ~ 1e-154 and a finite slot coordinate -- the canonical R = 0 moves the
// slot coordinate by no more -- instead of 0 * inf.  Its field is not finite,
// as the definition's is there.
__device__ __forceinline__ double norm2_fast(double d0, double d1, double d2)
{
    return fma(d2, d2, fma(d1, d1, fma(d0, d0, 0x1p-1022)));
}

// lw_fields in single precision for a mixed-precision record, whose betadot
// already carries the factor q/c (bdq = q bd / c) and whose g2ih is 1/(2 gamma^2):
// kappa = |w|^2 / 2 + g2ih, and with n.w = kappa for a unit n,
//   E = c1 w - bdq / (kappa^2 R),  c1 = (n.bdq + qvg / R) / (kappa^3 R),
// where qvg = qv g2i = 2 qv g2ih.
__device__ __forceinline__ void lw_fields_mixed(const float n[3], const float w[3], float rinv,
                                                const RecMix& st, float qv2, float F[6])
{
    const float kinv =
        __builtin_amdgcn_rcpf(fmaf(0.5f, w[0] * w[0] + w[1] * w[1] + w[2] * w[2], st.g2ih));
    const float nbd = n[0] * st.bdq[0] + n[1] * st.bdq[1] + n[2] * st.bdq[2];
    const float rk2 = rinv * (kinv * kinv);
    const float c1 = fmaf(qv2 * st.g2ih, rinv, nbd) * (rk2 * kinv);
    const float E0 = c1 * w[0] - rk2 * st.bdq[0];
    const float E1 = c1 * w[1] - rk2 * st.bdq[1];
    const float E2 = c1 * w[2] - rk2 * st.bdq[2];
    F[0] = E0;
    F[1] = E1;
    F[2] = E2;
    F[3] = n[1] * E2 - n[2] * E1;
    F[4] = n[2] * E0 - n[0] * E2;
    F[5] = n[0] * E1 - n[1] * E0;
}

// The mixed-precision field: double for what cancels (arrival time, slot
// coordinate, n - beta), single for the rest of Eq. 1, kappa included (a sum
// of positive terms formed from the double difference n - beta).  ub is the
// state's (t_s - t0) / dt_det; the slot coordinate is ub + R / (c dt_det).
// qv2 = 2 q times the weight of the velocity term.
__device__ __forceinline__ double field_mixed(const double xc[3], const RecMix& st, double ub,
                                              float qv2, const Consts& K, float F[6])
{
    double d[3] = {xc[0] - st.x[0], xc[1] - st.x[1], xc[2] - st.x[2]};
    double R, rinv;
    fast_norm(norm2_fast(d[0], d[1], d[2]), &R, &rinv);
    const double u = fma(R, K.kR, ub);
    double nd[3] = {d[0] * rinv, d[1] * rinv, d[2] * rinv};
    double wd[3] = {nd[0] - st.b[0], nd[1] - st.b[1], nd[2] - st.b[2]};
    const float n[3] = {(float)nd[0], (float)nd[1], (float)nd[2]};
    const float w[3] = {(float)wd[0], (float)wd[1], (float)wd[2]};
    lw_fields_mixed(n, w, (float)rinv, st, qv2, F);
    return u;
}

// Far-field geometry (Eq. 3): the cell's direction and distance from the
// origin, fc = {n0, n1, n2, R_cell}; arrival t + (R_cell - x.n) (1/c), the
// dot product in a fixed order without FMA.
__device__ __forceinline__ double canon_far_arrival(double t, const double fc[4],
                                                    const double x[3], double inv_c)
{
#pragma clang fp contract(off)
    const double dot = (x[0] * fc[0] + x[1] * fc[1]) + x[2] * fc[2];
    return t + (fc[3] - dot) * inv_c;
}

// w = n - beta with the cell's direction
__device__ __forceinline__ void canon_far_w(const double fc[4], const double b[3], double w[3])
{
#pragma clang fp contract(off)
    w[0] = fc[0] - b[0];
    w[1] = fc[1] - b[1];
    w[2] = fc[2] - b[2];
}

// ub = (t_s - t0) / dt_det, as for field_mixed
__device__ __forceinline__ double slot_far_mixed(const double fc[4], const double x[3], double ub,
                                                 const Consts& K)
{
    return fma(fc[3] - (x[0] * fc[0] + x[1] * fc[1] + x[2] * fc[2]), K.kR, ub);
}

__device__ __forceinline__ double slot_far_fp64(const double fc[4], const double x[3], double t_s,
                                                const Consts& K)
{
    return canon_slot(canon_far_arrival(t_s, fc, x, K.inv_c), K);
}

// Eq. 1 with the far-field geometry n = n_cell, R = R_cell; Rinv = 1/R_cell
__device__ __forceinline__ double field_far_fp64(const double fc[4], double Rinv,
                                                 const RecF64& st, double t_s, double qc,
                                                 double qv, const Consts& K, double F[6])
{
    double w[3];
    canon_far_w(fc, st.b, w);
    const double kinv = recip(canon_kappa(w, st.g2i));
    const double nwk = (fc[0] * w[0] + fc[1] * w[1] + fc[2] * w[2]) * kinv;
    lw_fields<double>(fc, w, kinv, Rinv, st.g2i, st.bd, qc, qv, nwk, F);
    return slot_far_fp64(fc, st.x, t_s, K);
}

__device__ __forceinline__ double field_far_mixed(const double fc[4], double Rinv,
                                                  const RecMix& st, double ub, float qv2,
                                                  const Consts& K, float F[6])
{
    const double u = slot_far_mixed(fc, st.x, ub, K);
    const double wd[3] = {fc[0] - st.b[0], fc[1] - st.b[1], fc[2] - st.b[2]};
    const float n[3] = {(float)fc[0], (float)fc[1], (float)fc[2]};
    const float w[3] = {(float)wd[0], (float)wd[1], (float)wd[2]};
    lw_fields_mixed(n, w, (float)Rinv, st, qv2, F);
    return u;
}

// 1/gamma^2 of a staged state
__device__ __forceinline__ double rec_g2i(const RecF64& st) { return st.g2i; }
__device__ __forceinline__ double rec_g2i(const RecMix& st) { return 2.0 * (double)st.g2ih; }

// Lienard-Wiechert potentials phi = q/(kappa R), A = q beta/(kappa R) at a
// staged state (the potentials option): F = (A_x, A_y, A_z, phi, 0, 0).  FAR:
// the cell's direction and distance.  (The caller takes the slot coordinate
// from the same expression its other deposits use.)
template <bool FAR, typename Rec, typename T>
__device__ __forceinline__ void potentials_at(const double xc[3], const double fc[4],
                                              const Rec& st, double q, T F[6])
{
    double kap, rinv;
    if constexpr (FAR) {
        double w[3];
        canon_far_w(fc, st.b, w);
        kap = canon_kappa(w, rec_g2i(st));
        rinv = 1.0 / fc[3];
    } else {
        double d[3] = {xc[0] - st.x[0], xc[1] - st.x[1], xc[2] - st.x[2]};
        const double R = canon_sqrt(canon_norm2(d[0], d[1], d[2]));
        rinv = 1.0 / R;
        double n[3], w[3];
        canon_direction(d, rinv, st.b, n, w);
        kap = canon_kappa(w, rec_g2i(st));
    }
    const double phi = q * rinv / kap;
    F[0] = T(phi * st.b[0]);
    F[1] = T(phi * st.b[1]);
    F[2] = T(phi * st.b[2]);
    F[3] = T(phi);
    F[4] = T(0);
    F[5] = T(0);
}

__device__ __forceinline__ double slot_coord_fp64(const double xc[3], const double x[3],
                                                  double t_s, const Consts& K)
{
    double d[3] = {xc[0] - x[0], xc[1] - x[1], xc[2] - x[2]};
    const double R = canon_sqrt(canon_norm2(d[0], d[1], d[2]));
    return canon_slot(canon_arrival(t_s, R, K.inv_c), K);
}

// ub = (t_s - t0) / dt_det, as for field_mixed
__device__ __forceinline__ double slot_coord_mixed(const double xc[3], const double x[3],
                                                   double ub, const Consts& K)
{
    double d[3] = {xc[0] - x[0], xc[1] - x[1], xc[2] - x[2]};
    double R, rinv;
    fast_norm(norm2_fast(d[0], d[1], d[2]), &R, &rinv);
    return fma(R, K.kR, ub);
}

// ---------------------------------------------------------------------------
// kernels
// ---------------------------------------------------------------------------

// One thread per (particle, state): the state record of mode M, particle-major.
// betadot of a state: kBdBackward (beta_s - beta_{s-1})/dt, zero at the chunk's first
// state (it carries no segment); kBdBackwardFirst the same but the forward difference
// at the first state (its field is held by the previous-state rule); kBdCentred
// (beta_{s+1} - beta_{s-1})/(2 dt), one-sided at the chunk's ends (linear rule)
constexpr int kBdBackward = 0, kBdBackwardFirst = 1, kBdCentred = 2;

// Mixed-precision records carry the particle's q/c in betadot and half of
// 1/gamma^2, the forms their field takes (q: [n_p] or nullptr, all -1).  x and
// u point at the job's state 0, with components `stride` elements apart; they
// hold states s_lo <= 0 .. s_hi >= n_s (a time slice of a longer chunk reads
// its neighbours, so that its records equal those of the whole chunk).
template <int M>
__global__ __launch_bounds__(256) void kinematics_kernel(const double* __restrict__ x,
                                                         const double* __restrict__ u,
                                                         const double* __restrict__ q,
                                                         int64_t n_p, int64_t n_s, int64_t stride,
                                                         int64_t s_lo, int64_t s_hi, double dt,
                                                         double inv_c, int bd_rule,
                                                         void* __restrict__ recs_out,
                                                         RingState* __restrict__ rings)
{
    if (blockIdx.x == 0 && threadIdx.x == 0)
        *rings = RingState{};  // for this deposit's ring choice

    using Rec = typename std::conditional<M == kModeF64, RecF64, RecMix>::type;
    Rec* recs = reinterpret_cast<Rec*>(recs_out);
    const int64_t n_states = n_s + 1;
    const int64_t total = n_p * n_states;
    for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < total;
         i += (int64_t)gridDim.x * blockDim.x) {
        const int64_t s = i / n_p;  // consecutive threads read consecutive particles
        const int64_t p = i - s * n_p;
        const int64_t off = s * n_p + p;
        Rec r;
        r.x[0] = x[off];
        r.x[1] = x[off + stride];
        r.x[2] = x[off + 2 * stride];
        double g2i;
        canon_kinematics(u[off], u[off + stride], u[off + 2 * stride], r.b, &g2i);
        double bd[3] = {0.0, 0.0, 0.0};
        if (bd_rule == kBdCentred && s_hi > s_lo) {
            const int64_t sa = s > s_lo ? s - 1 : s_lo;
            const int64_t sb = s < s_hi ? s + 1 : s_hi;
            double ba[3], bb[3], g;
            const int64_t oa = sa * n_p + p, ob = sb * n_p + p;
            canon_kinematics(u[oa], u[oa + stride], u[oa + 2 * stride], ba, &g);
            canon_kinematics(u[ob], u[ob + stride], u[ob + 2 * stride], bb, &g);
#pragma unroll
            for (int c = 0; c < 3; ++c)
                bd[c] = canon_betadot(bb[c], ba[c], (double)(sb - sa) * dt);
        } else if (s > s_lo || (bd_rule == kBdBackwardFirst && s_hi > s_lo)) {
            // backward difference; at the first state, the forward one
            double bo[3], go;
            const int64_t o2 = s > s_lo ? off - n_p : off + n_p;
            canon_kinematics(u[o2], u[o2 + stride], u[o2 + 2 * stride], bo, &go);
#pragma unroll
            for (int c = 0; c < 3; ++c)
                bd[c] = s > s_lo ? canon_betadot(r.b[c], bo[c], dt)
                                 : canon_betadot(bo[c], r.b[c], dt);
        }
        if constexpr (M == kModeF64) {
#pragma unroll
            for (int c = 0; c < 3; ++c)
                r.bd[c] = bd[c];
            r.g2i = g2i;
        } else {
            const double qc = (q ? q[p] : -1.0) * inv_c;
#pragma unroll
            for (int c = 0; c < 3; ++c)
                r.bdq[c] = (float)(qc * bd[c]);
            r.g2ih = (float)(0.5 * g2i);
        }
        recs[p * n_states + s] = r;
    }
}

// Counting sort of the particles of one chunk, per tile, by the light-travel
// distance from the tile's centre to each particle at state s_key, in bins of
// one slot (widened if the spread needs more than kOrderBins).  perm[tile][i]
// is the i-th particle in that order.
//
// Latency bound: a workgroup sorts one tile's particles for one group of runs,
// and there are tiles x groups of them.  Only the bins the spread covers are
// cleared and scanned, the scan is a wavefront scan (one thread walking all
// bins in LDS was 38 us of every order, whatever the particle count), and up
// to kOrderHeld particles a thread keep their key in registers over the three
// passes (range, histogram, scatter) instead of computing it again.
// Measured (a serial scan and three key passes before): one particle, 64 tiles
// 38.6 -> 6.8 us; 1000 particles, 1024 tiles x 128 groups 4348 -> 675 us.
constexpr int kOrderBins = 4096;
constexpr int kOrderHeld = 8;  // keys a thread holds (n_p <= 256 * kOrderHeld)

template <bool HELD>
__global__ __launch_bounds__(256) void order_kernel(const double* __restrict__ x, int64_t n_p,
                                                    int64_t n_s, int64_t xs_stride,
                                                    int64_t n_tiles, int64_t tile_cells,
                                                    int64_t steps_per_group,
                                                    const double* __restrict__ cells, int64_t n_c,
                                                    double inv_c, double inv_dt_det,
                                                    int32_t* __restrict__ perm, int64_t item0)
{
    __shared__ __align__(16) unsigned hist[kOrderBins];
    __shared__ double red[2][4];
    __shared__ unsigned wave_sum[4];
    const int tid = threadIdx.x;
    const int lane = tid % 64, wave = tid / 64;
    const int64_t item = item0 + blockIdx.x;
    const int64_t tile = item % n_tiles;
    const int64_t group = item / n_tiles;
    // the group's middle state
    const int64_t s_key = min(n_s, group * steps_per_group + steps_per_group / 2);
    const int64_t c0 = tile * tile_cells;
    const int64_t c1 = min(c0 + tile_cells, n_c);
    double ctr[3] = {0.0, 0.0, 0.0};  // the tile's centre (uniform: scalar loads)
    for (int64_t c = c0; c < c1; ++c)
#pragma unroll
        for (int k = 0; k < 3; ++k)
            ctr[k] += cells[3 * c + k];
#pragma unroll
    for (int k = 0; k < 3; ++k)
        ctr[k] /= (double)(c1 - c0);
    const int64_t stride = xs_stride;
    const int64_t base = s_key * n_p;
    auto key = [&](int64_t p) {
        const double d0 = ctr[0] - x[base + p];
        const double d1 = ctr[1] - x[base + p + stride];
        const double d2 = ctr[2] - x[base + p + 2 * stride];
        return __builtin_sqrt(d0 * d0 + d1 * d1 + d2 * d2) * (inv_c * inv_dt_det);
    };
    double held[kOrderHeld];
    double lo = 1e300, hi = -1e300;
    auto range = [&](double k) {
        if (k == k) {
            lo = fmin(lo, k);
            hi = fmax(hi, k);
        }
    };
    if constexpr (HELD) {
#pragma unroll
        for (int i = 0; i < kOrderHeld; ++i) {
            const int64_t p = tid + 256 * i;
            if (p < n_p) {
                held[i] = key(p);
                range(held[i]);
            }
        }
    } else {
        for (int64_t p = tid; p < n_p; p += 256)
            range(key(p));
    }
    for (int m = 32; m > 0; m >>= 1) {
        lo = fmin(lo, __shfl_xor(lo, m));
        hi = fmax(hi, __shfl_xor(hi, m));
    }
    if (lane == 0) {
        red[0][wave] = lo;
        red[1][wave] = hi;
    }
    __syncthreads();
    lo = fmin(fmin(red[0][0], red[0][1]), fmin(red[0][2], red[0][3]));
    hi = fmax(fmax(red[1][0], red[1][1]), fmax(red[1][2], red[1][3]));
    const double span = hi > lo ? hi - lo : 0.0;
    const double width = span < (double)(kOrderBins - 1) ? 1.0 : span / (double)(kOrderBins - 1);
    // bins in use; the last one also takes the particles without a key (NaN)
    const int last = (int)fmin(span / width, (double)(kOrderBins - 2)) + 1;
    const int n_bins = min(kOrderBins, (last + 1 + 1023) / 1024 * 1024);  // four a thread
    for (int i = tid; i < n_bins; i += 256)
        hist[i] = 0u;
    __syncthreads();
    auto bin_of = [&](double k) {
        const double b = (k - lo) / width;
        return (b == b) ? (int)fmin(fmax(b, 0.0), (double)last) : last;
    };
    if constexpr (HELD) {
#pragma unroll
        for (int i = 0; i < kOrderHeld; ++i)
            if (tid + 256 * i < n_p)
                atomicAdd(&hist[bin_of(held[i])], 1u);
    } else {
        for (int64_t p = tid; p < n_p; p += 256)
            atomicAdd(&hist[bin_of(key(p))], 1u);
    }
    __syncthreads();
    // exclusive scan, 1024 bins a round: four consecutive ones a thread
    unsigned before = 0u;  // particles in the rounds before
    for (int r = 0; r < n_bins; r += 1024) {
        uint4* h4 = reinterpret_cast<uint4*>(hist + r) + tid;
        const uint4 h = *h4;
        const unsigned own = h.x + h.y + h.z + h.w;
        unsigned incl = own;
        for (int m = 1; m < 64; m <<= 1) {
            const unsigned t = __shfl_up(incl, m);
            incl += lane >= m ? t : 0u;
        }
        if (lane == 63)
            wave_sum[wave] = incl;
        __syncthreads();
        unsigned off = before + incl - own;
        for (int w = 0; w < wave; ++w)
            off += wave_sum[w];
        before += wave_sum[0] + wave_sum[1] + wave_sum[2] + wave_sum[3];
        *h4 = make_uint4(off, off + h.x, off + h.x + h.y, off + h.x + h.y + h.z);
        __syncthreads();
    }
    int32_t* out = perm + (group * n_tiles + tile) * n_p;
    if constexpr (HELD) {
#pragma unroll
        for (int i = 0; i < kOrderHeld; ++i)
            if (tid + 256 * i < n_p)
                out[atomicAdd(&hist[bin_of(held[i])], 1u)] = tid + 256 * i;
    } else {
        for (int64_t p = tid; p < n_p; p += 256)
            out[atomicAdd(&hist[bin_of(key(p))], 1u)] = (int32_t)p;
    }
}

// The ring a deposit's tiles take (RingState::mode): the small ring keeps four or five
// workgroups on a CU, the large one two, so the large ring pays only where the small
// one would send many emissions to HBM.  A workgroup looks at one tile, or at a row of
// neighbouring tiles of a large detector: it replays sampled batches (places and runs
// by a sequence that spreads evenly over both, for the estimates with another start in
// each workgroup; with the same places and runs everywhere a sheet was taken for 0.4%
// outside the small ring where 2.3% were) at one cell each, places the rings the way the deposit does
// (below the batch's earliest start) and counts the slots a lane would emit outside
// them.  The large ring's runs are staged in halves, quarters, ... where a whole one
// would outgrow it: a shorter stretch pays a batch's staging and ring move for fewer
// segments, and helps only where it is the run, not the spread of the batch's
// particles, that is too long.
//
// The last workgroup to finish takes the cheapest ring by the estimates below, from
// the counts of all tiles.  One ring for all of them: tiles of the other ring are a
// second launch, which pays a round of its own however few they are, and a tile's own
// samples say less than all tiles' do.  Of 50 deposits timed with either ring for all
// tiles and with each tile's own, its own took up to 1.9 times as long as the better
// single ring, and was the faster by 10% at the most.  Only a detector whose tiles
// differ enough gets each tile's own: they choose by one half of their samples, the same
// places and runs for all, so that it is the tiles that differ, and what either way
// costs is estimated from the other half.
// Only speed depends on all this: emissions outside a ring go to HBM directly.
//
// Bound by latency: the order, then all states of a sampled run at once, which stay in
// registers; the lanes of a batch share their minima by shuffles.  With a workgroup per
// tile, a loop of dependent loads, LDS atomics and a step per slot crossed: 100 tiles 33
// us, 1024 tiles 68; now 24 and 28.

// Estimates, in picoseconds of the whole device per interaction, of an average of E slots
// emitted per segment, `out` of them outside the ring; fitted to 50 deposits a mode, each
// timed with either ring and with stretches of 16 to one segments (undulators, sheets
// at 0.4 to 6 slots a segment, waves, circular orbits, uneven sets; default shape, 0.1 to
// 1.6 slots a segment):
//   small ring  max(small + small_slot E, least + outside out): few adds to HBM hide
//               behind the fields
//   large ring  large + large_slot E + batch / L + missed out, L segments a stretch
struct RingCost {
    float small, small_slot, least, outside, large, large_slot, batch, missed;
};
constexpr RingCost kRingCost[3] = {
    {4.0f, 2.0f, 1.5f, 310.0f, 4.4f, 1.7f, 22.0f, 230.0f},   // double
    {2.6f, 2.0f, 1.0f, 310.0f, 3.4f, 1.8f, 22.0f, 230.0f},   // mixed
    {2.7f, 2.2f, 1.0f, 720.0f, 3.6f, 2.2f, 36.0f, 350.0f}};  // compensated: two adds a
                                                             // component, the first returning
// the linear hold's second field, with either ring: behind it more of the adds hide (300
// electrons x 1024 steps x 64 x 64 cells, mixed: small ring 6.5 ms, large 7.9; with the
// default hold both 6.3)
constexpr float kLinearField = 1.3f;
// what each tile's own ring has to gain: in a batch the other pairs fill its launches
constexpr float kOwnGain = 0.88f, kOwnGainBatch = 0.96f;
// a round's time with one workgroup a CU, of that with all that are resident (200 electrons
// x 200 steps x 16 x 16 cells, 624 items: 124 us in the small ring, 158 in the large one)
constexpr float kAloneSmall = 0.4f, kAloneLarge = 0.7f;
// Workgroups at most (4096 sampled batches): more add up to no better choice, and the
// loads of their samples took 79 us for 1024 tiles.
constexpr int64_t kChoiceBlocks = 256;

// counts of a run's slots: all emitted, outside the small ring, the segments, and the
// segments that end outside the large ring with stretches of L >> h
struct RingCounts {
    float all, out, segs, far[kRingShifts];
};

__device__ __forceinline__ float small_ring_cost(const RingCost& K, const RingCounts& c)
{
    return fmaxf(K.small + K.small_slot * c.all / c.segs, K.least + K.outside * c.out / c.segs);
}

// the cheapest stretch of runs of L segments and its cost
__device__ __forceinline__ float large_ring_cost(const RingCost& K, const RingCounts& c, int L,
                                                 int* shift)
{
    const float E = c.all / c.segs;
    float best = INFINITY;
    for (int h = 0; h < kRingShifts && (L >> h) > 0; ++h) {
        const float cost = K.large + K.large_slot * E + K.batch / (float)(L >> h) +
                           K.missed * E * c.far[h] / c.segs;
        if (cost < best) {
            best = cost;
            *shift = h;
        }
    }
    return best;
}

template <int L>
__global__ __launch_bounds__(256) void ring_choice_kernel(DepositJob J, int64_t rec_size,
                                                          RingCost K, int64_t tiles_each)
{
    constexpr int kShifts = L == 16 ? 4 : 3;  // stretches down to one segment
    static_assert((L >> kShifts) == 1 && kShifts < kRingShifts, "runs of 16 or 8 segments");
    enum { kAll, kOut, kSegs, kFar, kCounts = kFar + kRingShifts };  // as RingCounts
    __shared__ unsigned part[2][4][kCounts];  // by half of the samples
    const int tid = threadIdx.x;
    const int groups = J.groups;
    const int n_samples = 256 / groups;  // sampled batches, a thread per particle
    const int smp = tid / groups;
    const int gg = tid % groups;
    const int64_t tile_a = blockIdx.x * tiles_each;
    const int64_t n_here = min(tiles_each, J.n_tiles - tile_a);
    const int64_t tile = tile_a + (int64_t)smp * n_here / n_samples;
    const int64_t n_batches = (J.n_p + groups - 1) / groups;
    // runs and places: the plane sequence of the plastic number, the same for one half of
    // each workgroup's batches, shifted at random from workgroup to workgroup for the other
    unsigned rnd = (smp & 1 ? blockIdx.x + 1u : 0u) * 0x9e3779b9u;
    rnd = (rnd ^ (rnd >> 15)) * 0x85ebca6bu;
    rnd = (rnd ^ (rnd >> 13)) * 0xc2b2ae35u;
    rnd ^= rnd >> 16;
    const double id = (double)(smp / 2);
    const double at_run = id * 0.7548776662466927 + (double)(rnd & 0xffffu) * 0x1p-16;
    const double at_place = id * 0.5698402909980532 + (double)(rnd >> 16) * 0x1p-16;
    const int64_t run = min((int64_t)((at_run - floor(at_run)) * (double)J.n_runs), J.n_runs - 1);
    const int64_t bt =
        min((int64_t)((at_place - floor(at_place)) * (double)n_batches), n_batches - 1);
    const int64_t pi = bt * groups + gg;
    const int64_t s_a = run * L;
    const int len = (int)min((int64_t)L, J.n_s - s_a);
    const bool on = pi < J.n_p;
    const int64_t c0 = tile * J.tile_cells;
    const int64_t cell = c0 + (int64_t)(5 * smp) % min((int64_t)J.tile_cells, J.n_c - c0);
    const double* xc = J.cells + 3 * cell;
    const double* fc = J.far ? J.far + 4 * cell : nullptr;
    const int32_t* order = J.perm + ((run / J.runs_per_group) * J.n_tiles + tile) * J.n_p;
    const char* pr = reinterpret_cast<const char*>(J.recs) +
                     ((int64_t)order[on ? pi : 0] * (J.n_s + 1) + s_a) * rec_size;
    // slots of the run's states (a record starts with its position), and the lowest of
    // the batch's particles at each
    const int n_t = (int)J.n_t;
    int slot[L + 1], start[L + 1];
#pragma unroll
    for (int k = 0; k <= L; ++k) {
        const int kk = min(k, len);
        const double* x = reinterpret_cast<const double*>(pr + kk * rec_size);
        double dist;
        if (fc) {
            dist = fc[3] - (x[0] * fc[0] + x[1] * fc[1] + x[2] * fc[2]);
        } else {
            const double d0 = xc[0] - x[0], d1 = xc[1] - x[1], d2 = xc[2] - x[2];
            dist = __builtin_sqrt(d0 * d0 + d1 * d1 + d2 * d2);
        }
        const double u =
            ((J.t_first + (double)(J.s0 + s_a + kk) * J.dt) + dist * J.inv_c - J.t0) * J.inv_dt_det;
        slot[k] = (int)floor((u == u) ? fmin(fmax(u, -2.0), (double)n_t + 2.0) : -2.0);
        start[k] = on ? slot[k] : INT_MAX;
    }
    for (int m = groups / 2; m > 0; m >>= 1)
#pragma unroll
        for (int k = 0; k < L; ++k)
            start[k] = min(start[k], __shfl_xor(start[k], m));
    // where a ring of R slots starts that is placed at a batch's lowest slot
    auto placed = [&](int lo, int R) { return min(max(lo - kRingMargin, 0), max(n_t - R, 0)); };
    unsigned count[kCounts] = {};
    const int base = placed(start[0], kRingSmall);
    // slots [a, b) left: all within the window, and those outside the small ring
    auto emit = [&](int a, int b) {
        const int all = max(min(b, n_t) - max(a, 0), 0);
        const int in = max(min(min(b, n_t), base + kRingSmall) - max(a, base), 0);
        count[kAll] += (unsigned)all;
        count[kOut] += (unsigned)(all - in);
    };
    int base_large[kShifts + 1];
#pragma unroll
    for (int k = 1; k <= L; ++k) {
        const int prev = slot[k - 1], cur = slot[k];
        if (on && k <= len)
            emit(min(prev, cur), max(prev, cur));
#pragma unroll
        for (int h = 0; h <= kShifts; ++h) {  // the large ring, by length of stretch
            if (((k - 1) & ((L >> h) - 1)) == 0)
                base_large[h] = placed(start[k - 1], kRingLarge);
            count[kFar + h] += on && k <= len && cur >= 0 && cur < n_t &&
                                       (cur < base_large[h] || cur >= base_large[h] + kRingLarge)
                                   ? 1u
                                   : 0u;
        }
    }
    if (on) {
        emit(slot[L], slot[L] + 1);  // the run's last slot
        count[kSegs] = (unsigned)len;
    }
#pragma unroll
    for (int i = 0; i < kCounts; ++i) {
        for (int m = 32; m > 0; m >>= 1)
            if (m != groups)  // the even and the odd batches each for themselves
                count[i] += __shfl_xor(count[i], m);
        if ((tid % 64 & ~groups) == 0)
            part[(tid % 64) / groups][tid / 64][i] = count[i];
    }
    __syncthreads();
    if (tid >= 64)
        return;
    // every lane of the first wavefront: which ring the tiles by themselves would take
    auto of_half = [&](int half, int i) {
        return part[half][0][i] + part[half][1][i] + part[half][2][i] + part[half][3][i];
    };
    RingCounts c;
#pragma unroll
    for (int i = 0; i < kCounts; ++i)
        (&c.all)[i] = (float)of_half(0, i);
    int shift = 0;
    const int own = large_ring_cost(K, c, L, &shift) < small_ring_cost(K, c) ? 1 : 0;
    for (int64_t i = tid; i < n_here; i += 64)
        J.ring_sel[tile_a + i] = (uint8_t)own;
    // by the other half, the sums of either kind of tile; the last workgroup settles the
    // mode
    RingState* R = J.rings;
    auto add = [&](unsigned long long* to, int64_t v) {
        __hip_atomic_fetch_add(to, (unsigned long long)v, __ATOMIC_RELAXED,
                               __HIP_MEMORY_SCOPE_AGENT);
    };
    if (tid < kCounts) {
        add(&R->kind[own][tid], of_half(1, tid));
    } else if (tid == kCounts) {
        add(&R->tiles[own], n_here);
    }
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "agent");  // the wavefront's adds, before `done`
    if (tid != 0)
        return;
    const unsigned done =
        __hip_atomic_fetch_add(&R->done, 1u, __ATOMIC_ACQ_REL, __HIP_MEMORY_SCOPE_AGENT);
    if (done + 1u != gridDim.x)
        return;
    auto get = [&](unsigned long long* from) {
        return (float)__hip_atomic_load(from, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    };
    RingCounts kind[2], all;
    for (int i = 0; i < kCounts; ++i) {
        (&kind[0].all)[i] = get(&R->kind[0][i]);
        (&kind[1].all)[i] = get(&R->kind[1][i]);
        (&all.all)[i] = (&kind[0].all)[i] + (&kind[1].all)[i];
    }
    const float n[2] = {get(&R->tiles[0]), get(&R->tiles[1])};
    const float items = (float)(J.n_splits * J.n_parts);  // of a tile
    // time of a launch over n tiles of the cost, at least a round of resident workgroups,
    // which is shorter the fewer a CU has of them
    auto launch_small = [&](float tiles, const RingCounts& counts) {
        return small_ring_cost(K, counts) *
               fmaxf(tiles, kAloneSmall * (float)J.resident_small / items);
    };
    auto launch_large = [&](float tiles, const RingCounts& counts, int* h) {
        return large_ring_cost(K, counts, L, h) *
               fmaxf(tiles, kAloneLarge * (float)J.resident_large / items);
    };
    int shift_own = 0;
    const float small = launch_small(n[0] + n[1], all);
    const float large = launch_large(n[0] + n[1], all, &shift);
    unsigned mode = small <= large ? kRingSel16 : kRingSel64 + shift;
    if (kind[0].segs > 0.0f && kind[1].segs > 0.0f) {
        const float mixed =
            launch_small(n[0], kind[0]) + launch_large(n[1], kind[1], &shift_own);
        if (mixed < (J.rings_used ? kOwnGainBatch : kOwnGain) * fminf(small, large))
            mode = kRingsOwn | (kRingSel64 + shift_own);
    }
    R->mode = mode;
    if (J.rings_used) {  // a batch: which of its launches has work
        if (mode == kRingSel16 || (mode & kRingsOwn))
            __hip_atomic_fetch_or(J.rings_used, 1ull, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        if (mode != kRingSel16)
            __hip_atomic_fetch_or(J.rings_used + 1, 1ull, __ATOMIC_RELAXED,
                                  __HIP_MEMORY_SCOPE_AGENT);
    }
}

// The ring of a tile (kRingSel...)
__device__ __forceinline__ int ring_of(const DepositJob& J, int64_t tile)
{
    const unsigned mode = gptr(J.rings)->mode;
    if ((mode & kRingsOwn) == 0)
        return (int)mode;
    return gptr(J.ring_sel)[tile] != 0 ? (int)(mode & ~kRingsOwn) : kRingSel16;
}

// M: arithmetic of the deposit (field in double or single; accumulation in
// double or compensated single pairs)
template <int M>
struct ModeTypes {
    static constexpr bool MIX = (M != kModeF64);
    using T = typename std::conditional<MIX, float, double>::type;  // field and lane carry
    using Acc = typename std::conditional<M == kModeMixTwoSum, float, double>::type;
    using Rec = typename std::conditional<MIX, RecMix, RecF64>::type;  // staged state record
};

// LDS of one deposit workgroup of shape SH with rings of R slots
template <int M, int R, int SH>
struct DepositShared {
    using Acc = typename ModeTypes<M>::Acc;
    static constexpr int TC = shape_cells(SH);   // cells per tile
    static constexpr int GR = shape_groups(SH);  // particles per batch
    // the rings' words, cell fastest: an update of several cells by one instruction
    // meets no bank twice but for lanes of one cell
    static constexpr int kRingWords = TC * R * 6;
    static constexpr int L = shape_run(SH);
    typename ModeTypes<M>::Rec rec[GR][L + 1];  // staged batch: L segments per group
    double sq[GR];                      // its charges
    double tk[L + 1];                   // its states' time arguments (the same for every lane)
    double ring[kRingWords];            // per-cell slot rings, [slot][component][cell]
    int ring_base[TC];                  // per cell: where its ring starts,
    Acc* row[TC];                       // and its slots in HBM (null past the last cell)
    int nb[2][TC];                      // per cell: lowest start slot of a coming batch
    int ord[2][GR];                     // particles of the staged rows, per batch parity
    unsigned long long cnt[kCounters];  // clipped, nonmonotone, bypassed, large-ring interactions
};

// One work item: a tile of kTileCells cells against the runs
// [split * runs_per_split, ...) of the particles in batches
// [part * batches_per_part, ...) of the tile's particle order (job J).
// Called by all kDepositThreads threads of a workgroup.
// Lane (cell, group) = (lane % kTileCells, lane / kTileCells): the sixteen
// lanes of a wavefront's row hold different cells, so one ring update
// instruction touches different rings, and the four groups of a wavefront
// read their particles' records as LDS broadcasts.
// HOLD: which field a segment holds (0 the current state's, 1 the previous
// state's, 2 the linear interpolation between the two)
// G: bit 0 the far-field geometry, bit 1 potentials instead of fields
// DIV: the double slot coordinate divides (a divisor that fails the host check
// of canon_slot's corrections); a compile-time choice, so that the state loop
// carries no branch for it.
// sel: the tile's ring choice (large ring: the stretches its runs are staged in).
template <int M, int R, int G, int HOLD, int SH, bool DIV>
__device__ __forceinline__ void deposit_item(const DepositJob& J, int64_t tile, int64_t split,
                                             int64_t part, int sel, DepositShared<M, R, SH>& sh)
{
    constexpr int kTileCells = shape_cells(SH);  // this shape's tile, batch and run
    constexpr int kGroups = shape_groups(SH);
    constexpr int kRunL = shape_run(SH);
    constexpr bool FAR = (G & 1) != 0;
    constexpr bool POT = (G & 2) != 0;
    constexpr bool MIX = ModeTypes<M>::MIX;
    using T = typename ModeTypes<M>::T;
    using Acc = typename ModeTypes<M>::Acc;
    using Sink = CellSink<Acc, R, kTileCells>;
    using Rec = typename ModeTypes<M>::Rec;
    constexpr int RW = Sink::W;
    const Rec* recs = reinterpret_cast<const Rec*>(J.recs);

    const int tid = threadIdx.x;
    const int cl = tid % kTileCells;  // cell within the tile
    const int g = tid / kTileCells;   // particle group
    const int64_t row_i = tile * kTileCells + cl;  // internal (tile-ordered) cell row
    const bool active = row_i < J.n_c;
    const int n_t = (int)J.n_t;
    const Consts K{J.t0, J.inv_dt_det, J.inv_c, J.inv_c * J.inv_dt_det, J.dt_det, DIV};
    const double ntd = (double)n_t;
    // the time argument of the field and slot functions for state index sk: the
    // state time t_s (double mode, canonical rounding), or (t_s - t0) / dt_det
    const double ub0 = (J.t_first - J.t0) * J.inv_dt_det, dtu = J.dt * J.inv_dt_det;
    auto clock = [&](double sk) {
        if constexpr (MIX)
            return fma(sk, dtu, ub0);
        else
            return canon_state_time(J.t_first, sk, J.dt);
    };
    double xc[3] = {0.0, 0.0, 0.0};
    double fc[4] = {0.0, 0.0, 0.0, 1.0};  // far field: the cell's direction and distance
    RADIO_GLOBAL Acc* row = nullptr;
    if (active) {
        const RADIO_GLOBAL double* cells = gptr(J.cells);
        xc[0] = cells[3 * row_i];
        xc[1] = cells[3 * row_i + 1];
        xc[2] = cells[3 * row_i + 2];
        if constexpr (FAR) {
            const RADIO_GLOBAL double* f = gptr(J.far) + 4 * row_i;
            fc[0] = f[0];
            fc[1] = f[1];
            fc[2] = f[2];
            fc[3] = f[3];
        }
        row = gptr(reinterpret_cast<Acc*>(J.acc + row_i * J.n_t * 6));
    }
    const double Rinv = 1.0 / fc[3];
    // slot coordinate of a state, the same expression the field functions use
    auto slot_of = [&](const Rec& st, double tk) {
        if constexpr (FAR)
            return MIX ? slot_far_mixed(fc, st.x, tk, K) : slot_far_fp64(fc, st.x, tk, K);
        else
            return MIX ? slot_coord_mixed(xc, st.x, tk, K) : slot_coord_fp64(xc, st.x, tk, K);
    };
    RADIO_LDS double* my_ring = (RADIO_LDS double*)&sh.ring[cl];
    RADIO_LDS int* nb = (RADIO_LDS int*)&sh.nb[0][0];
    for (int i = g; i < R * RW; i += kGroups)
        my_ring[i * kTileCells] = 0.0;
    if (tid < kCounters)
        sh.cnt[tid] = 0;
    if (tid < 2 * kTileCells)
        nb[tid] = INT_MAX;
    if (tid < kTileCells) {
        sh.ring_base[tid] = 0;
        sh.row[tid] = (Acc*)row;
    }
    int base = 0;  // the ring covers [base, base + R), 0 <= base <= max(n_t - R, 0)
    unsigned n_clip = 0, n_back = 0, n_bypass = 0;
    unsigned n_large = 0;  // large ring: the lane's segments (its interactions)
    // the tile's particle order for run rb (one order per group of runs)
    auto order_of = [&](int64_t rb_) {
        return gptr(J.perm + ((rb_ >> J.group_shift) * J.n_tiles + tile) * J.n_p);
    };
    const RADIO_GLOBAL double* charges = J.q ? gptr(J.q) : nullptr;
    const int64_t n_states = J.n_s + 1;
    const int64_t bt_begin = part * J.batches_per_part;
    const int64_t bt_end = min(bt_begin + J.batches_per_part, (J.n_p + kGroups - 1) / kGroups);
    const int64_t n_batches = bt_end - bt_begin;  // per run
    // The item's runs [rb_begin, rb_end), staged in stretches of L segments: stretch
    // rb (states rb * L ... rb * L + L) of run rb >> ns_shift.
    // log2 of the stretches of a run
    const int ns_shift = R == kRingLarge ? sel - kRingSel64 : 0;
    const int L = kRunL >> ns_shift;
    const int64_t rb_begin = (split * J.runs_per_split) << ns_shift;
    const int64_t rb_end =
        min(min(split * J.runs_per_split + J.runs_per_split, J.n_runs) << ns_shift,
            (J.n_s + L - 1) / L);
    // The item's batches are taken part-major: part rb of the particles
    // order[bt * kGroups ...], bt = bt_begin .. bt_end - 1.
    // Before a batch is computed, one round of global loads brings its
    // records, its charges and the first positions of the next batch's
    // particles, whose lowest start slot per cell places the ring for that
    // batch before it is staged; the order entries these loads need were
    // fetched in the round before.
    auto advance = [&](int64_t& rb_, int64_t& bt_) {
        if (++bt_ == bt_end) {
            bt_ = bt_begin;
            ++rb_;
        }
    };
    // the lane's particle of batch (rb_, bt_), or -1 (the order of the part's run)
    auto lane_particle = [&](int64_t rb_, int64_t bt_, int lane_g) -> int {
        const int64_t i = bt_ * kGroups + lane_g;
        return (rb_ < rb_end && i < J.n_p) ? (int)order_of(rb_ >> ns_shift)[i] : -1;
    };
    // lowest start slot of the cell over a batch: the lane's particle starts at x
    // at state s_a (into nb[buf][cell])
    auto scout = [&](const double x[3], int64_t s_a, int buf) {
        const double t = canon_state_time(J.t_first, (double)(J.s0 + s_a), J.dt);
        double u;
        if constexpr (FAR) {
            u = (t + (fc[3] - (x[0] * fc[0] + x[1] * fc[1] + x[2] * fc[2])) * K.inv_c - K.t0) *
                K.inv_dt_det;
        } else {
            const double d0 = xc[0] - x[0], d1 = xc[1] - x[1], d2 = xc[2] - x[2];
            double dist, rinv;  // to ~1e-15: ample for placing the ring
            fast_norm(norm2_fast(d0, d1, d2), &dist, &rinv);
            u = (t + dist * K.inv_c - K.t0) * K.inv_dt_det;
        }
        if (u == u) {
            const int f = (int)floor(fmin(fmax(u, -1.0), (double)n_t + 1.0));
            __hip_atomic_fetch_min(nb + buf * kTileCells + cl, f, __ATOMIC_RELAXED,
                                   __HIP_MEMORY_SCOPE_WORKGROUP);
        }
    };
    auto first_position = [&](int p, int64_t s_a) {
        return gptr(reinterpret_cast<const double*>(recs + (int64_t)p * n_states + s_a));
    };

    // where the ring of a cell starts for a batch whose lowest start slot is lo_slot
    auto placed = [&](int lo_slot, int cur) {
        if (lo_slot == INT_MAX)
            return cur;
        return (int)fmin(fmax((double)lo_slot - (double)kRingMargin, 0.0),
                         fmax((double)(n_t - R), 0.0));
    };
    // Move the rings: slots leaving them go to HBM.  Eight lanes of one wavefront
    // (six of them at work, one per component) take a cell's slot, so that its adds
    // share a line; kSubs slots go to as many such groups, two a round.
    constexpr int kCellsPerWave = kTileCells / (kDepositThreads / 64);
    constexpr int kSubs = 64 / (8 * kCellsPerWave);
    static_assert(kCellsPerWave * 8 <= 64, "eight lanes of a wavefront per cell");
    auto move_rings = [&](int buf, bool all) {
        int t = tid;
        asm volatile("" : "+v"(t));  // derived per batch, not held through the field loop
        const int f_comp = t % 8;
        const int f_sub = (t % 64) / (8 * kCellsPerWave);
        const int f_cell = (t / 64) * kCellsPerWave + (t / 8) % kCellsPerWave;
        RADIO_GLOBAL Acc* f_row = gptr(sh.row[f_cell]);
        const int f_base = sh.ring_base[f_cell];
        const int new_base = all ? -1 : placed(nb[buf * kTileCells + f_cell], f_base);
        if (new_base == f_base || f_comp >= 6 || !f_row)
            return;
        RADIO_LDS double* comp = (RADIO_LDS double*)&sh.ring[f_comp * kTileCells + f_cell];
        // slots to flush: those before new_base, or all of them
        const int hi = new_base > f_base && new_base < f_base + R ? new_base : f_base + R;
        for (int j0 = f_base + f_sub; j0 < hi; j0 += 2 * kSubs) {
            double d[2];
#pragma unroll
            for (int i = 0; i < 2; ++i) {
                RADIO_LDS double* q = comp + ring_pos<R>(j0 + i * kSubs) * (RW * kTileCells);
                d[i] = j0 + i * kSubs < hi ? *q : 0.0;
                if (d[i] != 0.0)
                    *q = 0.0;
            }
#pragma unroll
            for (int i = 0; i < 2; ++i)
                if (d[i] != 0.0 && j0 + i * kSubs < n_t)
                    global_add_one(f_row, j0 + i * kSubs, f_comp, d[i]);
        }
        if (f_comp == 0 && f_sub == 0)
            sh.ring_base[f_cell] = new_base;
    };
    // Staging of a batch's records.  Single-precision kernels load them from
    // HBM straight into LDS (no registers held for them, which keeps their
    // register count at five wavefronts per SIMD); the double kernel, whose LDS
    // allows four workgroups per CU anyway, stages through registers with
    // kStageLanes threads per particle, which takes fewer instructions.  In
    // the latter the thread index passes through an empty asm so that what is
    // derived from it is recomputed per batch instead of being held in
    // registers across the field loop.
    // Large-ring workgroups (two per CU: their LDS allows no more) have too
    // few neighbours to hide a batch's loads, so they prefetch: the next
    // batch's records, charges and first positions are loaded into registers
    // while the current batch is computed, and written to LDS after it.
    constexpr bool kPrefetch = (R == kRingLarge);
    constexpr bool kStageDirect = MIX && !kPrefetch;
    constexpr int kStageLanes = kDepositThreads / kGroups;
    int t_stage = tid;
    asm volatile("" : "+v"(t_stage));
    // register staging: a thread holds pieces r0, r0 + kStageLanes, ... of the
    // records of particle t_stage / kStageLanes of the batch (pieces of 16
    // bytes where the record size allows, else of 8)
    using Piece = typename std::conditional<sizeof(Rec) % 16 == 0, v2i64, long long>::type;
    constexpr int kPieces = (int)(sizeof(Rec) / sizeof(Piece));
    constexpr int kIter = ((kRunL + 1) * kPieces + kStageLanes - 1) / kStageLanes;
    // the records (states s_a .. s_a + L, contiguous) and the charge of particle p
    auto load_records = [&](int p, int64_t s_a_, Piece(&v)[kIter], double& qs) {
        const int per = (int)(min((int64_t)L, J.n_s - s_a_) + 1) * kPieces;
        int t = t_stage;
        asm volatile("" : "+v"(t));
        const int r0 = t % kStageLanes;
        if (p >= 0) {
            const RADIO_GLOBAL Piece* src =
                gptr(reinterpret_cast<const Piece*>(recs + (int64_t)p * n_states + s_a_));
#pragma unroll
            for (int j = 0; j < kIter; ++j)
                if (r0 + j * kStageLanes < per)
                    v[j] = src[r0 + j * kStageLanes];
            if (r0 == 0)
                qs = charges ? charges[p] : -1.0;
        }
    };
    auto store_records = [&](int p, int len_, const Piece(&v)[kIter], double qs) {
        const int per = (len_ + 1) * kPieces;
        int t = t_stage;
        asm volatile("" : "+v"(t));
        const int gg = t / kStageLanes;
        const int r0 = t % kStageLanes;
        if (p >= 0) {
            Piece* dst = reinterpret_cast<Piece*>(&sh.rec[gg][0]);
#pragma unroll
            for (int j = 0; j < kIter; ++j)
                if (r0 + j * kStageLanes < per)
                    dst[r0 + j * kStageLanes] = v[j];
            if (r0 == 0)
                sh.sq[gg] = qs;
        }
    };
    int64_t rb = rb_begin, bt = bt_begin;  // the current batch
    int64_t rb1 = rb, bt1 = bt;     // the next one
    advance(rb1, bt1);
    int p_stage = -1, p_scout = -1;  // this thread's particle to stage; the lane's to scout
    int p_next = -1;                 // prefetch: this thread's particle of the next batch
    Piece v_pre[kPrefetch ? kIter : 1];  // prefetch: the records in flight
    double q_pre = 0.0;
    __syncthreads();  // rings and start slots cleared
    if (rb_begin < rb_end && n_batches > 0) {
        const int p0 = lane_particle(rb, bt, g);
        if (active && p0 >= 0) {
            const RADIO_GLOBAL double* x = first_position(p0, rb * L);
            const double xs[3] = {x[0], x[1], x[2]};
            scout(xs, rb * L, 0);
        }
        if constexpr (kStageDirect) {
            if (tid < kGroups)
                sh.ord[0][tid] = lane_particle(rb, bt, tid);
        } else {
            p_stage = lane_particle(rb, bt, t_stage / kStageLanes);
        }
        if constexpr (kPrefetch) {
            load_records(p_stage, rb * L, v_pre, q_pre);
            p_next = lane_particle(rb1, bt1, t_stage / kStageLanes);
        }
        p_scout = lane_particle(rb1, bt1, g);
    }
    __syncthreads();
    for (int buf = 0; rb < rb_end && n_batches > 0; buf ^= 1) {
        const int64_t s_a = rb * L;
        const int len = (int)min((int64_t)L, J.n_s - s_a);
        const int64_t i0 = bt * kGroups;
        const int np = (int)min((int64_t)kGroups, J.n_p - i0);
        // slide the ring to this batch's earliest start (every lane of the
        // previous batch is past the barrier that ended it)
        const int new_base = placed(nb[buf * kTileCells + cl], base);
        // dense arrivals seldom move a ring; a wavefront's lanes hold all cells (asked in
        // double alone: it has the registers, 5000 electrons x 30 steps x 64 x 64 cells 2.98
        // against 3.18 ms; the mixed sheet of 1e5 electrons took 196 ms instead of 194)
        if (M != kModeF64 || __ballot(new_base != base) != 0)
            move_rings(buf, false);
        base = new_base;
        int64_t rb2 = rb1, bt2 = bt1;  // the batch after the next
        advance(rb2, bt2);
        if constexpr (kStageDirect) {
            // The records go from HBM straight to LDS (16 bytes a lane, no
            // registers).  A wavefront stages whole rows: row gg (the run of
            // particle ord[gg], contiguous in HBM and in LDS) in rounds of 64
            // pieces, lane i taking piece h * 64 + i.  The particle is the same
            // for the whole wavefront, so the addressing is scalar but for the
            // lane's offset.  With the records, in the same round of loads: the
            // batch's charges, the order entries of the next batch and the next
            // batch's first positions for the ring.
            static_assert(sizeof(Rec) % 16 == 0, "records move in 16-byte pieces");
            constexpr int kPieces = (int)(sizeof(Rec) / 16);
            constexpr int kPer = (kRunL + 1) * kPieces;  // pieces of a full row
            constexpr int kWaves = kDepositThreads / 64;
            constexpr int kRowsPerWave = kGroups / kWaves;
            constexpr int kHalves = (kPer + 63) / 64;  // rounds per row
            const int per = (len + 1) * kPieces;
            const int wave = __builtin_amdgcn_readfirstlane(tid / 64);
            const int lane = tid % 64;
            RADIO_LDS char* rec_lds = (RADIO_LDS char*)&sh.rec[0][0];
            const RADIO_GLOBAL char* rec_hbm = reinterpret_cast<const RADIO_GLOBAL char*>(gptr(recs));
            int part[kRowsPerWave];  // the rows' particles, read before the first load writes LDS
#pragma unroll
            for (int k = 0; k < kRowsPerWave; ++k)
                part[k] = __builtin_amdgcn_readfirstlane(sh.ord[buf][wave + k * kWaves]);
#pragma unroll
            for (int k = 0; k < kRowsPerWave; ++k) {
                const int gg = wave + k * kWaves;
                if (gg < np) {
                    const RADIO_GLOBAL char* src =
                        rec_hbm + ((int64_t)part[k] * n_states + s_a) * (int64_t)sizeof(Rec);
#pragma unroll
                    for (int h = 0; h < kHalves; ++h)
                        if (h * 64 + lane < per)
                            __builtin_amdgcn_global_load_lds(src + (h * 64 + lane) * 16,
                                                             rec_lds + (gg * kPer + h * 64) * 16, 16,
                                                             0, 0);
                }
            }
            double qs = 0.0;
            if (tid < np)
                qs = charges ? charges[sh.ord[buf][tid]] : -1.0;
            const int ord_next = tid < kGroups ? lane_particle(rb1, bt1, tid) : -1;
            double xs[3] = {0.0, 0.0, 0.0};
            const bool scouting = active && p_scout >= 0;
            if (scouting) {
                const RADIO_GLOBAL double* x = first_position(p_scout, rb1 * L);
                xs[0] = x[0];
                xs[1] = x[1];
                xs[2] = x[2];
            }
            const int p_scout_next = lane_particle(rb2, bt2, g);
            if (tid < np)
                sh.sq[tid] = qs;
            if (tid < kGroups)
                sh.ord[buf ^ 1][tid] = ord_next;
            if (scouting)
                scout(xs, rb1 * L, buf ^ 1);
            p_scout = p_scout_next;
            asm volatile("s_waitcnt vmcnt(0)" ::: "memory");  // the records are in LDS
        } else if constexpr (kPrefetch) {
            // this batch's records came into registers while the previous one was computed
            store_records(p_stage, len, v_pre, q_pre);
        } else {
            const int per = (len + 1) * kPieces;
            int t = t_stage;
            asm volatile("" : "+v"(t));
            const int gg = t / kStageLanes;
            const int r0 = t % kStageLanes;
            // one round of loads: the records of particle p_stage (states
            // s_a .. s_a + len, contiguous), its charge, the next batch's first
            // position for the lane, and the order entries of the next round
            Piece v[kIter];
            double qs = 0.0;
            if (p_stage >= 0) {
                const RADIO_GLOBAL Piece* src =
                    gptr(reinterpret_cast<const Piece*>(recs + (int64_t)p_stage * n_states + s_a));
#pragma unroll
                for (int j = 0; j < kIter; ++j)
                    if (r0 + j * kStageLanes < per)
                        v[j] = src[r0 + j * kStageLanes];
                if (r0 == 0)
                    qs = charges ? charges[p_stage] : -1.0;
            }
            double xs[3] = {0.0, 0.0, 0.0};
            const bool scouting = active && p_scout >= 0;
            if (scouting) {
                const RADIO_GLOBAL double* x = first_position(p_scout, rb1 * L);
                xs[0] = x[0];
                xs[1] = x[1];
                xs[2] = x[2];
            }
            const int p_stage_next = lane_particle(rb1, bt1, gg);
            const int p_scout_next = lane_particle(rb2, bt2, g);
            if (p_stage >= 0) {
                Piece* dst = reinterpret_cast<Piece*>(&sh.rec[gg][0]);
#pragma unroll
                for (int j = 0; j < kIter; ++j)
                    if (r0 + j * kStageLanes < per)
                        dst[r0 + j * kStageLanes] = v[j];
                if (r0 == 0)
                    sh.sq[gg] = qs;
            }
            if (scouting)
                scout(xs, rb1 * L, buf ^ 1);
            p_stage = p_stage_next;
            p_scout = p_scout_next;
        }
        if (tid < len + 1)
            sh.tk[tid] = clock((double)(J.s0 + s_a + tid));
        __syncthreads();
        if (tid < kTileCells)  // read by every lane before the barrier; next used two batches on
            nb[buf * kTileCells + tid] = INT_MAX;
        // prefetch: in flight while this batch is computed, the next batch's
        // records and charges, its first positions (for its ring placement) and
        // the order entries of the batch after it
        double xs_next[3] = {0.0, 0.0, 0.0};
        bool scout_next = false;
        int p_stage_after = -1, p_scout_after = -1;
        if constexpr (kPrefetch) {
            load_records(p_next, rb1 * L, v_pre, q_pre);
            scout_next = active && p_scout >= 0;
            if (scout_next) {
                const RADIO_GLOBAL double* x = first_position(p_scout, rb1 * L);
                xs_next[0] = x[0];
                xs_next[1] = x[1];
                xs_next[2] = x[2];
            }
            p_stage_after = lane_particle(rb2, bt2, t_stage / kStageLanes);
            p_scout_after = lane_particle(rb2, bt2, g);
        }
        if (active && g < np) {
            if constexpr (R == kRingLarge)
                n_large += (unsigned)len;
            const double q = sh.sq[g];
            // (the mixed records carry q/c in their betadot)
            const T qc = T(q * J.inv_c), qv = T(q * J.vscale), qv2 = T(2.0 * q * J.vscale);
            // the field of one staged state and its slot coordinate
            auto field_at = [&](const Rec& st, double tk, T F[6]) {
                if constexpr (POT) {
                    potentials_at<FAR>(xc, fc, st, q, F);
                    return slot_of(st, tk);
                } else if constexpr (FAR) {
                    if constexpr (MIX)
                        return field_far_mixed(fc, Rinv, st, tk, qv2, K, F);
                    else
                        return field_far_fp64(fc, Rinv, st, tk, qc, qv, K, F);
                } else {
                    if constexpr (MIX)
                        return field_mixed(xc, st, tk, qv2, K, F);
                    else
                        return field_fp64(xc, st, tk, qc, qv, K, F);
                }
            };
            T Fp[6];  // the previous state's field (HOLD != 0)
            double u_prev;
            if constexpr (HOLD != 0)
                u_prev = field_at(sh.rec[g][0], sh.tk[0], Fp);
            else
                u_prev = slot_of(sh.rec[g][0], sh.tk[0]);
            // states 1 .. len through segment(); with the large ring the next state's
            // record is read from LDS while this one is worked on (two waves per SIMD
            // hide little of the LDS latency)
            auto walk = [&](auto&& segment) {
                if constexpr (kPrefetch) {
                    Rec cur = sh.rec[g][1];
                    double t_cur = sh.tk[1];
                    for (int k = 1; k <= len; ++k) {
                        const int kn = min(k + 1, len);
                        const Rec nxt = sh.rec[g][kn];
                        const double t_nxt = sh.tk[kn];
                        segment(cur, t_cur);
                        cur = nxt;
                        t_cur = t_nxt;
                    }
                } else {
                    for (int k = 1; k <= len; ++k)
                        segment(sh.rec[g][k], sh.tk[k]);
                }
            };
            // (a closure: written out in place, the small ring's mixed kernel took 104
            // registers instead of 94, four wavefronts a SIMD instead of five, and 5000
            // electrons x 128 steps x 64 x 64 cells 7.98 ms instead of 7.47)
            auto deposit_run = [&] {
                Sink sink{my_ring, row, base, n_t, &n_bypass};
                Carry<T> C;
                // open the slot where the run starts (a start far outside the window
                // leaves the first segment to the general path)
                const bool inside = u_prev >= -1.0 && u_prev < ntd + 1.0;
                carry_open(C, inside ? floor(u_prev) : (double)(INT_MIN / 2));
                C.lim = fast_limit(C.J1 - 1.0, u_prev, ntd);
                // segment k: the field of state k, held (or interpolated) over its arrivals
                walk([&](const Rec& st, double tk) {
                    T F[6];
                    const double uk = field_at(st, tk, F);
                    if constexpr (HOLD == 0) {
                        add_segment(C, sink, n_t, u_prev, uk, F, n_back, n_clip);
                    } else {
                        if constexpr (HOLD == 1)
                            add_segment(C, sink, n_t, u_prev, uk, Fp, n_back, n_clip);
                        else
                            add_segment_linear(C, sink, n_t, u_prev, uk, Fp, F, n_back, n_clip);
#pragma unroll
                        for (int c = 0; c < 6; ++c)
                            Fp[c] = F[c];
                    }
                    u_prev = uk;
                });
                sink.flush((int)(C.J1 - 1.0), C.V);
            };
            deposit_run();
        }
        if constexpr (kPrefetch) {
            if (scout_next)
                scout(xs_next, rb1 * L, buf ^ 1);
            p_stage = p_next;
            p_next = p_stage_after;
            p_scout = p_scout_after;
        }
        __syncthreads();  // records and rings are free for the next batch
        rb = rb1;
        bt = bt1;
        rb1 = rb2;
        bt1 = bt2;
    }
    move_rings(0, true);  // flush what the rings still hold
    if (n_clip)
        atomicAdd(&sh.cnt[0], (unsigned long long)n_clip);
    if (n_back)
        atomicAdd(&sh.cnt[1], (unsigned long long)n_back);
    if (n_bypass)
        atomicAdd(&sh.cnt[2], (unsigned long long)n_bypass);
    if (n_large)
        atomicAdd(&sh.cnt[3], (unsigned long long)n_large);
    __syncthreads();
    if (tid < kCounters && sh.cnt[tid])
        __hip_atomic_fetch_add(gptr(J.counters) + tid, sh.cnt[tid], __ATOMIC_RELAXED,
                               __HIP_MEMORY_SCOPE_AGENT);
}

// deposit_item with the slot-coordinate form of the job (the single-precision
// modes have one)
template <int M, int R, int G, int HOLD, int SH>
__device__ __forceinline__ void deposit_item_of(const DepositJob& J, int64_t tile, int64_t split,
                                                int64_t part, int sel,
                                                DepositShared<M, R, SH>& sh)
{
    if constexpr (M == kModeF64) {
        if (J.slot_div)
            deposit_item<M, R, G, HOLD, SH, true>(J, tile, split, part, sel, sh);
        else
            deposit_item<M, R, G, HOLD, SH, false>(J, tile, split, part, sel, sh);
    } else {
        deposit_item<M, R, G, HOLD, SH, false>(J, tile, split, part, sel, sh);
    }
}

// The work items item0 + [0, gridDim.x) of a single deposit, item =
// split * n_tiles + tile, one per workgroup (gridDim.x is a multiple of
// kXcds); items whose tile takes the other ring size leave at once.
// Waves per SIMD to ask of the register allocator.  A mixed-precision kernel with
// the small ring fits five wavefronts per SIMD in 96 VGPRs (its LDS allows five
// workgroups per CU).  For the exact-geometry, current-state kernel the
// allocator stays within that by itself and its own schedule is the faster
// one; the far-field, acceleration-only and held-field kernels go a few
// registers over, and keeping them at five waves (at the cost of a few spilled
// words in the hold kernels) is 4-6% faster on the undulator ensemble.  The
// double kernels are held to four workgroups per CU by their LDS; with both
// forms of the slot coordinate compiled in (see deposit_item_of) the default
// and previous-state kernels go a few registers over 128 by themselves and fit
// them on request (the previous-state hold with two spilled words), the linear
// hold would spill heavily and is left alone.  The other shapes: the 16-cell
// tile with runs of 8 segments has the LDS for five (single) or four (double)
// waves and is asked for them; the 8-cell tile's LDS allows three.
template <int M, int R, int G, int HOLD, int SH>
constexpr int kMinWaves =
    R != kRingSmall                      ? 1
    : SH == 1                            ? 1
    : M != kModeF64 && (G != 0 || HOLD != 0 || SH == 2) ? 5
    : M == kModeF64 && HOLD != 2         ? 4
                                         : 1;

template <int M, int R, int G, int HOLD, int SH>
__global__ __launch_bounds__(kDepositThreads)
__attribute__((amdgpu_waves_per_eu(kMinWaves<M, R, G, HOLD, SH>))) void deposit_kernel(
    DepositJob J, int64_t item0)
{
    __shared__ __align__(16) DepositShared<M, R, SH> sh;
    // Workgroups are dealt round-robin over the XCDs; give each XCD a contiguous
    // range of items, so that the workgroups resident on one XCD work on
    // neighbouring tiles of the same runs, whose records and particle orders
    // are alike, and share that XCD's L2.
    const int64_t per_xcd = (int64_t)gridDim.x / kXcds;
    const int64_t logical =
        item0 + (int64_t)(blockIdx.x % kXcds) * per_xcd + blockIdx.x / kXcds;
    if (logical >= J.n_tiles * J.n_splits * J.n_parts)
        return;
    const int64_t tile = logical % J.n_tiles;
    const int sel = ring_of(J, tile);
    if ((sel != kRingSel16) != (R == kRingLarge))
        return;
    const int64_t rest = logical / J.n_tiles;  // split-major, then part
    deposit_item_of<M, R, G, HOLD, SH>(J, tile, rest / J.n_parts, rest % J.n_parts, sel, sh);
}

// Persistent workgroups for many independent deposits: each takes the next work
// item (largest first, as ordered by the host) from a device counter until
// the list is exhausted, so uneven jobs share one launch without a tail of idle
// workgroups; items whose tile takes the other ring size are skipped.  Every
// workgroup leaves once the counter passes n_items.
// (The persistent loop costs registers: every single-precision variant with the
// small ring goes over 96 VGPRs by itself, and five waves per SIMD, with a few
// spilled words, make the 64-set batched benchmark 1.2% faster; the double
// small-ring variants are asked for the four waves their LDS allows.)
template <int M, int R, int G, int HOLD, int SH>
constexpr int kPersistentWaves = R != kRingSmall || SH == 1           ? 1
                                 : M != kModeF64                      ? 5
                                 : HOLD != 2                          ? 4
                                                                      : 1;

template <int M, int R, int G, int HOLD, int SH>
__global__ __launch_bounds__(kDepositThreads)
__attribute__((amdgpu_waves_per_eu(kPersistentWaves<M, R, G, HOLD, SH>))) void
deposit_persistent_kernel(
    const DepositJob* __restrict__ jobs, const WorkItem* __restrict__ items, int64_t n_items,
    unsigned long long* __restrict__ next, const unsigned long long* __restrict__ used)
{
    if (gptr(used)[R == kRingLarge ? 1 : 0] == 0)
        return;  // no job has a tile for this ring: each item would be claimed only to be left
    __shared__ __align__(16) DepositShared<M, R, SH> sh;
    __shared__ int64_t cur;
    for (;;) {
        __syncthreads();  // everyone has read the previous `cur`
        if (threadIdx.x == 0)
            cur = (int64_t)atomicAdd(next, 1ull);
        __syncthreads();
        const int64_t it = cur;
        if (it >= n_items)
            break;
        const WorkItem w = items[it];
        const DepositJob J = jobs[w.job];
        const int sel = ring_of(J, w.tile);
        if ((sel != kRingSel16) != (R == kRingLarge))
            continue;
        deposit_item_of<M, R, G, HOLD, SH>(J, w.tile, w.split, w.part, sel, sh);
    }
}

// ---------------------------------------------------------------------------
// few particles
// ---------------------------------------------------------------------------

// A chunk of a few particles leaves the particle lanes of deposit_kernel idle, and
// its four launches cost more than the work.  Here the lanes of a wavefront take
// consecutive states of one particle: lane l > 0 the segment from lane l - 1's
// state to its own, so that a state is evaluated once and its neighbour's arrival
// and beta come by a shuffle.  A wavefront keeps its states' kinematics (formed
// here, as kinematics_kernel forms them) in registers over kFewCells cells and all
// of the chunk's particles; for each cell its lanes add their slots into an LDS window of
// kFewWindow slots, which then goes to the detector as contiguous adds (2.5e10
// slots/s against 3.8e9 for a lane adding a slot's six words).  One launch, no
// workspace.  Bound by the latency of a wavefront's chain (field, LDS adds, flush) and,
// with several slots a segment, by the adds to HBM.  Measured, whole deposits: one
// electron x 2000 steps x 32 x 32 cells x 512 slots 163 -> 35 us, 25133 steps x 256
// cells x 65536 slots 1.3 -> 0.55 ms.
constexpr int kFewWindow = 192;  // slots; 64 segments of up to three slots, four workgroups a CU

template <int M, bool DIV>
__global__ __launch_bounds__(256) void few_kernel(DepositJob J, int64_t n_slabs, int64_t n_groups,
                                                  int cells_each)
{
    constexpr bool MIX = ModeTypes<M>::MIX;
    using T = typename ModeTypes<M>::T;
    using Acc = typename ModeTypes<M>::Acc;
    using Rec = typename ModeTypes<M>::Rec;
    __shared__ double window[4][kFewWindow * 6];
    const int lane = threadIdx.x % 64;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / 64);
    RADIO_LDS double* win = (RADIO_LDS double*)&window[wave][0];
    for (int i = lane; i < kFewWindow * 6; i += 64)
        win[i] = 0.0;
    const double ntd = (double)J.n_t;
    const Consts K{J.t0, J.inv_dt_det, J.inv_c, J.inv_c * J.inv_dt_det, J.dt_det, DIV};
    unsigned long long n_clip = 0, n_back = 0;  // of the wavefront
    for (int64_t task = (int64_t)blockIdx.x * 4 + wave; task < n_slabs * n_groups;
         task += (int64_t)gridDim.x * 4) {
        const int64_t slab = task / n_groups;
        const int64_t c_begin = (task - slab * n_groups) * cells_each;
        const int64_t c_end = min(c_begin + cells_each, J.n_c);
        const int64_t s = slab * 63 + lane;  // the lane's state
        const bool state = s <= J.n_s;
        const bool segment = state && lane > 0;
        const double sk = (double)(J.s0 + s);
        double tk;  // the field functions' time argument
        if constexpr (MIX)
            tk = fma(sk, J.dt * J.inv_dt_det, (J.t_first - J.t0) * J.inv_dt_det);
        else
            tk = canon_state_time(J.t_first, sk, J.dt);
        for (int64_t p = 0; p < J.n_p; ++p) {
            const int64_t off = (state ? s : J.n_s) * J.n_p + p;
            Rec st;
            double b[3], g2i;
    #pragma unroll
            for (int c = 0; c < 3; ++c)
                st.x[c] = gptr(J.x)[off + c * J.xs_stride];
            canon_kinematics(gptr(J.u)[off], gptr(J.u)[off + J.xs_stride],
                             gptr(J.u)[off + 2 * J.xs_stride], b, &g2i);
            const double q = J.q ? gptr(J.q)[p] : -1.0;
    #pragma unroll
            for (int c = 0; c < 3; ++c) {
                st.b[c] = b[c];
                const double bd = canon_betadot(b[c], __shfl_up(b[c], 1), J.dt);
                if constexpr (MIX)
                    st.bdq[c] = (float)((q * J.inv_c) * bd);
                else
                    st.bd[c] = bd;
            }
            if constexpr (MIX)
                st.g2ih = (float)(0.5 * g2i);
            else
                st.g2i = g2i;
            for (int64_t cell = c_begin; cell < c_end; ++cell) {
                const double* cp = J.cells + 3 * cell;
                const double xc[3] = {cp[0], cp[1], cp[2]};
                T F[6];
                double u;
                if constexpr (MIX)
                    u = field_mixed(xc, st, tk, T(2.0 * q * J.vscale), K, F);
                else
                    u = field_fp64(xc, st, tk, T(q * J.inv_c), T(q * J.vscale), K, F);
                const double a = __shfl_up(u, 1);
                double lo = 0.0, hi = 0.0;
                clamp_segment(a, u, ntd, lo, hi);
                const bool adds = segment && lo < hi;  // else empty, entirely outside, or NaN
                n_back += (unsigned)__popcll(__ballot(segment && u < a));
                n_clip += (unsigned)__popcll(__ballot(segment && clipped(a, u, ntd) != 0u));
                int j = adds ? (int)lo : INT_MAX;
                const int j_end = adds ? (int)ceil(hi) : -1;  // past the last slot touched
                // the slots the wavefront touches: as the arrivals advance with the lanes,
                // from the first lane's to the last one's (else the extremes)
                const unsigned long long on = __ballot(adds);
                if (on == 0)
                    continue;
                int w_lo = __builtin_amdgcn_readlane(j, __builtin_ctzll(on));
                int w_hi = __builtin_amdgcn_readlane(j_end, 63 - __builtin_clzll(on));
                if (__ballot(adds && (j < w_lo || j_end > w_hi)) != 0) {
                    w_lo = j;
                    w_hi = j_end;
                    for (int m = 32; m > 0; m >>= 1) {
                        w_lo = min(w_lo, __shfl_xor(w_lo, m));
                        w_hi = max(w_hi, __shfl_xor(w_hi, m));
                    }
                    w_lo = __builtin_amdgcn_readfirstlane(w_lo);
                    w_hi = __builtin_amdgcn_readfirstlane(w_hi);
                }
                // few slots: as many copies of them as fit (at most 16), one per lane in
                // turn, so that the lanes of one slot do not queue at one address
                const int words = min(w_hi - w_lo, kFewWindow) * 6;
                int copies = 1;
                while (copies < 16 && 2 * copies * (words + 1) <= kFewWindow * 6)
                    copies *= 2;
                RADIO_LDS double* mine = win + (lane & (copies - 1)) * (words + 1);
                RADIO_GLOBAL Acc* row = gptr(reinterpret_cast<Acc*>(J.acc + cell * J.n_t * 6));
                for (int w0 = w_lo; w0 < w_hi; w0 += kFewWindow) {
                    const int w1 = min(w0 + kFewWindow, w_hi);
                    for (; j < min(j_end, w1); ++j) {
                        const double jd = (double)j;
                        const T wt = T(fmin(hi, jd + 1.0) - fmax(lo, jd));
                        RADIO_LDS double* slot = mine + (j - w0) * 6;
    #pragma unroll
                        for (int k = 0; k < 6; ++k)
                            __hip_atomic_fetch_add(slot + k, (double)(F[k] * wt), __ATOMIC_RELAXED,
                                                   __HIP_MEMORY_SCOPE_WORKGROUP);
                    }
                    // the window is this wavefront's: its LDS accesses are done in order
                    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
                    for (int i = lane; i < (w1 - w0) * 6; i += 64) {
                        double v = 0.0;
                        for (int c = 0; c < copies; ++c) {
                            v += win[c * (words + 1) + i];
                            win[c * (words + 1) + i] = 0.0;
                        }
                        if (v != 0.0)
                            global_add_one(row, w0 + i / 6, i % 6, v);
                    }
                    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
                }
            }
        }
    }
    if (lane == 0 && n_clip)
        __hip_atomic_fetch_add(gptr(J.counters), n_clip, __ATOMIC_RELAXED,
                               __HIP_MEMORY_SCOPE_AGENT);
    if (lane == 0 && n_back)
        __hip_atomic_fetch_add(gptr(J.counters) + 1, n_back, __ATOMIC_RELAXED,
                               __HIP_MEMORY_SCOPE_AGENT);
}

// E and B from the slot accumulator: E[c][j][0..2] and B[c][j][0..2] for the
// caller's cell index c of internal row r.  The compensated single
// accumulator holds (hi, lo) pairs, folded to double.  One thread per slot.
template <bool PAIRS>
__global__ __launch_bounds__(256) void readout_kernel(const double* __restrict__ acc, int64_t n_c,
                                                      int64_t n_t,
                                                      const int64_t* __restrict__ user_index,
                                                      double* __restrict__ E,
                                                      double* __restrict__ B)
{
    const int64_t total = n_c * n_t;
    for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < total;
         i += (int64_t)gridDim.x * blockDim.x) {
        const int64_t r = i / n_t;
        const int64_t j = i - r * n_t;
        double v[6];
        if (PAIRS) {
            const float* q = reinterpret_cast<const float*>(acc) + i * 12;
#pragma unroll
            for (int k = 0; k < 6; ++k)
                v[k] = (double)q[k] + (double)q[6 + k];
        } else {
#pragma unroll
            for (int k = 0; k < 6; ++k)
                v[k] = acc[i * 6 + k];
        }
        const int64_t o = (user_index[r] * n_t + j) * 3;
        if (E) {
            E[o] = v[0];
            E[o + 1] = v[1];
            E[o + 2] = v[2];
        }
        if (B) {
            B[o] = v[3];
            B[o + 1] = v[4];
            B[o + 2] = v[5];
        }
    }
}

// a detector's slots and counters in one launch
__global__ void reset_kernel(double* p, int64_t n, unsigned long long* counters)
{
    if (blockIdx.x == 0 && threadIdx.x < kCounters)
        counters[threadIdx.x] = 0ull;
    for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < n;
         i += (int64_t)gridDim.x * blockDim.x)
        p[i] = 0.0;
}

__global__ void zero_u64_kernel(unsigned long long* p, int64_t n)
{
    for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < n;
         i += (int64_t)gridDim.x * blockDim.x)
        p[i] = 0ull;
}

__global__ void arrival_kernel(const double* cells, const double* pts, const double* t, int64_t n,
                               double inv_c, double* out)
{
    const int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
    if (i < n) {
        double d0 = cells[3 * i] - pts[3 * i];
        double d1 = cells[3 * i + 1] - pts[3 * i + 1];
        double d2 = cells[3 * i + 2] - pts[3 * i + 2];
        out[i] = canon_arrival(t[i], canon_sqrt(canon_norm2(d0, d1, d2)), inv_c);
    }
}

// slot coordinates (t + |x_cell - x|/c - t0) / dt_det of explicit triples, as the
// double deposit rounds them
__global__ void slot_coord_kernel(const double* cells, const double* pts, const double* t,
                                  int64_t n, double inv_c, double t0, double dt_det,
                                  double inv_dt_det, int slot_div, double* out)
{
    const int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
    if (i < n) {
        double d0 = cells[3 * i] - pts[3 * i];
        double d1 = cells[3 * i + 1] - pts[3 * i + 1];
        double d2 = cells[3 * i + 2] - pts[3 * i + 2];
        const double tau = canon_arrival(t[i], canon_sqrt(canon_norm2(d0, d1, d2)), inv_c);
        out[i] = canon_slot(tau, t0, dt_det, inv_dt_det, slot_div != 0);
    }
}

}  // namespace

// workgroups of one launch: what has more of them runs in several (a launch takes fewer
// than 2^32 threads)
constexpr int64_t kMaxDepositGrid = int64_t(1) << 22;

void set_shape(DepositJob& job, int shape)
{
    job.shape = shape;
    job.tile_cells = shape_cells(shape);
    job.groups = shape_groups(shape);
    job.run_l = shape_run(shape);
}

void plan_job(DepositJob& job, int target_blocks, int64_t capacity)
{
    job.n_runs = (job.n_s + job.run_l - 1) / job.run_l;
    job.n_tiles = (job.n_c + job.tile_cells - 1) / job.tile_cells;
    int64_t splits = 1;
    if (target_blocks > 0) {
        splits = (target_blocks + job.n_tiles - 1) / job.n_tiles;
    } else {
        // short items (at least kMinItemBatches batches, so that an item's
        // set-up and final ring flush stay small), unless that leaves fewer
        // items than the device holds at once
        const int64_t n_batches = std::max<int64_t>((job.n_p + job.groups - 1) / job.groups, 1);
        const int64_t rps = std::max<int64_t>(1, (kMinItemBatches + n_batches - 1) / n_batches);
        splits = (job.n_runs + rps - 1) / rps;
        if (job.n_tiles * splits < capacity)
            splits = job.n_runs;
    }
    if (splits < 1)
        splits = 1;
    if (splits > job.n_runs)
        splits = job.n_runs;
    job.runs_per_split = (job.n_runs + splits - 1) / splits;
    job.n_splits = (job.n_runs + job.runs_per_split - 1) / job.runs_per_split;
    // few runs (a short chunk): ranges of the sorted particles as well
    const int64_t n_batches = std::max<int64_t>((job.n_p + job.groups - 1) / job.groups, 1);
    int64_t parts = 1;
    const int64_t items = job.n_tiles * job.n_splits;
    if (target_blocks <= 0 && items < 2 * capacity) {
        parts = (2 * capacity + items - 1) / items;
        parts = std::max<int64_t>(1, std::min<int64_t>(parts, n_batches / 4));
    }
    set_parts(job, parts);
}

int64_t max_order_groups(const DepositJob& job, size_t rec_bytes, int64_t budget_mib)
{
    const double per_group = (double)job.n_tiles * (double)job.n_p * sizeof(int32_t);
    const double budget =
        budget_mib > 0 ? (double)budget_mib * (double)(int64_t(1) << 20)
                       : std::max((double)(job.n_s + 1) * (double)job.n_p * (double)rec_bytes,
                                  (double)(int64_t(1) << 30));
    return (int64_t)std::max(1.0, std::min(budget / per_group, (double)INT32_MAX));
}

void set_groups(DepositJob& job, int64_t max_groups)
{
    int64_t groups = std::min(job.n_runs, std::max<int64_t>(1, max_groups));
    // a few batches gain nothing from re-sorting, and each order costs a histogram
    if (job.n_p < min_group_particles(job))
        groups = 1;
    groups = std::max<int64_t>(1, groups);
    const int64_t want = (job.n_runs + groups - 1) / groups;
    job.group_shift = 0;
    while ((int64_t(1) << job.group_shift) < want)
        ++job.group_shift;
    job.runs_per_group = int64_t(1) << job.group_shift;
    job.n_groups = (job.n_runs + job.runs_per_group - 1) / job.runs_per_group;
}

void set_parts(DepositJob& job, int64_t parts)
{
    const int64_t n_batches = std::max<int64_t>((job.n_p + job.groups - 1) / job.groups, 1);
    parts = std::max<int64_t>(1, std::min<int64_t>(parts, n_batches));
    job.batches_per_part = (n_batches + parts - 1) / parts;
    job.n_parts = (n_batches + job.batches_per_part - 1) / job.batches_per_part;
}

hipError_t launch_reset(double* p, int64_t n, unsigned long long* counters, hipStream_t s)
{
    const int64_t blocks = std::max<int64_t>(1, std::min<int64_t>((n + 255) / 256, 8192));
    hipLaunchKernelGGL(reset_kernel, dim3((unsigned)blocks), dim3(256), 0, s, p, n, counters);
    return hipGetLastError();
}

hipError_t launch_zero_u64(unsigned long long* p, int64_t n, hipStream_t s)
{
    if (n <= 0)
        return hipSuccess;
    hipLaunchKernelGGL(zero_u64_kernel, dim3(1), dim3(64), 0, s, p, n);
    return hipGetLastError();
}

hipError_t launch_kinematics(const DepositJob& job, int mode, hipStream_t s)
{
    const int64_t total = job.n_p * (job.n_s + 1);
    int64_t blocks = (total + 255) / 256;
    if (blocks > 65536)
        blocks = 65536;
    const int rule = job.hold == 2 ? kBdCentred : (job.hold == 1 ? kBdBackwardFirst : kBdBackward);
    if (mode == kModeF64)
        hipLaunchKernelGGL(kinematics_kernel<kModeF64>, dim3((unsigned)blocks), dim3(256), 0, s,
                           job.x, job.u, job.q, job.n_p, job.n_s, job.xs_stride, -job.s_before,
                           job.n_s + job.s_after, job.dt, job.inv_c, rule, job.recs, job.rings);
    else
        hipLaunchKernelGGL(kinematics_kernel<kModeMix>, dim3((unsigned)blocks), dim3(256), 0, s,
                           job.x, job.u, job.q, job.n_p, job.n_s, job.xs_stride, -job.s_before,
                           job.n_s + job.s_after, job.dt, job.inv_c, rule, job.recs, job.rings);
    return hipGetLastError();
}

hipError_t launch_order(const DepositJob& job, hipStream_t s)
{
    auto kernel = job.n_p <= 256 * kOrderHeld ? order_kernel<true> : order_kernel<false>;
    // a long chunk has an order per tile for every run or two of it
    const int64_t n_items = job.n_tiles * job.n_groups;
    for (int64_t item0 = 0; item0 < n_items; item0 += kMaxDepositGrid)
        hipLaunchKernelGGL(kernel,
                           dim3((unsigned)std::min<int64_t>(n_items - item0, kMaxDepositGrid)),
                           dim3(256), 0, s, job.x, job.n_p, job.n_s, job.xs_stride, job.n_tiles,
                           (int64_t)job.tile_cells, job.runs_per_group * job.run_l, job.cells,
                           job.n_c, job.inv_c, job.inv_dt_det, job.perm, item0);
    return hipGetLastError();
}

hipError_t launch_ring_choice(const DepositJob& job, int mode, hipStream_t s)
{
    if (job.n_tiles <= 0)
        return hipSuccess;
    const int64_t each = (job.n_tiles + kChoiceBlocks - 1) / kChoiceBlocks;
    const dim3 grid((unsigned)((job.n_tiles + each - 1) / each));
    RingCost cost = kRingCost[mode];
    if (job.hold == 2) {
        cost.small += kLinearField;
        cost.large += kLinearField;
    }
    auto kernel = job.run_l == 16 ? ring_choice_kernel<16> : ring_choice_kernel<8>;
    hipLaunchKernelGGL(kernel, grid, dim3(256), 0, s, job, (int64_t)rec_bytes(mode), cost, each);
    return hipGetLastError();
}

// kernel variants (kernel_variant): precision mode x geometry/quantity (far
// field, potentials) x hold rule for the default shape; precision mode for the
// other shapes with the default options; each with both ring sizes
template <int V>
struct VariantOf {
    static constexpr bool kOpt = V < kOptionVariants;
    static constexpr int M = kOpt ? V % 3 : (V - kOptionVariants) % 3;
    static constexpr int G = kOpt ? (V / 3) % 4 : 0;
    static constexpr int HOLD = kOpt ? V / 12 : 0;
    static constexpr int SH = kOpt ? 0 : 1 + (V - kOptionVariants) / 3;
};

template <int V>
static void launch_deposit_index(const DepositJob& job, dim3 grid, hipStream_t s)
{
    using K = VariantOf<V>;
    // more items than one launch holds run in several launches
    const int64_t n_items = job.n_tiles * job.n_splits * job.n_parts;
    for (int64_t item0 = 0; item0 < n_items; item0 += grid.x)
        hipLaunchKernelGGL((deposit_kernel<K::M, kRingSmall, K::G, K::HOLD, K::SH>), grid,
                           dim3(kDepositThreads), 0, s, job, item0);
    for (int64_t item0 = 0; item0 < n_items; item0 += grid.x)
        hipLaunchKernelGGL((deposit_kernel<K::M, kRingLarge, K::G, K::HOLD, K::SH>), grid,
                           dim3(kDepositThreads), 0, s, job, item0);
}

template <int V>
static void launch_persistent_index(const DepositJob* jobs, const WorkItem* items,
                                    int64_t n_items, unsigned long long* next,
                                    const unsigned long long* used, int blocks_small,
                                    int blocks_large, hipStream_t s)
{
    using K = VariantOf<V>;
    hipLaunchKernelGGL((deposit_persistent_kernel<K::M, kRingSmall, K::G, K::HOLD, K::SH>),
                       dim3((unsigned)blocks_small), dim3(kDepositThreads), 0, s, jobs, items,
                       n_items, next, used);
    hipLaunchKernelGGL((deposit_persistent_kernel<K::M, kRingLarge, K::G, K::HOLD, K::SH>),
                       dim3((unsigned)blocks_large), dim3(kDepositThreads), 0, s, jobs, items,
                       n_items, next + 1, used);
}

template <int V>
static int blocks_per_cu_index(bool large_ring)
{
    int n = 0;
    using K = VariantOf<V>;
    const void* f =
        large_ring
            ? reinterpret_cast<const void*>(
                  deposit_persistent_kernel<K::M, kRingLarge, K::G, K::HOLD, K::SH>)
            : reinterpret_cast<const void*>(
                  deposit_persistent_kernel<K::M, kRingSmall, K::G, K::HOLD, K::SH>);
    const hipError_t e = hipOccupancyMaxActiveBlocksPerMultiprocessor(&n, f, kDepositThreads, 0);
    return (e == hipSuccess && n > 0) ? n : 1;
}

template <int... V>
struct VariantTable {
    using Single = void (*)(const DepositJob&, dim3, hipStream_t);
    using Launch = void (*)(const DepositJob*, const WorkItem*, int64_t, unsigned long long*,
                            const unsigned long long*, int, int, hipStream_t);
    using Occ = int (*)(bool);
    static constexpr Single single[] = {&launch_deposit_index<V>...};
    static constexpr Launch launch[] = {&launch_persistent_index<V>...};
    static constexpr Occ occupancy[] = {&blocks_per_cu_index<V>...};
};
template <int... V>
constexpr VariantTable<V...> make_table(std::integer_sequence<int, V...>)
{
    return {};
}
using Variants = decltype(make_table(std::make_integer_sequence<int, kKernelVariants>{}));

hipError_t launch_deposit(const DepositJob& job, int mode, int64_t max_grid, hipStream_t s)
{
    int64_t blocks = job.n_tiles * job.n_splits * job.n_parts;
    if (blocks <= 0)
        return hipSuccess;
    blocks = (blocks + kXcds - 1) / kXcds * kXcds;  // a multiple of the XCD count
    // more items than max_grid (and kMaxDepositGrid) run in several launches
    const int64_t cap = std::max<int64_t>(kXcds, std::min<int64_t>(max_grid, kMaxDepositGrid));
    blocks = std::min<int64_t>(blocks, cap / kXcds * kXcds);
    const int v = kernel_variant(mode, job);
    if (v < 0 || v >= kKernelVariants)
        return hipErrorInvalidValue;
    Variants::single[v](job, dim3((unsigned)blocks), s);
    return hipGetLastError();
}

bool few_particles(const DepositJob& job)
{
    if (job.n_p > kFewParticles || job.hold != 0 || job.potentials || job.far)
        return false;
    // dense: slots of several steps, or more segments than the window's slots can take
    const bool dense = job.dt_det >= kFewDense * job.dt || job.n_s >= kFewCrowded * job.n_t;
    return job.n_p <= kFewAlways || !dense ||
           (double)job.n_p * (double)job.n_s * (double)job.n_c <=
               kFewWork[job.n_p - kFewAlways - 1];
}

hipError_t launch_few(const DepositJob& job, int mode, int64_t n_cus, hipStream_t s)
{
    const int64_t n_slabs = (job.n_s + 62) / 63;
    // cells a wavefront takes: while sixteen wavefronts a CU remain
    const int64_t each =
        std::max<int64_t>(1, std::min<int64_t>(kFewCells, n_slabs * job.n_c / (16 * n_cus)));
    const int64_t n_groups = (job.n_c + each - 1) / each;
    const dim3 grid(
        (unsigned)std::min<int64_t>((n_slabs * n_groups + 3) / 4, kMaxDepositGrid));
    if (mode == kModeF64 && job.slot_div)
        hipLaunchKernelGGL((few_kernel<kModeF64, true>), grid, dim3(256), 0, s, job, n_slabs,
                           n_groups, (int)each);
    else if (mode == kModeF64)
        hipLaunchKernelGGL((few_kernel<kModeF64, false>), grid, dim3(256), 0, s, job, n_slabs,
                           n_groups, (int)each);
    else if (mode == kModeMix)
        hipLaunchKernelGGL((few_kernel<kModeMix, false>), grid, dim3(256), 0, s, job, n_slabs,
                           n_groups, (int)each);
    else
        hipLaunchKernelGGL((few_kernel<kModeMixTwoSum, false>), grid, dim3(256), 0, s, job,
                           n_slabs, n_groups, (int)each);
    return hipGetLastError();
}

hipError_t launch_deposit_batch(const DepositJob* jobs, const WorkItem* items, int64_t n_items,
                                unsigned long long* next, const unsigned long long* used,
                                int variant, int blocks_small, int blocks_large, hipStream_t s)
{
    if (n_items <= 0)
        return hipSuccess;
    if (variant < 0 || variant >= kKernelVariants)
        return hipErrorInvalidValue;
    Variants::launch[variant](jobs, items, n_items, next, used, blocks_small, blocks_large, s);
    return hipGetLastError();
}

int persistent_blocks_per_cu(int variant, bool large_ring)
{
    if (variant < 0 || variant >= kKernelVariants)
        return 1;
    // a property of the code object: asked once per kernel
    static std::atomic<int> known[kKernelVariants][2];
    const int r = large_ring ? 1 : 0;
    int n = known[variant][r].load(std::memory_order_relaxed);
    if (n <= 0) {
        n = Variants::occupancy[variant](large_ring);
        known[variant][r].store(n, std::memory_order_relaxed);
    }
    return n;
}

hipError_t launch_readout(const double* acc, int64_t n_c, int64_t n_t, const int64_t* user_index,
                          bool pairs, double* E, double* B, hipStream_t s)
{
    if (n_c <= 0)
        return hipSuccess;
    int64_t blocks = (n_c * n_t + 255) / 256;
    if (blocks > 65536)
        blocks = 65536;
    if (pairs)
        hipLaunchKernelGGL(readout_kernel<true>, dim3((unsigned)blocks), dim3(256), 0, s, acc, n_c,
                           n_t, user_index, E, B);
    else
        hipLaunchKernelGGL(readout_kernel<false>, dim3((unsigned)blocks), dim3(256), 0, s, acc, n_c,
                           n_t, user_index, E, B);
    return hipGetLastError();
}

hipError_t launch_arrival(const double* cells, const double* pts, const double* t, int64_t n,
                          double inv_c, double* out, hipStream_t s)
{
    if (n <= 0)
        return hipSuccess;
    hipLaunchKernelGGL(arrival_kernel, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, s, cells,
                       pts, t, n, inv_c, out);
    return hipGetLastError();
}

hipError_t launch_slot_coords(const double* cells, const double* pts, const double* t, int64_t n,
                              double inv_c, double t0, double dt_det, double inv_dt_det,
                              bool slot_div, double* out, hipStream_t s)
{
    if (n <= 0)
        return hipSuccess;
    hipLaunchKernelGGL(slot_coord_kernel, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, s, cells,
                       pts, t, n, inv_c, t0, dt_det, inv_dt_det, slot_div ? 1 : 0, out);
    return hipGetLastError();
}

}  // namespace radio
