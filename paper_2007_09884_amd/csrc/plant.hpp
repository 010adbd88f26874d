// Device-side model of the 18-parameter oculomotor plant (arXiv 2007.09884,
// Section 2.1 and Section 2.2.1 / Table 1) for one candidate per lane.
//
// Units: time in ms (viscosities scaled by 1e3, inertia by 1e6 from Table 1's
// second-based units), angles in degrees, forces in grams.
//
// State x = (theta, omega, x_ag, x_ant, F_ag, F_ant).  The plant is linear and
// time-invariant on each piece of the pulse-step control (pulse on [0, PW)
// with the activation time constants, step afterwards with the deactivation
// time constants), so one sample period dt advances the deviation from the
// piece's equilibrium by a fixed matrix: d_{k+1} = Phi d_k (run_blocks advances
// four samples at a time, with Phi^4 and the theta rows of Phi^1..Phi^3).
// Phi = exp(A dt) is a Taylor polynomial of A on a fraction of the sample, doubled
// up to it, carried as a polynomial of degree 3 in A ("Transitions as
// polynomials" below) in "D-form", D = Phi - I: storing Phi - I keeps the slow
// modes (|1 - mu| ~ 0.02 per ms) at full relative precision.  The recurrence type R
// is FP64 by default (FP32 stays buildable); candidates are FP32.  The sample
// that contains the pulse end is split exactly at PW with two Taylor
// exponential-vector products.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

namespace opmm {

constexpr int P = 18;

// keep(x): x is computed here.  Without it the compiler sinks what only the post piece reads (its
// coupling columns and rows) behind the pulse loop and keeps their operands live until then (with
// the doublings on matrices: 166 registers instead of 128 in the FP32 pass, 95 spilled instead of none
// in the FP64 kernels, an FP64 round of 256 x 65536 candidates 2.32 ms instead of 1.42).
template <class T>
__device__ __forceinline__ void keep(T& x)
{
#ifdef __HIP_DEVICE_COMPILE__
    asm volatile("" : "+v"(x));
#endif
}

// Precision of the per-sample recurrence and of the transition matrix.
#ifndef OPMM_REC_T
#define OPMM_REC_T double
#endif
using R = OPMM_REC_T;

__device__ __forceinline__ float fmr(float a, float b, float c) { return __fmaf_rn(a, b, c); }
__device__ __forceinline__ double fmr(double a, double b, double c) { return __fma_rn(a, b, c); }

// Taylor degree and squarings of the one-sample transition, and the degree of
// the exponential-vector product of the split sample, per precision: each
// set puts the truncation error below that precision's rounding floor over
// +/-25% boxes (FP64: ~5e-9 deg on 150-sample traces; FP32: the RMSE of a
// candidate stays within ~8e-6 deg of its FP64 value with degrees 7 and 6,
// as with 8 and 8, while a degree-6 transition doubles that).
// The scalar setup (matrix entries, equilibria) and the squared-residual sum
// run in FP64 for the FP64 recurrence; the FP32 recurrence screens candidates
// only, so its setup and sum stay in FP32 (the FP32 rate is twice the FP64
// rate on this chip) and their rounding joins the screening error budget.
#ifndef OPMM_F32_TAYLOR_M
#define OPMM_F32_TAYLOR_M 7
#endif
#ifndef OPMM_F32_EXPMV_M
#define OPMM_F32_EXPMV_M 6
#endif
template <class RT>
struct Prec {
    static constexpr int taylor_m = sizeof(RT) == 8 ? 6 : OPMM_F32_TAYLOR_M;
    static constexpr int taylor_sq = sizeof(RT) == 8 ? 2 : 0;
    static constexpr int expmv_m = sizeof(RT) == 8 ? 11 : OPMM_F32_EXPMV_M;
    using scalar = RT;  // type of plant_scalars
    using acc = RT;     // type of the squared-residual sum
};

// Table 1 nominal values, in the table's order and units.  The pulse width
// (index 17) is the saccade duration minus 6 ms.
__host__ __device__ inline float nominal_param(int j, float dur_ms)
{
    switch (j) {
    case 0: return 2.5f;       // K_SE_AG
    case 1: return 2.5f;       // K_SE_ANT
    case 2: return 1.2f;       // K_LT_AG
    case 3: return 1.2f;       // K_LT_ANT
    case 4: return 0.046f;     // B_AG
    case 5: return 0.022f;     // B_ANT
    case 6: return 0.06f;      // B_P
    case 7: return 0.8f;       // N_C_AG
    case 8: return 0.5f;       // N_C_ANT
    case 9: return 0.000043f;  // J
    case 10: return 11.7f;     // tau_AC_AG
    case 11: return 2.4f;      // tau_AC_ANT
    case 12: return 2.0f;      // tau_DE_AG
    case 13: return 1.9f;      // tau_DE_ANT
    case 14: return 14.0f;     // N_C_FIX
    case 15: return 55.0f;     // N_SAC_AG
    case 16: return 0.5f;      // N_SAC_ANT
    default: return dur_ms - 6.0f; // PW
    }
}

// Table 1 in FP64 (the decimal values as printed), for methods whose iterates
// live in FP64 relative to nominal.
__host__ __device__ inline double nominal_param_f64(int j, double dur_ms)
{
    switch (j) {
    case 0: return 2.5;
    case 1: return 2.5;
    case 2: return 1.2;
    case 3: return 1.2;
    case 4: return 0.046;
    case 5: return 0.022;
    case 6: return 0.06;
    case 7: return 0.8;
    case 8: return 0.5;
    case 9: return 0.000043;
    case 10: return 11.7;
    case 11: return 2.4;
    case 12: return 2.0;
    case 13: return 1.9;
    case 14: return 14.0;
    case 15: return 55.0;
    case 16: return 0.5;
    default: return dur_ms - 6.0;
    }
}

// ---------------------------------------------------------------------------
// Candidate stream
// ---------------------------------------------------------------------------

// SplitMix64 (Steele, Lea & Flood 2014): output n of the generator seeded
// with `seed` is mix(seed + n * golden_gamma).
__device__ __forceinline__ uint64_t splitmix64(uint64_t seed, uint64_t n)
{
    uint64_t z = seed + n * 0x9E3779B97F4A7C15ull;
    z = (z ^ (z >> 30)) * 0xBF58476D1CE4E5B9ull;
    z = (z ^ (z >> 27)) * 0x94D049BB133111EBull;
    return z ^ (z >> 31);
}

__device__ __forceinline__ uint64_t stream_counter(uint32_t round, uint32_t idx, uint32_t k)
{
    return 1ull + (((uint64_t)round << 36) | ((uint64_t)idx << 4) | (uint64_t)k);
}

// 24-bit uniform u -> s = u/2^23 - 1 (exact) -> clamp(fma(w, s, c)).
__device__ __forceinline__ float box_draw(uint32_t u, float c, float w, float lo, float hi)
{
    float s = __fmaf_rn((float)u, 0x1p-23f, -1.0f);
    float v = __fmaf_rn(w, s, c);
    return __builtin_amdgcn_fmed3f(v, lo, hi);  // = clamp to [lo, hi] (lo <= hi, v finite)
}

struct Box {
    float c[P], w[P], lo[P], hi[P];
};

// The 9-parameter model (Table 2) shares one series elasticity and one
// length-tension value between the muscles.
__host__ __device__ inline bool fixed_in_model9(int j) { return (j >= 10 && j <= 13) || j >= 15; }

// Full candidate `idx` of round `round` (index 0 is the centre).
__device__ __forceinline__ void draw_candidate(uint64_t seed, uint32_t round, uint32_t idx,
                                               const Box& b, float p[P], int model = 18)
{
#pragma unroll
    for (int k = 0; k < 9; ++k) {
        const uint64_t z = splitmix64(seed, stream_counter(round, idx, k));
        uint32_t ua = (uint32_t)(z >> 40);
        // seen as a shifted 64-bit value, ua would be converted to float as one (five more instructions a draw)
        keep(ua);
        const uint32_t ub = (uint32_t)(z >> 16) & 0xFFFFFFu;
        p[2 * k] = box_draw(ua, b.c[2 * k], b.w[2 * k], b.lo[2 * k], b.hi[2 * k]);
        p[2 * k + 1] = box_draw(ub, b.c[2 * k + 1], b.w[2 * k + 1], b.lo[2 * k + 1], b.hi[2 * k + 1]);
    }
    if (idx == 0) {
#pragma unroll
        for (int j = 0; j < P; ++j) p[j] = b.c[j];
    }
    if (model == 9) {
        p[1] = p[0];
        p[3] = p[2];
    }
}

// Only the pulse width of candidate idx (last draw, low half).
__device__ __forceinline__ float draw_pw(uint64_t seed, uint32_t round, uint32_t idx, const Box& b)
{
    uint64_t z = splitmix64(seed, stream_counter(round, idx, 8));
    uint32_t ub = (uint32_t)(z >> 16) & 0xFFFFFFu;
    float v = box_draw(ub, b.c[17], b.w[17], b.lo[17], b.hi[17]);
    return idx == 0 ? b.c[17] : v;
}

// ---------------------------------------------------------------------------
// Plant coefficients of one candidate
// ---------------------------------------------------------------------------

template <class RT>
struct PlantT {
    // system matrix entries per base step, omega per base step; theta' = omega is implicit
    RT a10, a11, a12, a13;      // omega row: theta, omega, x_ag, x_ant
    RT a20, a22, g2;            // x_ag row: theta, x_ag, F_ag
    RT a30, a33, g3;            // x_ant row: theta, x_ant, F_ant
    RT q[4];                    // F rows: -1/tau; pulse (ag, ant: activation), then post (deactivation)
    // transition of a number of samples in D-form (Phi - I), see run_blocks
    RT m[4][4];                 // mechanical block
    RT x[4][4];                 // coupling to F: pulse (ag, ant), then post (ag, ant)
    RT e[4];                    // F decay factor minus one: pulse (ag, ant), then post (ag, ant)
    // equilibria and switching
    RT th1;                     // theta at the pulse equilibrium
    RT amp;                     // theta at the post equilibrium (= amplitude)
    RT sh[6];                   // pulse equilibrium minus post equilibrium
    RT d0[6];                   // resting state minus pulse equilibrium
    double pwd;                // PW in sample periods
};
using Plant = PlantT<R>;

__device__ __forceinline__ float rcp(float x) { return __builtin_amdgcn_rcpf(x); }

// 1/x in FP64: hardware reciprocal refined by two Newton steps (the relative
// error of the seed squares each step), within an ulp or two of the rounded quotient.
__device__ __forceinline__ double rcp64(double x)
{
    double y = __builtin_amdgcn_rcp(x);
    double e = __fma_rn(-x, y, 1.0);
    y = __fma_rn(y, e, y);
    e = __fma_rn(-x, y, 1.0);
    return __fma_rn(y, e, y);
}
// The FP32 counterpart for plant_scalars<float>: one Newton step on the hardware reciprocal.
__device__ __forceinline__ float rcp64(float x)
{
    float y = rcp(x);
    return __fmaf_rn(y, __fmaf_rn(-x, y, 1.0f), y);
}

// Type of the decimal constants in plant_scalars: the scalar itself for plain
// types, FP64 for the dual numbers of the sensitivity pass.
template <class S> struct LitT { using type = double; };
template <> struct LitT<float> { using type = float; };
// 1 / k in that type, rounded once
template <class S>
__device__ constexpr typename LitT<S>::type inverse(int k) { return typename LitT<S>::type(1) / (typename LitT<S>::type)k; }

// Continuous-time coefficients (per ms) and the statics of candidate p for a
// saccade of amplitude amp (deg): the matrix entries of the mechanical block,
// the force couplings and active-state rates of both pieces, the pulse
// equilibrium's theta, and the deviations rest - pulse equilibrium and pulse
// equilibrium - post equilibrium (Section 2.1).  Generic in the scalar so that
// the sensitivity pass runs the very same formulas on dual numbers.
template <class S>
struct PlantScalars {
    S a10, a11, a12, a13, a20, a22, g2, a30, a33, g3;
    S q1a, q1n, q2a, q2n;
    S th1;
    S d0[6];
    S sh[6];
};

template <class S>
__device__ __forceinline__ void plant_scalars(const S p[P], S amp, PlantScalars<S>& o)
{
    using L = typename LitT<S>::type;
    const S kse_a = p[0], kse_n = p[1], klt_a = p[2], klt_n = p[3];
    const S b_a = p[4] * L(1e3), b_n = p[5] * L(1e3), b_p = p[6] * L(1e3);
    const S nc_a = p[7], nc_n = p[8];
    const S kp = nc_a + nc_n;            // passive elasticity = sum of tension slopes
    const S jm = p[9] * L(1e6);
    const S ij = rcp64(jm), iba = rcp64(b_a), ibn = rcp64(b_n);
    o.a10 = -(kse_a + kse_n + kp) * ij;
    o.a11 = -b_p * ij;
    o.a12 = kse_a * ij;
    o.a13 = -kse_n * ij;
    o.a20 = kse_a * iba;
    o.a22 = -(klt_a + kse_a) * iba;
    o.g2 = iba;
    o.a30 = -kse_n * ibn;
    o.a33 = -(klt_n + kse_n) * ibn;
    o.g3 = ibn;
    o.q1a = -rcp64(p[10]);
    o.q1n = -rcp64(p[11]);
    o.q2a = -rcp64(p[12]);
    o.q2n = -rcp64(p[13]);

    // statics: c_m = K_SE/(K_SE + K_LT) is the share of the active state the series element carries
    const S iksa = rcp64(kse_a), iksn = rcp64(kse_n);
    const S ica = L(1.0) + klt_a * iksa, icn = L(1.0) + klt_n * iksn;  // 1/c_m
    const S ca = kse_a * rcp64(kse_a + klt_a), cn = kse_n * rcp64(kse_n + klt_n);
    const S kt = kp + ca * klt_a + cn * klt_n;
    const S nfix = p[14], ns_a = p[15], ns_n = p[16], a = amp;
    // rest: theta = 0, fixation tension N_C_FIX on both muscles
    const S xa0 = nfix * iksa, xn0 = nfix * iksn;
    const S fa0 = nfix * ica, fn0 = nfix * icn;
    // pulse piece equilibrium (active states at the pulse heights)
    const S th1 = (ca * ns_a - cn * ns_n) * rcp64(kt);
    const S ta1 = ca * (ns_a - klt_a * th1), tn1 = cn * (ns_n + klt_n * th1);
    const S xa1 = th1 + ta1 * iksa, xn1 = tn1 * iksn - th1;
    // post piece equilibrium: the step holds the eye at the amplitude
    const S ta2 = nfix + nc_a * a, tn2 = nfix - nc_n * a;
    const S xa2 = a + ta2 * iksa, xn2 = tn2 * iksn - a;
    const S fa2 = ta2 * ica + klt_a * a, fn2 = tn2 * icn - klt_n * a;
    o.th1 = th1;
    o.d0[0] = -th1; o.d0[1] = S(0.0); o.d0[2] = xa0 - xa1; o.d0[3] = xn0 - xn1;
    o.d0[4] = fa0 - ns_a; o.d0[5] = fn0 - ns_n;
    o.sh[0] = th1 - a; o.sh[1] = S(0.0); o.sh[2] = xa1 - xa2; o.sh[3] = xn1 - xn2;
    o.sh[4] = ns_a - fa2; o.sh[5] = ns_n - fn2;
}

// Coefficients and equilibria c (per ms) in units of the base step h = dt / 2^taylor_sq of discretisation D
// (omega included: rest and equilibria have none, so no state is rescaled).
template <class D, class RT, class ST>
__device__ __forceinline__ void plant_scale(const PlantScalars<ST>& c, RT amp, RT dt, PlantT<RT>& pl)
{
    const RT h = dt * (1.0f / (float)(1 << D::taylor_sq));
    const RT hh = h * h;
    pl.a10 = (RT)c.a10 * hh; pl.a11 = (RT)c.a11 * h; pl.a12 = (RT)c.a12 * hh; pl.a13 = (RT)c.a13 * hh;
    pl.a20 = (RT)c.a20 * h; pl.a22 = (RT)c.a22 * h; pl.g2 = (RT)c.g2 * h;
    pl.a30 = (RT)c.a30 * h; pl.a33 = (RT)c.a33 * h; pl.g3 = (RT)c.g3 * h;
    pl.q[0] = (RT)c.q1a * h; pl.q[1] = (RT)c.q1n * h; pl.q[2] = (RT)c.q2a * h; pl.q[3] = (RT)c.q2n * h;
    pl.th1 = (RT)c.th1;
    pl.amp = amp;
#pragma unroll
    for (int i = 0; i < 6; ++i) { pl.d0[i] = (RT)c.d0[i]; pl.sh[i] = (RT)c.sh[i]; }
}

// Candidate p for a saccade of amplitude amp (deg), sample period dt (ms).  The scalar part is formed in ST
// and rounded once to RT.  FP32 chains of reciprocals shift the equilibria by
// a few ulps of ~10 deg, i.e. ~1e-6 deg on every sample: below the FP32
// recurrence's own error, and a bias the FP64 recurrence does not take.
template <class RT, class ST = typename Prec<RT>::scalar>
__device__ __forceinline__ void plant_setup(const float p[P], float amp, float dt, PlantT<RT>& pl)
{
    ST pd[P];
#pragma unroll
    for (int j = 0; j < P; ++j) pd[j] = p[j];
    PlantScalars<ST> c;
    plant_scalars(pd, (ST)amp, c);
    plant_scale<Prec<RT>>(c, (RT)amp, (RT)dt, pl);
    pl.pwd = (double)p[17] * rcp64((double)dt);
}

// ---------------------------------------------------------------------------
// Transitions as polynomials
// ---------------------------------------------------------------------------
// In units of a base step (time in steps, omega per step; see plant_setup) let B be the mechanical block.
// Every transition D = Phi - I over whole steps is F(B) for a polynomial F, and by Cayley-Hamilton that of
// degree 3 which F leaves modulo the characteristic polynomial chi(z) = z^4 - c3 z^3 - c2 z^2 - c1 z - c0 of
// B: four numbers a[] instead of a matrix.  The coupling column of an active state with rate q is the
// divided difference (F(B) - F(q)) / (B - q) g = (a-part + s Q(B)) g, with Q = (chi(z) - chi(q)) / (z - q) and
// s the value at q of the quotient of F by chi, so each rate carries s and f = F(q): no division, and
// nothing singular where a rate meets an eigenvalue.  Doubling a step costs ~60 operations here and
// 172 on matrices, and B is sparse enough that F(B)'s entries are short closed forms.  The Taylor
// polynomial, the base step and so the truncation are those of a Horner evaluation on matrices; the
// rounding is a few units (relative rms of the FP32 entries 4e-8 to 1.3e-7, Horner's 6e-8 to 1.4e-7).
template <class RT>
struct PolyBasis {
    RT c0, c1, c2, c3;  // chi
    RT u, v;            // a12 a20, a13 a30
};

template <class RT>
struct Poly {
    RT a[4];        // F modulo chi
    RT s[4], f[4];  // per rate (pulse ag, ant, post ag, ant): the quotient's value and F
};

template <class RT>
__device__ __forceinline__ void poly_basis(const PlantT<RT>& pl, PolyBasis<RT>& b)
{
    b.u = pl.a20 * pl.a12;
    b.v = pl.a30 * pl.a13;
    const RT sg = pl.a22 + pl.a33, pi = pl.a22 * pl.a33;
    b.c3 = pl.a11 + sg;
    b.c2 = fmr(-pl.a11, sg, pl.a10 - pi);
    b.c1 = fmr(pl.a11, pi, fmr(-pl.a10, sg, b.u + b.v));
    b.c0 = fmr(pl.a10, pi, fmr(-b.u, pl.a33, -b.v * pl.a22));
}

// F(z) = sum_{k=1..M} z^k / k!
template <int M, class RT>
__device__ __forceinline__ void poly_exp(const PlantT<RT>& pl, const PolyBasis<RT>& b, Poly<RT>& p)
{
    static_assert(M >= 4, "degree");
    RT a[M + 1];
    a[0] = RT(0);
    double r = 1.0;
#pragma unroll
    for (int k = 1; k <= M; ++k) { r /= k; a[k] = (RT)(typename LitT<RT>::type)r; }
#pragma unroll
    for (int c = 0; c < 4; ++c) {
        RT f = a[M];
#pragma unroll
        for (int k = M - 1; k >= 1; --k) f = fmr(f, pl.q[c], a[k]);
        p.f[c] = f * pl.q[c];
    }
#pragma unroll
    for (int k = M; k >= 4; --k) {  // the leading coefficient joins the quotient
        a[k - 1] = fmr(b.c3, a[k], a[k - 1]);
        a[k - 2] = fmr(b.c2, a[k], a[k - 2]);
        a[k - 3] = fmr(b.c1, a[k], a[k - 3]);
        a[k - 4] = fmr(b.c0, a[k], a[k - 4]);
    }
#pragma unroll
    for (int c = 0; c < 4; ++c) {
        RT s = a[M];
#pragma unroll
        for (int k = M - 1; k >= 4; --k) s = fmr(s, pl.q[c], a[k]);
        p.s[c] = s;
        p.a[c] = a[c];
    }
}

// o = the transition over x's and y's steps together: (1 + x)(1 + y) - 1 modulo chi.  t[0..6]: the
// coefficients of x y + x + y.  (o may be x or y.)
template <class RT>
__device__ __forceinline__ void poly_reduce(const PlantT<RT>& pl, const PolyBasis<RT>& b, const RT (&t)[7],
                                            const Poly<RT>& x, const Poly<RT>& y, Poly<RT>& o)
{
    const RT e2 = t[6], e1 = fmr(b.c3, e2, t[5]), e0 = fmr(b.c3, e1, fmr(b.c2, e2, t[4]));  // the quotient
    Poly<RT> r;
    r.a[3] = fmr(b.c3, e0, fmr(b.c2, e1, fmr(b.c1, e2, t[3])));
    r.a[2] = fmr(b.c2, e0, fmr(b.c1, e1, fmr(b.c0, e2, t[2])));
    r.a[1] = fmr(b.c1, e0, fmr(b.c0, e1, t[1]));
    r.a[0] = fmr(b.c0, e0, t[0]);
#pragma unroll
    for (int c = 0; c < 4; ++c) {
        const RT q = pl.q[c], eq = fmr(q, fmr(q, e2, e1), e0);
        const RT xq = fmr(q, fmr(q, fmr(q, x.a[3], x.a[2]), x.a[1]), x.a[0]);
        r.s[c] = fmr(x.s[c], y.f[c] + RT(1), fmr(y.s[c], xq + RT(1), eq));
        r.f[c] = fmr(x.f[c], y.f[c], x.f[c] + y.f[c]);
    }
    o = r;
}
template <class RT>
__device__ __forceinline__ void poly_twice(const PlantT<RT>& pl, const PolyBasis<RT>& b, const Poly<RT>& x, Poly<RT>& o)
{
    const RT a0 = x.a[0], a1 = x.a[1], a2 = x.a[2], a3 = x.a[3];
    const RT d0 = a0 + a0, d1 = a1 + a1, d2 = a2 + a2, d3 = a3 + a3;
    const RT t[7] = {fmr(a0, a0, d0), fmr(d1, a0, d1), fmr(a1, a1, fmr(d2, a0, d2)), fmr(d2, a1, fmr(d3, a0, d3)),
                     fmr(a2, a2, d3 * a1), d3 * a2, a3 * a3};
    poly_reduce(pl, b, t, x, x, o);
}
template <class RT>
__device__ __forceinline__ void poly_join(const PlantT<RT>& pl, const PolyBasis<RT>& b, const Poly<RT>& x,
                                          const Poly<RT>& y, Poly<RT>& o)
{
    const RT* p = x.a;
    const RT* q = y.a;
    const RT t[7] = {fmr(p[0], q[0], p[0] + q[0]),
                     fmr(p[1], q[0], fmr(p[0], q[1], p[1] + q[1])),
                     fmr(p[2], q[0], fmr(p[1], q[1], fmr(p[0], q[2], p[2] + q[2]))),
                     fmr(p[3], q[0], fmr(p[2], q[1], fmr(p[1], q[2], fmr(p[0], q[3], p[3] + q[3])))),
                     fmr(p[3], q[1], fmr(p[2], q[2], p[1] * q[3])),
                     fmr(p[3], q[2], p[2] * q[3]), p[3] * q[3]};
    poly_reduce(pl, b, t, x, y, o);
}

// Row 0 (theta) of F(B), and theta's coupling to the four active states.
template <class RT>
__device__ __forceinline__ void poly_theta_row(const PlantT<RT>& pl, const PolyBasis<RT>& b, const Poly<RT>& p,
                                               RT (&m)[4], RT (&x)[4])
{
    const RT a0 = p.a[0], a1 = p.a[1], a2 = p.a[2], a3 = p.a[3];
    m[0] = fmr(a2, pl.a10, fmr(a3, fmr(pl.a10, pl.a11, b.u + b.v), a0));
    m[1] = fmr(a3, pl.a10, fmr(pl.a11, fmr(pl.a11, a3, a2), a1));
    m[2] = pl.a12 * fmr(a3, pl.a11 + pl.a22, a2);
    m[3] = pl.a13 * fmr(a3, pl.a11 + pl.a33, a2);
#pragma unroll
    for (int c = 0; c < 4; ++c)
        x[c] = ((c & 1) ? pl.g3 * pl.a13 : pl.g2 * pl.a12) * fmr(p.s[c], pl.q[c] - ((c & 1) ? pl.a22 : pl.a33), a3);
}

// Rows 1..3 of F(B) from its row 0.  Row 1: B's row 0 is the unit row 1, so row 1 of F(B) is row 0 of
// B F(B) = F(B) B.
template <class RT>
__device__ __forceinline__ void poly_block(const PlantT<RT>& pl, const PolyBasis<RT>& b, const Poly<RT>& p,
                                           RT (&m)[4][4])
{
    const RT a0 = p.a[0], a1 = p.a[1], a2 = p.a[2], a3 = p.a[3];
    const RT l2 = fmr(pl.a22, fmr(pl.a22, a3, a2), a1), l3 = fmr(pl.a33, fmr(pl.a33, a3, a2), a1);
    m[1][0] = fmr(m[0][1], pl.a10, fmr(m[0][2], pl.a20, m[0][3] * pl.a30));
    m[1][1] = fmr(m[0][1], pl.a11, m[0][0]);
    m[1][2] = fmr(m[0][1], pl.a12, m[0][2] * pl.a22);
    m[1][3] = fmr(m[0][1], pl.a13, m[0][3] * pl.a33);
    m[2][0] = pl.a20 * fmr(a3, pl.a10, l2);
    m[2][1] = pl.a20 * fmr(a3, pl.a11 + pl.a22, a2);
    m[2][2] = fmr(a3, b.u, fmr(pl.a22, l2, a0));
    m[2][3] = a3 * (pl.a20 * pl.a13);
    m[3][0] = pl.a30 * fmr(a3, pl.a10, l3);
    m[3][1] = pl.a30 * fmr(a3, pl.a11 + pl.a33, a2);
    m[3][2] = a3 * (pl.a30 * pl.a12);
    m[3][3] = fmr(a3, b.v, fmr(pl.a33, l3, a0));
}

// The divided difference of F at rate q as n[0] + n[1] z + n[2] z^2 + n[3] z^3.
template <class RT>
__device__ __forceinline__ void poly_difference(const PolyBasis<RT>& b, RT q, RT a1, RT a2, RT a3, RT s, RT (&n)[4])
{
    const RT q2 = q - b.c3, q1 = fmr(q, q2, -b.c2), q0 = fmr(q, q1, -b.c1);  // Q = z^3 + q2 z^2 + q1 z + q0
    const RT n1 = fmr(q, a3, a2);
    n[3] = s;
    n[2] = fmr(s, q2, a3);
    n[1] = fmr(s, q1, n1);
    n[0] = fmr(s, q0, fmr(q, n1, a1));
}

// Rows 1..3 of coupling column c (its polynomial at B, applied to g's muscle: row 2 or 3).
template <class RT>
__device__ __forceinline__ void poly_column(const PlantT<RT>& pl, const PolyBasis<RT>& b, const Poly<RT>& p, int c,
                                            RT (&x)[4][4])
{
    const bool ant = (c & 1) != 0;
    const RT g = ant ? pl.g3 : pl.g2, sd = ant ? pl.a33 : pl.a22, s1 = ant ? pl.a13 : pl.a12;
    RT n[4];
    poly_difference(b, pl.q[c], p.a[1], p.a[2], p.a[3], p.s[c], n);
    const RT k = fmr(n[3], pl.a11 + sd, n[2]);
    x[1][c] = g * s1 * fmr(sd, k, fmr(n[3], pl.a10, fmr(pl.a11, fmr(pl.a11, n[3], n[2]), n[1])));
    const RT own = g * fmr(n[3], ant ? b.v : b.u, fmr(sd, fmr(sd, fmr(sd, n[3], n[2]), n[1]), n[0]));
    const RT other = g * n[3] * (ant ? pl.a20 * pl.a13 : pl.a30 * pl.a12);
    x[2][c] = ant ? other : own;
    x[3][c] = ant ? own : other;
}

// d <- Phi d in the pulse piece for the transition p.
template <class RT>
__device__ __forceinline__ void poly_apply(const PlantT<RT>& pl, const PolyBasis<RT>& b, const Poly<RT>& p, RT d[6])
{
    const RT* a = p.a;
    RT na[4], nn[4];
    poly_difference(b, pl.q[0], a[1], a[2], a[3], p.s[0], na);
    poly_difference(b, pl.q[1], a[1], a[2], a[3], p.s[1], nn);
    const RT ga = pl.g2 * d[4], gn = pl.g3 * d[5];
    RT w0 = a[3] * d[0], w1 = a[3] * d[1], w2 = fmr(ga, na[3], a[3] * d[2]), w3 = fmr(gn, nn[3], a[3] * d[3]);
#pragma unroll
    for (int j = 2; j >= 0; --j) {  // w <- B w + a_j d + n_j g F
        const RT r0 = fmr(a[j], d[0], w1);
        const RT r1 = fmr(pl.a10, w0, fmr(pl.a11, w1, fmr(pl.a12, w2, fmr(pl.a13, w3, a[j] * d[1]))));
        const RT r2 = fmr(pl.a20, w0, fmr(pl.a22, w2, fmr(ga, na[j], a[j] * d[2])));
        const RT r3 = fmr(pl.a30, w0, fmr(pl.a33, w3, fmr(gn, nn[j], a[j] * d[3])));
        w0 = r0; w1 = r1; w2 = r2; w3 = r3;
    }
    d[0] = d[0] + w0; d[1] = d[1] + w1; d[2] = d[2] + w2; d[3] = d[3] + w3;
    d[4] = fmr(p.f[0], d[4], d[4]);
    d[5] = fmr(p.f[1], d[5], d[5]);
}

// d <- Phi d for one step of pl's transition (D-form: d + D d) in the pulse (PIECE 0) or post (1) piece
template <int PIECE, class RT>
__device__ __forceinline__ void step(const PlantT<RT>& pl, RT d[6])
{
    RT n[4];
    // the row's own state is the addend of the first fma
    n[0] = fmr(pl.m[0][0], d[0], d[0]);
    n[1] = fmr(pl.m[1][1], d[1], d[1]);
    n[2] = fmr(pl.m[2][2], d[2], d[2]);
    n[3] = fmr(pl.m[3][3], d[3], d[3]);
#pragma unroll
    for (int i = 0; i < 4; ++i) {
#pragma unroll
        for (int c = 0; c < 4; ++c)
            if (c != i) n[i] = fmr(pl.m[i][c], d[c], n[i]);
        n[i] = fmr(pl.x[i][2 * PIECE], d[4], n[i]);
        n[i] = fmr(pl.x[i][2 * PIECE + 1], d[5], n[i]);
    }
    d[4] = fmr(pl.e[2 * PIECE], d[4], d[4]);
    d[5] = fmr(pl.e[2 * PIECE + 1], d[5], d[5]);
#pragma unroll
    for (int i = 0; i < 4; ++i) d[i] = n[i];
}

// v <- exp(A t) v (t in base steps) by a Taylor polynomial of degree D::expmv_m in Horner form, in
// the pulse (PIECE 0) or post (1) piece; t is at most one sample.
template <class D, int PIECE, class RT>
__device__ __forceinline__ void expmv(const PlantT<RT>& pl, RT t, RT v[6])
{
    RT w[6];
#pragma unroll
    for (int i = 0; i < 6; ++i) w[i] = v[i];
#pragma unroll
    for (int k = D::expmv_m; k >= 1; --k) {
        RT s = t * inverse<RT>(k);
        keep(s);
        RT aw[6];
        aw[0] = w[1];
        aw[1] = fmr(pl.a13, w[3], fmr(pl.a12, w[2], fmr(pl.a11, w[1], pl.a10 * w[0])));
        aw[2] = fmr(pl.g2, w[4], fmr(pl.a22, w[2], pl.a20 * w[0]));
        aw[3] = fmr(pl.g3, w[5], fmr(pl.a33, w[3], pl.a30 * w[0]));
        aw[4] = pl.q[2 * PIECE] * w[4];
        aw[5] = pl.q[2 * PIECE + 1] * w[5];
#pragma unroll
        for (int i = 0; i < 6; ++i) w[i] = fmr(s, aw[i], v[i]);
    }
#pragma unroll
    for (int i = 0; i < 6; ++i) v[i] = w[i];
}

// The sample that contains the pulse end: pulse dynamics for frac of it, switch to the post piece's
// coordinates, post dynamics for the rest.
template <class D, class RT>
__device__ __forceinline__ void split_step(const PlantT<RT>& pl, RT frac, RT d[6])
{
    constexpr float steps = (float)(1 << D::taylor_sq);  // base steps per sample
    expmv<D, 0>(pl, frac * steps, d);
#pragma unroll
    for (int i = 0; i < 6; ++i) d[i] = d[i] + pl.sh[i];
    expmv<D, 1>(pl, (RT(1) - frac) * steps, d);
}

// wave-wide min of an int (64 lanes)
__device__ __forceinline__ int wave_min(int v)
{
#pragma unroll
    for (int o = 32; o >= 1; o >>= 1) v = min(v, __shfl_xor(v, o));
    return v;
}

// Integer sample index that holds the pulse end (-1: no pulse), clamped to
// [-1, T], and the fraction of that sample spent in the pulse.
template <class RT>
__device__ __forceinline__ int pulse_end_sample(double pw, int T, RT& frac)
{
    double fl = floor(pw);
    int k0;
    if (!(pw > 0.0)) { k0 = -1; frac = RT(0); }
    else if (fl >= (double)T) { k0 = T; frac = RT(0); }
    else { k0 = (int)fl; frac = (RT)(pw - fl); }
    return k0;
}

// Samples advanced per step of the block recurrence (run_blocks).
constexpr int BLOCK = 4;

// Theta rows of the transitions over 1, 2 and 3 samples in D-form: theta_{k+j} = theta_k + row_j . d_k.
template <class RT>
struct ThetaRows {
    RT m[BLOCK - 1][4];  // theta, omega, x_ag, x_ant
    RT x[BLOCK - 1][4];  // F_ag, F_ant in the pulse piece, then in the post piece
};

// sink.begin(k, u), minus row_j . d, handed to sink.end: one sample of a block at offset j >= 1.
template <int PIECE, class RT, class Sink>
__device__ __forceinline__ void row_sample(const ThetaRows<RT>& rw, int j, int k, RT u, const RT d[6], Sink& sink)
{
    RT t = sink.begin(k, u);
#pragma unroll
    for (int c = 0; c < 4; ++c) t = fmr(-rw.m[j - 1][c], d[c], t);
    t = fmr(-rw.x[j - 1][2 * PIECE], d[4], t);
    t = fmr(-rw.x[j - 1][2 * PIECE + 1], d[5], t);
    sink.end(k, t);
}

// One block: samples k .. k+3 from the state d at sample k, then d at sample k+4.
template <int PIECE, class RT, class Sink>
__device__ __forceinline__ void block_step(const PlantT<RT>& pl, const ThetaRows<RT>& rw, int k, RT theq, RT d[6],
                                           Sink& sink)
{
    const RT u = d[0] + theq;
    sink.end(k, sink.begin(k, u));
#pragma unroll
    for (int j = 1; j < BLOCK; ++j) row_sample<PIECE>(rw, j, k + j, u, d, sink);
    step<PIECE>(pl, d);
}

// Run the trajectory theta_k, k = 0..T-1: for each sample, t = sink.begin(k, u) and sink.end(k, t - v)
// with theta_k = u + v; sink.block_end() after each whole block (at most 7 samples lie outside blocks).
// pl's transition (m, x, e) is set to that of a block.
//
// Bound by VALU issue.  A block of four samples costs one step of the four-sample transition (26
// multiply-adds) and three rows (6 each) instead of four one-sample steps: 53 operations per block with a
// squared residual instead of 116.  The transitions over 1, 2, 3 and 4 samples come as polynomials
// (~320 operations with the rows; as matrices, Horner and two doublings, ~870).  Measured on a
// round of 256 x 65536 candidates (mean T 57), one-sample steps -> blocks -> blocks from polynomials:
// FP32 0.841 -> 0.708 -> 0.604 ms, FP64 1.724 -> 1.425 -> 1.191 ms.  Blocks of two save less on long
// traces (18 operations per sample), blocks of eight need 42 more row coefficients in registers.
// The lane's blocks end at its own pulse-end sample: the first k0 mod 4 samples take their rows and a
// jump, so a candidate's arithmetic depends on the candidate alone; lanes of a wave whose pulse ends
// differ by a block mask a block each.
template <class D, class RT, class Sink>
__device__ __forceinline__ void run_blocks_as(PlantT<RT>& pl, int T, int k0, RT frac, Sink& sink)
{
    RT d[6];
#pragma unroll
    for (int i = 0; i < 6; ++i) d[i] = pl.d0[i];
    RT theq = pl.th1;
    if (k0 < 0) {  // PW <= 0: no pulse, the step acts from t = 0
#pragma unroll
        for (int i = 0; i < 6; ++i) d[i] = d[i] + pl.sh[i];
        theq = pl.amp;
    }
    ThetaRows<RT> rw;
    PolyBasis<RT> pb;
    Poly<RT> f1, f2;
    poly_basis(pl, pb);
    poly_exp<D::taylor_m>(pl, pb, f1);
#pragma unroll
    for (int q = 0; q < D::taylor_sq; ++q) poly_twice(pl, pb, f1, f1);
    poly_theta_row(pl, pb, f1, rw.m[0], rw.x[0]);
    poly_twice(pl, pb, f1, f2);
    poly_theta_row(pl, pb, f2, rw.m[1], rw.x[1]);
    const int np = max(k0, 0), head = np % BLOCK;  // samples before the pulse end (k0 <= T), and before the blocks
    int k = 0;
    if (head) {
        const RT u = d[0] + theq;
        sink.end(0, sink.begin(0, u));
        if (head > 1) row_sample<0>(rw, 1, 1, u, d, sink);
        if (head > 2) row_sample<0>(rw, 2, 2, u, d, sink);
        if (head & 2) poly_apply(pl, pb, f2, d);
        if (head & 1) poly_apply(pl, pb, f1, d);
        k = head;
    }
    poly_join(pl, pb, f1, f2, f1);
    poly_theta_row(pl, pb, f1, rw.m[2], rw.x[2]);
    poly_twice(pl, pb, f2, f2);
    poly_theta_row(pl, pb, f2, pl.m[0], pl.x[0]);
    poly_block(pl, pb, f2, pl.m);
#pragma unroll
    for (int c = 0; c < 4; ++c) { poly_column(pl, pb, f2, c, pl.x); pl.e[c] = f2.f[c]; }
#pragma unroll
    for (int c = 2; c < 4; ++c) {
#pragma unroll
        for (int i = 0; i < 4; ++i) keep(pl.x[i][c]);
#pragma unroll
        for (int j = 0; j < BLOCK - 1; ++j) keep(rw.x[j][c]);
        keep(pl.e[c]);
    }
#pragma unroll 1
    for (; k < np; k += BLOCK) {
        block_step<0>(pl, rw, k, theq, d, sink);
        sink.block_end();
    }
    if (k0 >= 0 && k0 < T) {
        sink.end(k, sink.begin(k, d[0] + theq));
        split_step<D>(pl, frac, d);
        theq = pl.amp;
        ++k;
    }
#pragma unroll 1
    for (; k + BLOCK <= T; k += BLOCK) {
        block_step<1>(pl, rw, k, theq, d, sink);
        sink.block_end();
    }
    // the last samples need no further state: their rows alone
    if (k < T) {
        const RT u = d[0] + theq;
        sink.end(k, sink.begin(k, u));
#pragma unroll
        for (int j = 1; j < BLOCK - 1; ++j)
            if (k + j < T) row_sample<1>(rw, j, k + j, u, d, sink);
    }
}

// run_blocks_as in the search's discretisation.
template <class RT, class Sink>
__device__ __forceinline__ void run_blocks(PlantT<RT>& pl, int T, int k0, RT frac, Sink& sink)
{
    run_blocks_as<Prec<RT>>(pl, T, k0, frac, sink);
}

}  // namespace opmm
