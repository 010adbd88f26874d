// libopmm: the paper's own estimator -- a parallel Nelder-Mead per saccade
// (Section 3.3, Algorithm 1): one task per saccade, all simplex transforms of
// an iteration evaluated simultaneously, the simplex sorted every iteration,
// both exit tolerances or an iteration cap.
//
// One to three saccades per 64-lane wave, a group of lanes each.  Lane j of a group holds coordinate j of
// all 19 vertices (FP64, relative to the Table 1 nominal, sorted by value) in registers and lane i the
// value of vertex i; a new vertex goes to its rank by a ballot and a shift, so nothing is sorted but
// after a shrink.  An evaluation runs on a quad of lanes: each lane one column of the transition, then
// one row of the recurrence.  An iteration evaluates reflection, expansion, outside and inside
// contraction at once on four quads; the 18 shrink vertices follow on every quad of the group in
// the few iterations that the Lagarias decision (reflection 1, expansion 2, contraction 1/2, shrink 1/2)
// asks for them.  Each evaluation is the same plant simulation and RMSE as the box search (points
// clamped to the search box and rounded to FP32, the candidate format).
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <cstring>
#include <vector>

#include "../../include/opmm.h"
#include "plant.hpp"
#include "runtime.hpp"

using namespace opmm;
using opmm_rt::SacDev;

namespace {

constexpr int NV = P + 1;   // simplex vertices
constexpr int PTS = 20;     // floats per row of points in LDS (P and padding to 16 bytes)

// Lanes of a group of a wave with G groups: whole quads, a lane per vertex at least.
constexpr int group_lanes(int g) { return g == 1 ? 64 : g == 2 ? 32 : 20; }
static_assert(group_lanes(3) >= NV && group_lanes(3) % 4 == 0 && 3 * group_lanes(3) <= 64, "lane groups");

// ---- quad exchange ----------------------------------------------------------
constexpr int quad(int a, int b, int c, int d) { return a | (b << 2) | (c << 4) | (d << 6); }
template <int CTRL>
__device__ __forceinline__ double quad_perm(double x)
{
    const int lo = __builtin_amdgcn_mov_dpp(__double2loint(x), CTRL, 0xf, 0xf, true);
    const int hi = __builtin_amdgcn_mov_dpp(__double2hiint(x), CTRL, 0xf, 0xf, true);
    return __hiloint2double(hi, lo);
}
template <int K>
__device__ __forceinline__ double quad_bcast(double x) { return quad_perm<quad(K, K, K, K)>(x); }

// Least x over the wave, for an x that is the same on the four lanes of a quad (a scalar).
__device__ __forceinline__ int min_over_quads(int x)
{
    x = min(x, __builtin_amdgcn_mov_dpp(x, 0x124, 0xf, 0xf, true));  // row_ror:4
    x = min(x, __builtin_amdgcn_mov_dpp(x, 0x128, 0xf, 0xf, true));  // row_ror:8
    return min(min(__builtin_amdgcn_readlane(x, 0), __builtin_amdgcn_readlane(x, 16)),
               min(__builtin_amdgcn_readlane(x, 32), __builtin_amdgcn_readlane(x, 48)));
}

// One of four values by lane.  (The pins keep the choice among registers: seen as a choice among struct
// fields it becomes an indexed load, and the struct goes to scratch memory.)
__device__ __forceinline__ double pick(int i, double a, double b, double c, double d)
{
    keep(a); keep(b); keep(c); keep(d);
    return i == 0 ? a : i == 1 ? b : i == 2 ? c : d;
}

// ---- one evaluation on a quad -------------------------------------------------
// The simplex's iterates depend on every rounding of its costs, so that its results stay the bits they were this
// file keeps the sample-by-sample evaluation: the transition by Horner's rule and squarings on matrices, one
// step per sample.  (run_blocks in plant.hpp gives the same trajectories to ~1e-14 deg, well within what the
// decisions' comparison with the oracle allows.)  A quad only spreads that evaluation's operations over four
// lanes; each result goes through the same operations in the same order as on one.

// Column c of the one-sample transition in D-form (D = Phi - I): mechanical block m[.][c], coupling x[.][c]
// of active state c (pulse ag, pulse ant, post ag, post ant) and that state's factor minus one e.
// Horner on the step dt/4 with scaled iterates (B = hA: Q_M = M I + B, Q_k = c_k I + B Q_{k+1}, c_k = k c_{k+1},
// D = B Q_2 / M!), then two squarings D_2h = D_h^2 + 2 D_h.  A column of a product needs the left factor
// whole: its columns come from the other lanes.
__device__ __forceinline__ void transition_column(const PlantScalars<double>& pc, double dt, int c, double m[4],
                                                  double x[4], double& e)
{
    constexpr int M = Prec<double>::taylor_m, SQ = Prec<double>::taylor_sq;
    const double h = dt * (1.0 / (double)(1 << SQ));
    const double s10 = pc.a10 * h, s11 = pc.a11 * h, s12 = pc.a12 * h, s13 = pc.a13 * h;
    const double s20 = pc.a20 * h, s22 = pc.a22 * h, s30 = pc.a30 * h, s33 = pc.a33 * h;
    const bool ant = (c & 1) != 0;
    const double sg = pick(c & 1, pc.g2, pc.g3, 0.0, 0.0) * h;
    const double q = pick(c, pc.q1a, pc.q1n, pc.q2a, pc.q2n);
    const double sq = q * h;
    {   // Q_M = M I + B
        const double mm = (double)M;
        m[0] = c == 0 ? mm : c == 1 ? h : 0.0;
        m[1] = c == 0 ? s10 : c == 1 ? mm + s11 : c == 2 ? s12 : s13;
        m[2] = c == 0 ? s20 : c == 2 ? mm + s22 : 0.0;
        m[3] = c == 0 ? s30 : c == 3 ? mm + s33 : 0.0;
        x[0] = 0.0;
        x[1] = 0.0;
        x[2] = ant ? 0.0 : sg;
        x[3] = ant ? sg : 0.0;
        e = mm + sq;
    }
    double ck = (double)M;
#pragma unroll
    for (int k = M - 1; k >= 1; --k) {
        double one, t10, t11, t12, t13, t20, t22, t30, t33, tv, tg, tq;
        if (k >= 2) {
            ck = ck * (double)k;
            one = ck;
            t10 = s10; t11 = s11; t12 = s12; t13 = s13; t20 = s20; t22 = s22; t30 = s30; t33 = s33;
            tv = h; tg = sg; tq = sq;
        } else {
            const double f = 1.0 / ck;  // 1 / M!, rounded once
            one = 0.0;
            t10 = s10 * f; t11 = s11 * f; t12 = s12 * f; t13 = s13 * f;
            t20 = s20 * f; t22 = s22 * f; t30 = s30 * f; t33 = s33 * f;
            tv = h * f; tg = sg * f; tq = sq * f;
        }
        double n[4], y[4];
        n[0] = fmr(tv, m[1], c == 0 ? one : 0.0);
        n[1] = fmr(t13, m[3], fmr(t12, m[2], fmr(t11, m[1], fmr(t10, m[0], c == 1 ? one : 0.0))));
        n[2] = fmr(t22, m[2], fmr(t20, m[0], c == 2 ? one : 0.0));
        n[3] = fmr(t33, m[3], fmr(t30, m[0], c == 3 ? one : 0.0));
        const double g = tg * e;
        y[0] = fmr(tv, x[1], 0.0);
        y[1] = fmr(t13, x[3], fmr(t12, x[2], fmr(t11, x[1], fmr(t10, x[0], 0.0))));
        y[2] = fmr(t22, x[2], fmr(t20, x[0], ant ? 0.0 : g));
        y[3] = fmr(t33, x[3], fmr(t30, x[0], ant ? g : 0.0));
        e = fmr(tq, e, one);
#pragma unroll
        for (int i = 0; i < 4; ++i) { m[i] = n[i]; x[i] = y[i]; }
    }
#pragma unroll
    for (int s = 0; s < SQ; ++s) {
        double n[4], y[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const double l0 = quad_bcast<0>(m[i]), l1 = quad_bcast<1>(m[i]), l2 = quad_bcast<2>(m[i]),
                         l3 = quad_bcast<3>(m[i]);
            n[i] = fmr(l3, m[3], fmr(l2, m[2], fmr(l1, m[1], fmr(l0, m[0], m[i] + m[i]))));
            y[i] = fmr(l3, x[3], fmr(l2, x[2], fmr(l1, x[1], fmr(l0, x[0], x[i] * (e + 2.0)))));
        }
#pragma unroll
        for (int i = 0; i < 4; ++i) { m[i] = n[i]; x[i] = y[i]; }
        e = e * (e + 2.0);
    }
}

// v <- exp(A t) v by a Taylor polynomial (degree Prec::expmv_m) in Horner form (t <= dt).
__device__ __forceinline__ void nm_expmv(const PlantScalars<double>& pc, double qa, double qn, double t, double v[6])
{
    double w[6];
#pragma unroll
    for (int i = 0; i < 6; ++i) w[i] = v[i];
#pragma unroll
    for (int k = Prec<double>::expmv_m; k >= 1; --k) {
        double s = t * (1.0 / (double)k);
        asm volatile("" : "+v"(s));
        double aw[6];
        aw[0] = w[1];
        aw[1] = fmr(pc.a13, w[3], fmr(pc.a12, w[2], fmr(pc.a11, w[1], pc.a10 * w[0])));
        aw[2] = fmr(pc.g2, w[4], fmr(pc.a22, w[2], pc.a20 * w[0]));
        aw[3] = fmr(pc.g3, w[5], fmr(pc.a33, w[3], pc.a30 * w[0]));
        aw[4] = qa * w[4];
        aw[5] = qn * w[5];
#pragma unroll
        for (int i = 0; i < 6; ++i) w[i] = fmr(s, aw[i], v[i]);
    }
#pragma unroll
    for (int i = 0; i < 6; ++i) v[i] = w[i];
}

// One row of the recurrence on the lane that holds state i: d <- d + D d, own term first, then the others
// by column, then the active states (fa, fn, the same on all four lanes).
struct Row {
    double own, o0, o1, o2, xa, xn;
};
__device__ __forceinline__ void row_step(const Row& w, double ea, double en, double& d, double& fa, double& fn)
{
    const double d0 = quad_perm<quad(1, 0, 0, 0)>(d), d1 = quad_perm<quad(2, 2, 1, 1)>(d),
                 d2 = quad_perm<quad(3, 3, 3, 2)>(d);
    double n = fmr(w.own, d, d);
    n = fmr(w.o0, d0, n);
    n = fmr(w.o1, d1, n);
    n = fmr(w.o2, d2, n);
    n = fmr(w.xa, fa, n);
    n = fmr(w.xn, fn, n);
    fa = fmr(ea, fa, fa);
    fn = fmr(en, fn, fn);
    d = n;
}

// Orders LDS accesses among the lanes of the wave (a block is one wave).
__device__ __forceinline__ void wave_sync()
{
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// RMSE of the point p (LDS, the candidate itself) on this lane's quad, the same value on its four lanes.
// All lanes of the wave call it; quads with run = false return without a meaningful value.  tr: 32
// doubles of LDS for the quad.
__device__ __forceinline__ double quad_eval(const float* p, const R* r, double* tr, bool run, const SacDev& sd,
                                            double qorth, float dt)
{
    const int i = threadIdx.x & 3;
    PlantScalars<double> pc;
    double pd[P];
#pragma unroll
    for (int j = 0; j < P; ++j) pd[j] = p[j];
    plant_scalars(pd, (double)sd.amp, pc);
    double e1a, e1n, e2a, e2n;
    Row w1, w2;
    {
        double m[4], x[4], e;
        transition_column(pc, (double)dt, i, m, x, e);
        e1a = quad_bcast<0>(e);
        e1n = quad_bcast<1>(e);
        e2a = quad_bcast<2>(e);
        e2n = quad_bcast<3>(e);
        wave_sync();  // the quad's previous evaluation has read its scratch
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            tr[4 * k + i] = m[k];
            tr[16 + 4 * k + i] = x[k];
        }
        wave_sync();
        const double* mr = tr + 4 * i;
        w1.own = mr[i];
        w1.o0 = mr[i == 0 ? 1 : 0];
        w1.o1 = mr[i <= 1 ? 2 : 1];
        w1.o2 = mr[i <= 2 ? 3 : 2];
        w2 = w1;
        w1.xa = tr[16 + 4 * i];
        w1.xn = tr[16 + 4 * i + 1];
        w2.xa = tr[16 + 4 * i + 2];
        w2.xn = tr[16 + 4 * i + 3];
    }
    const int T = sd.T;
    R frac;
    const int k0 = pulse_end_sample((double)p[17] * rcp64((double)dt), T, frac);
    double d = pick(i, pc.d0[0], pc.d0[1], pc.d0[2], pc.d0[3]), fa = pc.d0[4], fn = pc.d0[5];
    double theq = pc.th1, sse = 0.0;
    int k = 0;
    if (k0 < 0) {  // PW <= 0: no pulse, the step acts from t = 0
        d += pick(i, pc.sh[0], pc.sh[1], pc.sh[2], pc.sh[3]);
        fa += pc.sh[4];
        fn += pc.sh[5];
        theq = (double)sd.amp;
    }
    // theta is lane 0's state; the other lanes' sums go nowhere
    const int np = run ? max(k0, 0) : 0, nt = run ? T : 0;
    // n samples in the piece of row w: a stretch that every running quad of the wave has, counted on the
    // scalar unit, then the lane's own rest.  The next sample is read a step ahead (its latency is as
    // long as a step; r has a spare element).
    double rk = r[0];
    auto samples = [&](const Row& w, double ea, double en, int end) {
        auto one = [&]() {
            const double err = (rk - theq) - d;
            rk = r[k + 1];
            row_step(w, ea, en, d, fa, fn);
            sse = fmr(err, err, sse);
            ++k;
        };
        int common = min_over_quads(run ? max(end - k, 0) : 0x7FFFFFFF);
        if (common != 0x7FFFFFFF && run) {
            for (; common >= 4; common -= 4) { one(); one(); one(); one(); }
        }
#pragma unroll 1
        while (k < end) one();
    };
    samples(w1, e1a, e1n, np);
    if (run && k0 >= 0 && k0 < T) {
        const double err = (rk - theq) - d;
        rk = r[k + 1];
        sse = fmr(err, err, sse);
        double v[6] = {quad_bcast<0>(d), quad_bcast<1>(d), quad_bcast<2>(d), quad_bcast<3>(d), fa, fn};
        nm_expmv(pc, pc.q1a, pc.q1n, frac * (R)dt, v);
#pragma unroll
        for (int j = 0; j < 6; ++j) v[j] += pc.sh[j];
        nm_expmv(pc, pc.q2a, pc.q2n, (1.0 - frac) * (R)dt, v);
        d = pick(i, v[0], v[1], v[2], v[3]);
        fa = v[4];
        fn = v[5];
        theq = (double)sd.amp;
        ++k;
    }
    samples(w2, e2a, e2n, nt);
    sse = quad_bcast<0>(sse);
    const double rm = sqrt((sse + qorth) / ((double)T * sd.C));
    return (rm >= 0.0 && rm <= 1.7976931348623157e308) ? rm : INFINITY;
}

// One task's shared state.
struct NmGroup {
    float pt[NV][PTS];  // points to evaluate: clamped to the box, scaled, rounded to FP32
    double fp[NV];      // their values
    double tv[NV][P];   // sort staging
};

// G tasks per 64-lane wave: lane group g works on saccade order[G * block + g] (order: the batch sorted by
// T, so that a wave's tasks simulate traces of similar length).  Every group runs the same instruction
// stream; a finished group's lanes idle until the last one ends.  Each group's arithmetic is that of a
// wave of its own.  deadline_ticks > 0: a task still iterating when that many ticks of the wall clock
// (wall_clock64) have passed since the launch started ends there with OPMM_ST_DEADLINE.
//
// Bound by the latency of one wave's FP64 chains: a lone wave issues an independent FP64 instruction every
// ~5 cycles and a dependent one every 10.  With 22 points on 22 lanes, each lane a whole simulation, and
// the simplex in LDS an iteration took 36k cycles at T = 57 (241 a sample, 14k for points, sort and exit
// test); on quads, with the simplex in registers, 97 a sample and 12k in all.  256 saccades x 500
// iterations: 9.05 -> 3.5 ms; 4096 x 200: 9.27 -> 2.17 ms.  The bound of 256 registers leaves room for two
// waves per SIMD (4096 saccades 2.41 -> 2.17 ms, 8192 3.99 -> 3.24 ms against one).
template <int G>
__global__ __launch_bounds__(64, 2) void nm_kernel(int S, const SacDev* __restrict__ sacs, const int* __restrict__ order,
                                                const float* __restrict__ proj,
                                                const double* __restrict__ qorth, const int32_t* __restrict__ status_in,
                                                const float* __restrict__ seed_opc, int max_iter, double tol_x,
                                                double tol_f, double lo, double hi, float dt, int max_T,
                                                uint64_t deadline_ticks, float* opc_out, float* rmse_out,
                                                int32_t* iters_out, int8_t* dec_out, int32_t* status_out)
{
    constexpr int LG = group_lanes(G), NQ = LG / 4;
    __shared__ NmGroup gs[G];
    __shared__ double trs[16][33];  // transposition scratch of a quad (odd stride: quads on different banks)
    extern __shared__ R rbuf[];     // [G][max_T + 1] projected traces
    const int lane = threadIdx.x;
    const bool member = lane < G * LG;
    const int gi = member ? lane / LG : 0, base = gi * LG;
    const int l = member ? lane - base : LG - 1 + (lane & 3);  // lanes past the groups: no role (l >= NV)
    const uint64_t gmask = (LG == 64 ? ~0ull : ((1ull << (LG & 63)) - 1)) << base;
    const bool have = member && G * (int)blockIdx.x + gi < S;
    const int s = have ? order[G * blockIdx.x + gi] : 0;
    NmGroup& g = gs[gi];
    R* r = rbuf + gi * (max_T + 1);
    double* tr = trs[lane >> 2];
    const SacDev sd = sacs[s];
    const double q = qorth[sd.slot];
    const int32_t st0 = status_in[sd.slot];
    const bool bad = !have || (st0 & OPMM_ST_NONFINITE_INPUT);
    const uint64_t t0 = wall_clock64();
    if (have && bad) {
        if (l < P) opc_out[(int64_t)s * P + l] = __int_as_float(0x7FC00000);
        if (l == 0) {
            rmse_out[s] = __int_as_float(0x7FC00000);
            if (iters_out) iters_out[s] = 0;
            if (status_out) status_out[s] = st0;
        }
    }
    if (!bad)
        for (int k = l; k < sd.T; k += LG) r[k] = (R)proj[sd.proj_off + k];
    const double nom = nominal_param_f64(l < P ? l : 0, (double)sd.dur);
    // x on lane base + i of every lane's group (one task per wave: a scalar read)
    auto at = [&](double x, int i) {
        if (G > 1) return __shfl(x, base + i);
        return __hiloint2double(__builtin_amdgcn_readlane(__double2hiint(x), i),
                                __builtin_amdgcn_readlane(__double2loint(x), i));
    };
    // the candidate format of coordinate x on this lane
    auto clampf = [&](double x) { return (float)(fmin(fmax(x, lo), hi) * nom); };
    double v[NV];  // this lane's coordinate of every vertex
    {   // initial simplex: x0 and x0 with one coordinate scaled by 1.05
        const double x0 = (seed_opc && !bad && l < P) ? (double)seed_opc[(int64_t)s * P + l] / nom : 1.0;
#pragma unroll
        for (int i = 0; i < NV; ++i) v[i] = (i == l + 1) ? x0 * 1.05 : x0;
    }
    double f = INFINITY;  // value of vertex l

    // Stable sort of a group's simplex by value: vertex i goes to rank #{k : f_k < f_i} + #{k < i : f_k == f_i}.
    auto sort_all = [&](bool on) {
        int rank = 0;
        for (int k = 0; k < NV; ++k) {
            const double fk = __shfl(f, base + k);
            rank += (fk < f) || (k < l && fk == f);
        }
#pragma unroll
        for (int i = 0; i < NV; ++i) {
            const int ri = __shfl(rank, base + i);
            if (on && l < P) g.tv[ri][l] = v[i];
        }
        if (on && l < NV) g.fp[rank] = f;
        wave_sync();
        if (on) {
            if (l < P) {
#pragma unroll
                for (int i = 0; i < NV; ++i) v[i] = g.tv[i][l];
            }
            if (l < NV) f = g.fp[l];
        }
        wave_sync();
    };

    bool active = !bad;
    if (active && l < P) {
#pragma unroll
        for (int i = 0; i < NV; ++i) g.pt[i][l] = clampf(v[i]);
    } else if (!active) {
        for (int j = l; j < NV * PTS && member; j += LG) (&g.pt[0][0])[j] = 1.0f;  // something finite to simulate
    }
    int it = -1, iters = 0;  // turn -1 evaluates the initial simplex, the way a shrink does
    int32_t extra = 0;       // OPMM_ST_DEADLINE when the wall-clock budget ended the task
    for (;;) {
        bool all = active && it < 0;  // every vertex is new: evaluate the list and sort
        if (it >= 0) {
            if (it >= max_iter) break;
            // exit test (max over vertices and coordinates; fmax is exact, so the order does not matter)
            // and the centroid of the best P vertices, one coordinate per lane
            double dx = 0.0, acc = 0.0;
#pragma unroll
            for (int i = 1; i < NV; ++i) dx = fmax(dx, fabs(v[i] - v[0]));
#pragma unroll
            for (int i = 0; i < P; ++i) acc += v[i];
            const double xb = acc / (double)P;
            const double f0 = at(f, 0);
            // a NaN difference (two infinite values) does not count, as in a running fmax
            const bool wide = (l < P && !(dx <= tol_x)) || (l < NV && fabs(f - f0) > tol_f);
            const bool within = (__ballot(wide) & gmask) == 0;
            const bool late = deadline_ticks > 0 &&
                              __builtin_amdgcn_readfirstlane((int)(wall_clock64() - t0 >= deadline_ticks)) != 0;
            if (active && (within || late)) {
                if (!within) extra = OPMM_ST_DEADLINE;
                active = false;
                iters = it;
            }
            if (!__any(active)) break;
            // the four points, on the lanes that hold their coordinates
            const double w = v[NV - 1];
            const double xr = xb + (xb - w), xe = xb + 2.0 * (xb - w), xo = xb + 0.5 * (xb - w), xi = xb - 0.5 * (xb - w);
            wave_sync();
            if (active && l < P) {
                g.pt[0][l] = clampf(xr);
                g.pt[1][l] = clampf(xe);
                g.pt[2][l] = clampf(xo);
                g.pt[3][l] = clampf(xi);
            }
            wave_sync();
            const int qd = l >> 2;
            const double y = quad_eval(g.pt[qd & 3], r, tr, active && qd < 4, sd, q, dt);
            const double fr = at(y, 0), fe = at(y, 4), fo = at(y, 8), fi = at(y, 12);
            const double fn = at(f, NV - 2), fw = at(f, NV - 1);
            int dcs;
            if (fr < f0) dcs = fe < fr ? 1 : 0;
            else if (fr < fn) dcs = 0;
            else if (fr < fw) dcs = fo <= fr ? 2 : 4;
            else dcs = fi < fw ? 3 : 4;
            if (active && l == 0 && dec_out) dec_out[(int64_t)s * max_iter + it] = (int8_t)dcs;
            {   // the accepted point replaces the worst vertex and moves to its rank: after every value <= its own
                const bool put = active && dcs < 4;
                const double fnew = dcs == 0 ? fr : dcs == 1 ? fe : dcs == 2 ? fo : fi;
                const double xnew = dcs == 0 ? xr : dcs == 1 ? xe : dcs == 2 ? xo : xi;
                const int rank = __popcll(__ballot(l < NV - 1 && f <= fnew) & gmask);
                const double fprev = __shfl_up(f, 1);
                if (put) {
                    f = l < rank ? f : l == rank ? fnew : fprev;
#pragma unroll
                    for (int i = NV - 1; i >= 0; --i) v[i] = i < rank ? v[i] : (i == rank || i == 0) ? xnew : v[i - 1];
                }
            }
            all = active && dcs == 4;
            if (all) {  // every vertex but the best moves half way to it
#pragma unroll
                for (int i = 1; i < NV; ++i) {
                    v[i] = v[0] + 0.5 * (v[i] - v[0]);
                    if (l < P) g.pt[i][l] = clampf(v[i]);
                }
            }
        }
        if (__any(all)) {
            const int first = it < 0 ? 0 : 1;  // a shrink keeps the best vertex and its value
            wave_sync();
            for (int p0 = first; p0 < NV; p0 += NQ) {
                const int i = p0 + (l >> 2);
                const bool run = all && member && i < NV;
                const double y = quad_eval(g.pt[run ? i : 0], r, tr, run, sd, q, dt);
                if (run && (l & 3) == 0) g.fp[i] = y;
            }
            wave_sync();
            if (all && l >= first && l < NV) f = g.fp[l];
            sort_all(all);
        }
        ++it;
    }
    if (bad) return;
    if (active) iters = it;  // ran to the iteration cap
    if (l < P) {
        const double x = fmin(fmax(v[0], lo), hi);
        opc_out[(int64_t)s * P + l] = (float)(x * nom);
    }
    if (l == 0) {
        rmse_out[s] = (float)f;
        if (iters_out) iters_out[s] = iters;
        if (status_out) status_out[s] = st0 | extra;
    }
}

// Whether three tasks per wave (which share its instructions) finish a batch sooner than one.  While every task
// has a SIMD to itself, one does: a wave of three takes 1.2 times as long.  Up to two waves per SIMD all
// run at once, the S - simds shortest tasks beside a longer one, which the longest of them slows most: by
// nothing where a task of its length takes 0.4 of the longest's time, 1.03 times at 0.5, 1.12 at 0.6, 1.2 at 0.64,
// 1.3 at 0.73, 1.5 at 1 (an evaluation takes the time of 67 samples besides its trace's).  Past that, waves
// queue.  Measured, 400 iterations, one / three per wave: T 26-87, 1024 saccades 2.82 / 3.42 ms, 1100 3.40 /
// 3.39, 1500 3.66 / 3.43, 3072 5.28 / 3.45; T 20-150, 1100 3.86 / 4.60, 1500 4.37 / 4.62, 1900 4.72 / 4.68; all of
// 26 samples, 1025 2.52 / 2.10.
bool three_per_wave(const opmm_saccade* sacs, int S, int max_T, int simds)
{
    if (S <= simds) return false;
    if (S > 2 * simds) return true;
    int count[OPMM_MAX_T + 1] = {};
    for (int i = 0; i < S; ++i) ++count[sacs[i].T];
    int T = 0;  // of the longest among the S - simds shortest
    for (int n = 0; n < S - simds;) n += count[++T];
    return T + 67 > 0.64 * (max_T + 67);
}

}  // namespace

extern "C" {

void opmm_nm_params_default(opmm_nm_params* p)
{
    if (!p) return;
    p->max_iter = 500;
    p->tol_x = 1e-4f;
    p->tol_f = 1e-6f;
    p->box_frac = 0.25f;
    p->dt_ms = 1.0f;
    p->max_ms = 0.0f;
    p->tasks_per_wave = 0;
}

int opmm_fit_nm(opmm_ctx* ctx, const float* pos, int64_t pos_len, const opmm_saccade* sacs, int32_t S,
                const opmm_nm_params* prm, const float* seed_opc, float* opc_out, float* rmse_out, int32_t* iters_out,
                int8_t* decisions_out, int32_t* status_out, void* stream)
{
    if (!ctx) return OPMM_EINVAL;
    if (!prm || prm->max_iter < 0 || !(prm->tol_x >= 0) || !(prm->tol_f >= 0) ||
        !(prm->box_frac > 0 && prm->box_frac < 1) || !(prm->dt_ms > 0 && prm->dt_ms <= 1) || !(prm->max_ms >= 0) ||
        prm->tasks_per_wave < 0 || prm->tasks_per_wave > 2)
        return opmm_rt::fail(ctx, OPMM_EINVAL, "bad Nelder-Mead parameters");
    if (S < 0 || (S > 0 && (!pos || !sacs || !opc_out || !rmse_out))) return opmm_rt::fail(ctx, OPMM_EINVAL, "bad arguments");
    if (S == 0) return OPMM_OK;
    const hipError_t dev = hipSetDevice(opmm_rt::ctx_device(ctx));
    if (dev != hipSuccess) return opmm_rt::hip_fail(ctx, dev, "hipSetDevice");
    hipStream_t st = (hipStream_t)stream;
    opmm_rt::Ordered ord(opmm_rt::ctx_order(ctx), st);
    if (ord.error() != hipSuccess) return opmm_rt::hip_fail(ctx, ord.error(), "stream ordering");
    const SacDev* d_sacs;
    const float* proj;
    const double* qorth;
    const int32_t* status;
    int rc = opmm_rt::project_batch_full(ctx, pos, pos_len, sacs, S, &d_sacs, &proj, &qorth, &status, st);
    if (rc != OPMM_OK) return rc;
    int max_T = 1;
    for (int i = 0; i < S; ++i) max_T = std::max(max_T, (int)sacs[i].T);
    // Three staged traces of more than 1024 samples leave room for no more tasks per CU than one does (160 KB
    // of LDS), and three of the longest would not fit a block's 64 KB.
    const int G = prm->tasks_per_wave ? prm->tasks_per_wave
                  : max_T <= 1024 && three_per_wave(sacs, S, max_T, 4 * opmm_rt::ctx_cu_count(ctx)) ? 3 : 1;
    uint64_t ticks = 0;
    if (prm->max_ms > 0.0f) {
        int khz = 0;
        hipError_t e = hipDeviceGetAttribute(&khz, hipDeviceAttributeWallClockRate, opmm_rt::ctx_device(ctx));
        if (e != hipSuccess || khz <= 0) return opmm_rt::fail(ctx, OPMM_EDEVICE, "wall clock rate unavailable");
        ticks = std::max<uint64_t>(1, (uint64_t)((double)prm->max_ms * (double)khz));
    }
    const size_t lds = sizeof(R) * (size_t)G * (max_T + 1);
    const int grid = (S + G - 1) / G;
    const int* order = opmm_rt::batch_order(ctx);
    auto launch = [&](auto kernel) {
        hipLaunchKernelGGL(kernel, dim3(grid), dim3(64), lds, st, S, d_sacs, order, proj, qorth, status, seed_opc,
                           prm->max_iter, (double)prm->tol_x, (double)prm->tol_f, 1.0 - (double)prm->box_frac,
                           1.0 + (double)prm->box_frac, prm->dt_ms, max_T, ticks, opc_out, rmse_out, iters_out,
                           decisions_out, status_out);
    };
    if (G == 3) launch(nm_kernel<3>);
    else if (G == 2) launch(nm_kernel<2>);
    else launch(nm_kernel<1>);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return opmm_rt::hip_fail(ctx, e, "nm_kernel");
    return OPMM_OK;
}

}  // extern "C"
