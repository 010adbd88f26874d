// libopmm: the paper's own estimator -- a parallel Nelder-Mead per saccade
// (Section 3.3, Algorithm 1): one task per saccade, all simplex transforms of
// an iteration evaluated simultaneously, the simplex sorted every iteration,
// both exit tolerances or an iteration cap.
//
// One or two saccades per 64-lane wave.  The simplex (19 vertices x 18
// coordinates, FP64, relative to the Table 1 nominal) and the projected trace
// (sized to the batch's longest) live in LDS.  Every iteration lanes 0..21 of
// a task build and evaluate reflection, expansion, outside and inside
// contraction and the 18 shrink vertices at once; lane 0 of the task takes the
// Lagarias decision (reflection 1, expansion 2, contraction 1/2, shrink 1/2);
// the exit test, the vertex update and the stable re-sort run one coordinate
// or one vertex per lane.  Each evaluation is the same plant
// simulation and RMSE as the box search (points clamped to the search box and
// rounded to FP32, the candidate format).
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
constexpr int NPT = 4 + P;  // points per iteration: r, e, oc, ic, 18 shrink

// One task's simplex state (the trace lives in dynamic LDS after the groups).
struct NmGroup {
    double v[NV][P];
    double f[NV];
    double pt[NPT][P];
    double fp[NPT];
    double xb[P];
    double nom[P];
    double tv[NV][P];  // sort staging
    double tf[NV];
    double dxc[P];     // per-coordinate spread of the simplex
    int flag;          // exit test passed
    int dec;
    int active;        // still iterating
    int iters;         // iterations taken (set when the task stops)
};

// The simplex's iterates depend on every rounding of its costs, so this file keeps the sample-by-sample
// evaluation its results are defined by: the transition by Horner's rule on matrices and one step per
// sample (run_blocks in plant.hpp gives the same trajectories to ~1e-14 deg).
struct NmPlant {
    R a10, a11, a12, a13;       // per ms; omega row: theta, omega, x_ag, x_ant
    R a20, a22, g2;             // x_ag row: theta, x_ag, F_ag
    R a30, a33, g3;             // x_ant row: theta, x_ant, F_ant
    R q1a, q1n, q2a, q2n;       // F rows: -1/tau, pulse (activation) and post (deactivation)
    R m[4][4], x1[4][2], x2[4][2], e1[2], e2[2];  // one-sample transition in D-form (Phi - I), both pieces
    R th1, amp, sh[6], d0[6];   // equilibria (theta), pulse minus post, rest minus pulse
    double pwd;                 // PW in sample periods
};

// mechanical rows of (s*A) V, plus `acc` on the diagonal of column `diag` (-1: none)
#define OPMM_MV(s10, s11, s12, s13, s20, s22, s30, s33, sv, V0, V1, V2, V3, o0, o1, o2, o3, i0, i1, i2, i3) \
    do {                                                                                               \
        o0 = fmr(sv, V1, i0);                                                                    \
        o1 = fmr(s13, V3, fmr(s12, V2, fmr(s11, V1, fmr(s10, V0, i1))));       \
        o2 = fmr(s22, V2, fmr(s20, V0, i2));                                               \
        o3 = fmr(s33, V3, fmr(s30, V0, i3));                                               \
    } while (0)

// Horner evaluation of D = sum_{k=1..M} (hA)^k / k! for the augmented block
// matrix [[Mech, G1, G2], [0, Q1, 0], [0, 0, Q2]] whose off-diagonal blocks
// give the pulse-piece and post-piece coupling columns at once, on the step
// h/2^SQ, then SQ squarings in D-form: D_2h = D_h^2 + 2 D_h.  The Horner
// iterates P_k = I + (B/k) P_{k+1} (B = hA) are carried scaled, Q_k = c_k P_k
// with c_M = M and c_k = k c_{k+1}: then Q_M = M I + B, Q_k = c_k I + B Q_{k+1}
// and D = B Q_2 / M!, so the entries of B are formed once instead of once per
// step (fewer instructions and fewer live registers).
__device__ __forceinline__ void transition_dform(NmPlant& pl, R hfull)
{
    constexpr int M = Prec<R>::taylor_m, SQ = Prec<R>::taylor_sq;
    const R h = hfull * (R(1) / R(1 << SQ));
    const R qv[4] = {pl.q1a, pl.q1n, pl.q2a, pl.q2n};
    const R s10 = pl.a10 * h, s11 = pl.a11 * h, s12 = pl.a12 * h, s13 = pl.a13 * h;
    const R s20 = pl.a20 * h, s22 = pl.a22 * h, s30 = pl.a30 * h, s33 = pl.a33 * h;
    const R sg2 = pl.g2 * h, sg3 = pl.g3 * h;
    R sq[4];
#pragma unroll
    for (int c = 0; c < 4; ++c) sq[c] = qv[c] * h;
    R pm[4][4], px[4][4], pd[4];
    {   // Q_M = M I + B
        const R m = R(M);
        pm[0][0] = m;   pm[0][1] = h;      pm[0][2] = R(0);    pm[0][3] = R(0);
        pm[1][0] = s10; pm[1][1] = m + s11; pm[1][2] = s12;     pm[1][3] = s13;
        pm[2][0] = s20; pm[2][1] = R(0);  pm[2][2] = m + s22;  pm[2][3] = R(0);
        pm[3][0] = s30; pm[3][1] = R(0);  pm[3][2] = R(0);    pm[3][3] = m + s33;
#pragma unroll
        for (int c = 0; c < 4; ++c) {
            px[0][c] = R(0); px[1][c] = R(0);
            px[2][c] = (c & 1) ? R(0) : sg2;
            px[3][c] = (c & 1) ? sg3 : R(0);
            pd[c] = m + sq[c];
        }
    }
    R ck = R(M);
#pragma unroll
    for (int k = M - 1; k >= 1; --k) {
        // k >= 2: Q_k = c_k I + B Q_{k+1};  k == 1: D = (B / M!) Q_2
        R one, t10, t11, t12, t13, t20, t22, t30, t33, tv, tg2, tg3, tq[4];
        if (k >= 2) {
            ck = ck * R(k);
            one = ck;
            t10 = s10; t11 = s11; t12 = s12; t13 = s13; t20 = s20; t22 = s22; t30 = s30; t33 = s33;
            tv = h; tg2 = sg2; tg3 = sg3;
#pragma unroll
            for (int c = 0; c < 4; ++c) tq[c] = sq[c];
        } else {
            const R f = R(1) / ck;  // 1 / M!, rounded once
            one = R(0);
            t10 = s10 * f; t11 = s11 * f; t12 = s12 * f; t13 = s13 * f;
            t20 = s20 * f; t22 = s22 * f; t30 = s30 * f; t33 = s33 * f;
            tv = h * f; tg2 = sg2 * f; tg3 = sg3 * f;
#pragma unroll
            for (int c = 0; c < 4; ++c) tq[c] = sq[c] * f;
        }
        R nm[4][4], nx[4][4], nd[4];
#pragma unroll
        for (int c = 0; c < 4; ++c) {
            OPMM_MV(t10, t11, t12, t13, t20, t22, t30, t33, tv, pm[0][c], pm[1][c], pm[2][c], pm[3][c],
                    nm[0][c], nm[1][c], nm[2][c], nm[3][c],
                    c == 0 ? one : R(0), c == 1 ? one : R(0), c == 2 ? one : R(0), c == 3 ? one : R(0));
        }
#pragma unroll
        for (int c = 0; c < 4; ++c) {
            const R ga = (c & 1) ? R(0) : tg2 * pd[c];
            const R gn = (c & 1) ? tg3 * pd[c] : R(0);
            OPMM_MV(t10, t11, t12, t13, t20, t22, t30, t33, tv, px[0][c], px[1][c], px[2][c], px[3][c],
                    nx[0][c], nx[1][c], nx[2][c], nx[3][c], R(0), R(0), ga, gn);
            nd[c] = fmr(tq[c], pd[c], one);
        }
#pragma unroll
        for (int i = 0; i < 4; ++i) {
#pragma unroll
            for (int c = 0; c < 4; ++c) { pm[i][c] = nm[i][c]; px[i][c] = nx[i][c]; }
            pd[i] = nd[i];
        }
    }
#pragma unroll
    for (int q = 0; q < SQ; ++q) {
        R nm[4][4], nx[4][4];
#pragma unroll
        for (int i = 0; i < 4; ++i) {
#pragma unroll
            for (int c = 0; c < 4; ++c) {
                R a = pm[i][c] + pm[i][c];
#pragma unroll
                for (int k = 0; k < 4; ++k) a = fmr(pm[i][k], pm[k][c], a);
                nm[i][c] = a;
                R b = px[i][c] * (pd[c] + R(2));
#pragma unroll
                for (int k = 0; k < 4; ++k) b = fmr(pm[i][k], px[k][c], b);
                nx[i][c] = b;
            }
        }
#pragma unroll
        for (int i = 0; i < 4; ++i) {
#pragma unroll
            for (int c = 0; c < 4; ++c) { pm[i][c] = nm[i][c]; px[i][c] = nx[i][c]; }
            pd[i] = pd[i] * (pd[i] + R(2));
        }
    }
#pragma unroll
    for (int i = 0; i < 4; ++i) {
#pragma unroll
        for (int c = 0; c < 4; ++c) pl.m[i][c] = pm[i][c];
        pl.x1[i][0] = px[i][0]; pl.x1[i][1] = px[i][1];
        pl.x2[i][0] = px[i][2]; pl.x2[i][1] = px[i][3];
    }
    pl.e1[0] = pd[0]; pl.e1[1] = pd[1];
    pl.e2[0] = pd[2]; pl.e2[1] = pd[3];
}


__device__ __forceinline__ void nm_setup(const float p[P], float amp, float dt, NmPlant& pl)
{
    double pd[P];
#pragma unroll
    for (int j = 0; j < P; ++j) pd[j] = p[j];
    PlantScalars<double> c;
    plant_scalars(pd, (double)amp, c);
    pl.a10 = c.a10; pl.a11 = c.a11; pl.a12 = c.a12; pl.a13 = c.a13;
    pl.a20 = c.a20; pl.a22 = c.a22; pl.g2 = c.g2;
    pl.a30 = c.a30; pl.a33 = c.a33; pl.g3 = c.g3;
    pl.q1a = c.q1a; pl.q1n = c.q1n; pl.q2a = c.q2a; pl.q2n = c.q2n;
    transition_dform(pl, (R)dt);
    pl.th1 = c.th1;
    pl.amp = amp;
#pragma unroll
    for (int i = 0; i < 6; ++i) { pl.d0[i] = c.d0[i]; pl.sh[i] = c.sh[i]; }
    pl.pwd = (double)p[17] * rcp64((double)dt);
}

// d <- Phi d for one sample (D-form: d + D d)
__device__ __forceinline__ void step(const NmPlant& pl, const R (&x)[4][2], const R (&e)[2], R d[6])
{
    R n[4];
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
        n[i] = fmr(x[i][0], d[4], n[i]);
        n[i] = fmr(x[i][1], d[5], n[i]);
    }
    d[4] = fmr(e[0], d[4], d[4]);
    d[5] = fmr(e[1], d[5], d[5]);
#pragma unroll
    for (int i = 0; i < 4; ++i) d[i] = n[i];
}

// v <- exp(A t) v by a Taylor polynomial (degree Prec::expmv_m) in Horner form (t <= dt).
__device__ __forceinline__ void expmv(const NmPlant& pl, R qa, R qn, R t, R v[6])
{
    R w[6];
#pragma unroll
    for (int i = 0; i < 6; ++i) w[i] = v[i];
#pragma unroll
    for (int k = Prec<R>::expmv_m; k >= 1; --k) {
        R s = t * (R(1) / R(k));
        asm volatile("" : "+v"(s));
        R aw[6];
        aw[0] = w[1];
        aw[1] = fmr(pl.a13, w[3], fmr(pl.a12, w[2], fmr(pl.a11, w[1], pl.a10 * w[0])));
        aw[2] = fmr(pl.g2, w[4], fmr(pl.a22, w[2], pl.a20 * w[0]));
        aw[3] = fmr(pl.g3, w[5], fmr(pl.a33, w[3], pl.a30 * w[0]));
        aw[4] = qa * w[4];
        aw[5] = qn * w[5];
#pragma unroll
        for (int i = 0; i < 6; ++i) w[i] = fmr(s, aw[i], v[i]);
    }
#pragma unroll
    for (int i = 0; i < 6; ++i) v[i] = w[i];
}

// The sample that contains the pulse end: pulse dynamics for frac*dt, switch
// to the post piece's coordinates, post dynamics for the rest of the sample.
__device__ __forceinline__ void split_step(const NmPlant& pl, R frac, R dt, R d[6])
{
    expmv(pl, pl.q1a, pl.q1n, frac * dt, d);
#pragma unroll
    for (int i = 0; i < 6; ++i) d[i] += pl.sh[i];
    expmv(pl, pl.q2a, pl.q2n, (R(1) - frac) * dt, d);
}

// Run the trajectory theta_k, k = 0..T-1, calling sink(k, dtheta, theta_eq)
// with theta_k = dtheta + theta_eq.  kmin/kmax: wave-uniform bounds of the
// lanes' pulse-end samples; samples below kmin are pulse for every lane and
// samples above kmax post for every lane, so only [kmin, kmax] branches.
template <int UNROLL, class Sink>
__device__ __forceinline__ void run_steps(const NmPlant& pl, int T, R dt, int k0, R frac,
                                               int kmin, int kmax, Sink& sink)
{
    R d[6];
#pragma unroll
    for (int i = 0; i < 6; ++i) d[i] = pl.d0[i];
    R theq = pl.th1;
    if (k0 < 0) {  // PW <= 0: no pulse, the step acts from t = 0
#pragma unroll
        for (int i = 0; i < 6; ++i) d[i] += pl.sh[i];
        theq = pl.amp;
    }
    int k = 0;
    const int ka = min(kmin, T);
#pragma unroll UNROLL
    for (; k < ka; ++k) {
        sink(k, d[0], theq);
        step(pl, pl.x1, pl.e1, d);
    }
    const int kb = min(kmax, T - 1);
#pragma unroll 1
    for (; k <= kb; ++k) {
        sink(k, d[0], theq);
        if (k < k0) {
            step(pl, pl.x1, pl.e1, d);
        } else if (k == k0) {
            split_step(pl, frac, dt, d);
            theq = pl.amp;
        } else {
            step(pl, pl.x2, pl.e2, d);
        }
    }
#pragma unroll UNROLL
    for (; k < T; ++k) {
        sink(k, d[0], theq);
        step(pl, pl.x2, pl.e2, d);
    }
}

struct SseSinkNm {
    const R* r;
    double sse;
    __device__ __forceinline__ void operator()(int k, R dth, R theq)
    {
        R e = (r[k] - theq) - dth;
        sse = fma((double)e, (double)e, sse);
    }
};

// RMSE of point x (relative to nominal) for this lane; all 64 lanes call it
// (wave-uniform bounds), `valid` lanes' results are meaningful.
__device__ double nm_eval(const NmGroup& g, const R* r, const double* x, bool valid, const SacDev& sd, double q,
                          float dt, double lo, double hi)
{
    float p[P];
#pragma unroll
    for (int j = 0; j < P; ++j) {
        double v = valid ? x[j] : 1.0;
        v = fmin(fmax(v, lo), hi);
        p[j] = (float)(v * g.nom[j]);
    }
    NmPlant pl;
    nm_setup(p, sd.amp, dt, pl);
    R frac;
    int k0 = pulse_end_sample(pl.pwd, sd.T, frac);
    int kmin = __builtin_amdgcn_readfirstlane(wave_min(valid ? k0 : 0x7FFFFFFF));
    int kmax = __builtin_amdgcn_readfirstlane(wave_max(valid ? k0 : -0x7FFFFFFF));
    SseSinkNm sink{r, 0.0};
    if (valid) run_steps<2>(pl, sd.T, (R)dt, k0, frac, kmin, kmax, sink);
    double rm = sqrt((sink.sse + q) / ((double)sd.T * sd.C));
    return (rm >= 0.0 && rm <= 1.7976931348623157e308) ? rm : INFINITY;
}

// Stable sort of a simplex by value, in parallel: vertex i goes to rank
// #{k : f_k < f_i} + #{k < i : f_k == f_i} (the order a stable insertion sort
// gives), each lane of the group moves one row.  Every lane of the wave calls it.
__device__ void nm_sort(NmGroup& g, int l, bool on)
{
    if (on && l < NV) {
        const double fi = g.f[l];
        int rank = 0;
        for (int k = 0; k < NV; ++k) rank += (g.f[k] < fi) || (k < l && g.f[k] == fi);
        for (int j = 0; j < P; ++j) g.tv[rank][j] = g.v[l][j];
        g.tf[rank] = fi;
    }
    __syncthreads();
    if (on && l < NV) {
        for (int j = 0; j < P; ++j) g.v[l][j] = g.tv[l][j];
        g.f[l] = g.tf[l];
    }
    __syncthreads();
}

// G tasks per 64-lane wave (1 or 2): lanes 64/G * g .. of group g work on saccade G * block + g, 22
// of them evaluating.  Every group runs the same instruction stream; a finished group's lanes idle
// until the other one ends.  deadline_ticks > 0: a task still iterating when that many ticks of the
// wall clock (wall_clock64) have passed since the launch started ends there with OPMM_ST_DEADLINE.
template <int G>
__global__ __launch_bounds__(64) void nm_kernel(int S, const SacDev* __restrict__ sacs, const float* __restrict__ proj,
                                                const double* __restrict__ qorth, const int32_t* __restrict__ status_in,
                                                const float* __restrict__ seed_opc, int max_iter, double tol_x,
                                                double tol_f, double lo, double hi, float dt, int max_T,
                                                uint64_t deadline_ticks, float* opc_out, float* rmse_out,
                                                int32_t* iters_out, int8_t* dec_out, int32_t* status_out)
{
    constexpr int LG = 64 / G;
    __shared__ NmGroup gs[G];
    __shared__ int s_stop;
    extern __shared__ R rbuf[];  // [G][max_T] projected traces
    const int lane = threadIdx.x, gi = lane / LG, l = lane % LG;
    const int s = G * blockIdx.x + gi;
    const bool have = s < S;
    NmGroup& g = gs[gi];
    R* r = rbuf + (int64_t)gi * max_T;
    const SacDev sd = sacs[have ? s : 0];
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
    if (!bad) {
        for (int k = l; k < sd.T; k += LG) r[k] = (R)proj[sd.proj_off + k];
        if (l < P) g.nom[l] = nominal_param_f64(l, (double)sd.dur);
    }
    if (l == 0) g.active = bad ? 0 : 1;
    __syncthreads();
    if (!bad && l < NV) {  // initial simplex: x0 and x0 with one coordinate scaled by 1.05
        for (int j = 0; j < P; ++j) g.v[l][j] = seed_opc ? (double)seed_opc[(int64_t)s * P + j] / g.nom[j] : 1.0;
        if (l > 0) g.v[l][l - 1] = g.v[l][l - 1] * 1.05;
    }
    __syncthreads();
    {
        const bool valid = !bad && l < NV;
        double fv = nm_eval(g, r, g.v[valid ? l : 0], valid, sd, q, dt, lo, hi);
        if (valid) g.f[l] = fv;
    }
    __syncthreads();
    nm_sort(g, l, !bad);
    int it = 0;
    int32_t extra = 0;  // OPMM_ST_DEADLINE when the wall-clock budget ended the task
    for (; it < max_iter; ++it) {
        const bool on = g.active != 0;
        // exit test (max over vertices and coordinates; fmax is exact, so the order does not matter)
        // and the centroid of the best P vertices, one coordinate per lane
        if (on && l < P) {
            double dx = 0.0, acc = 0.0;
            for (int i = 1; i < NV; ++i) dx = fmax(dx, fabs(g.v[i][l] - g.v[0][l]));
            for (int i = 0; i < P; ++i) acc += g.v[i][l];
            g.dxc[l] = dx;
            g.xb[l] = acc / (double)P;
        }
        __syncthreads();
        if (on && l == 0) {
            double dx = 0.0, df = 0.0;
            for (int i = 1; i < NV; ++i) df = fmax(df, fabs(g.f[i] - g.f[0]));
            for (int j = 0; j < P; ++j) dx = fmax(dx, g.dxc[j]);
            g.flag = (dx <= tol_x && df <= tol_f) ? 1 : 0;
        }
        if (lane == 0) s_stop = deadline_ticks > 0 && wall_clock64() - t0 >= deadline_ticks ? 1 : 0;
        __syncthreads();
        const bool stop_now = on && (g.flag || s_stop);  // uniform over the group
        if (stop_now && !g.flag) extra = OPMM_ST_DEADLINE;
        __syncthreads();  // every lane has read the flags before the group stops
        if (stop_now && l == 0) {
            g.active = 0;
            g.iters = it;
        }
        __syncthreads();
        // the loop ends when no group is still iterating
        int any = 0;
#pragma unroll
        for (int k = 0; k < G; ++k) any |= gs[k].active;
        if (!any) break;
        const bool act = g.active != 0;
        if (act && l < NPT) {
            for (int j = 0; j < P; ++j) {
                const double xb = g.xb[j], w = g.v[NV - 1][j];
                double x;
                if (l == 0) x = xb + (xb - w);
                else if (l == 1) x = xb + 2.0 * (xb - w);
                else if (l == 2) x = xb + 0.5 * (xb - w);
                else if (l == 3) x = xb - 0.5 * (xb - w);
                else x = g.v[0][j] + 0.5 * (g.v[l - 3][j] - g.v[0][j]);
                g.pt[l][j] = x;
            }
        }
        __syncthreads();
        {
            const bool valid = act && l < NPT;
            double fv = nm_eval(g, r, g.pt[valid ? l : 0], valid, sd, q, dt, lo, hi);
            if (valid) g.fp[l] = fv;
        }
        __syncthreads();
        if (act && l == 0) {
            const double fr = g.fp[0];
            int d;
            if (fr < g.f[0]) d = g.fp[1] < fr ? 1 : 0;
            else if (fr < g.f[NV - 2]) d = 0;
            else if (fr < g.f[NV - 1]) d = g.fp[2] <= fr ? 2 : 4;
            else d = g.fp[3] < g.f[NV - 1] ? 3 : 4;
            g.dec = d;
            if (dec_out) dec_out[(int64_t)s * max_iter + it] = (int8_t)d;
        }
        __syncthreads();
        if (act) {
            // the accepted point replaces the worst vertex, or the shrink replaces all but the best;
            // one coordinate per lane
            const int d = g.dec;
            if (l < P) {
                if (d < 4) g.v[NV - 1][l] = g.pt[d][l];
                else
                    for (int i = 1; i < NV; ++i) g.v[i][l] = g.pt[3 + i][l];
            }
            if (l == 0) {
                if (d < 4) g.f[NV - 1] = g.fp[d];
                else
                    for (int i = 1; i < NV; ++i) g.f[i] = g.fp[3 + i];
            }
        }
        __syncthreads();
        nm_sort(g, l, act);
    }
    if (bad) return;
    if (l == 0 && g.active) g.iters = it;  // ran to the iteration cap
    if (l < P) {
        double x = fmin(fmax(g.v[0][l], lo), hi);
        opc_out[(int64_t)s * P + l] = (float)(x * g.nom[l]);
    }
    if (l == 0) {
        rmse_out[s] = (float)g.f[0];
        if (iters_out) iters_out[s] = g.iters;
        if (status_out) status_out[s] = st0 | extra;
    }
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
    // two tasks per wave once the batch has more tasks than the device holds waves of this kernel (one
    // per SIMD: it takes 256 VGPRs and ~110 AGPRs); a wave's time is its slower task's, so below that
    // one per wave is as fast.  Measured on 4096 full-estimation saccades: 32k -> 51k saccades/s.
    const int cus = opmm_rt::ctx_cu_count(ctx);
    const int G = prm->tasks_per_wave ? prm->tasks_per_wave : (S > 4 * cus ? 2 : 1);
    uint64_t ticks = 0;
    if (prm->max_ms > 0.0f) {
        int khz = 0;
        hipError_t e = hipDeviceGetAttribute(&khz, hipDeviceAttributeWallClockRate, opmm_rt::ctx_device(ctx));
        if (e != hipSuccess || khz <= 0) return opmm_rt::fail(ctx, OPMM_EDEVICE, "wall clock rate unavailable");
        ticks = std::max<uint64_t>(1, (uint64_t)((double)prm->max_ms * (double)khz));
    }
    const size_t lds = sizeof(R) * (size_t)G * max_T;
    const int grid = (S + G - 1) / G;
    if (G == 2)
        hipLaunchKernelGGL(nm_kernel<2>, dim3(grid), dim3(64), lds, st, S, d_sacs, proj, qorth, status, seed_opc,
                           prm->max_iter, (double)prm->tol_x, (double)prm->tol_f, 1.0 - (double)prm->box_frac,
                           1.0 + (double)prm->box_frac, prm->dt_ms, max_T, ticks, opc_out, rmse_out, iters_out,
                           decisions_out, status_out);
    else
        hipLaunchKernelGGL(nm_kernel<1>, dim3(grid), dim3(64), lds, st, S, d_sacs, proj, qorth, status, seed_opc,
                           prm->max_iter, (double)prm->tol_x, (double)prm->tol_f, 1.0 - (double)prm->box_frac,
                           1.0 + (double)prm->box_frac, prm->dt_ms, max_T, ticks, opc_out, rmse_out, iters_out,
                           decisions_out, status_out);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return opmm_rt::hip_fail(ctx, e, "nm_kernel");
    return OPMM_OK;
}

}  // extern "C"
