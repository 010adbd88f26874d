// libopmm: saccade extraction from a raw gaze stream by velocity threshold
// (I-VT, Salvucci & Goldberg 2000), the identification step the paper runs
// before estimation (Section 3.1: recorded, cleaned, saccades extracted;
// Section 4: I-VT, saccades shorter than 6 ms discarded).
//
// A sample k >= 1 is a saccade sample when its point-to-point speed
// |g_k - g_{k-1}| / dt exceeds the threshold; a saccade is a maximal run of
// saccade samples, its trace the run with the sample before it (the last
// fixation sample) prepended, re-based to that sample.  Runs with duration
// (T - 1) * dt below min_dur_ms or amplitude below min_amp_deg are dropped.
// Output order is the stream order.  Two launches: ivt_pass<false> counts each tile's kept runs and
// their samples, ivt_pass<true> sums the tiles before its own and emits (a stream with more records than the
// kept host staging holds is passed once more for those).  Both find the runs the same
// way: the tile's saccade samples as bit words (a ballot per 64 samples), the last sample of a run from
// a word and its neighbour, its length from the bits before it.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <cstring>

#include "../../include/opmm.h"
#include "runtime.hpp"

namespace {

constexpr int IVT_TPB = 256;
constexpr int CHUNK = 2048;                  // samples whose flags a block holds at a time
constexpr int WORDS = CHUNK / 64;
constexpr int MAX_TILES = 4096;              // a tile is as many chunks as this bound needs (one up to 8.4 M samples)
constexpr int HOST_RECS = 16384;             // records written straight to pinned host memory
static_assert(WORDS <= 64 && WORDS % (IVT_TPB / 64) == 0, "one lane of wave 0 per word");

// A gaze or trace sample; the caller's buffers are aligned to a float.
struct __attribute__((packed, aligned(4))) Sample { float x, y; };

struct IvtArgs {
    const Sample* g;
    int64_t N;
    float thr2, dt, min_dur, min_amp;
    int32_t max_T;
    int chunks_per_tile;
    // per tile: kept runs and their samples (written by the first pass)
    int32_t* cnt;
    int64_t* len;
    // second pass
    uint64_t seed_base;
    int32_t max_out;
    int64_t pos_cap;
    Sample* pos;
    opmm_saccade* recs;  // records first .. first + n_recs - 1: pinned host, or device (first > 0: no traces then)
    int64_t* src;
    int32_t first, n_recs;
    int32_t* emitted;    // pinned host, per tile
};

__device__ __forceinline__ bool fast(const IvtArgs& A, int64_t k)
{
    if (k < 1 || k >= A.N) return false;
    const Sample p = A.g[k], q = A.g[k - 1];
    const float dx = p.x - q.x, dy = p.y - q.y;
    return dx * dx + dy * dy > A.thr2;
}

__device__ __forceinline__ int64_t wave_sum(int64_t v)
{
#pragma unroll
    for (int o = 32; o >= 1; o >>= 1) v += (int64_t)__shfl_xor((long long)v, o);
    return v;
}

// Bound by latency, not bandwidth: 2048 samples per block put a ten-minute 1 kHz stream (580 k samples, 4.6 MB)
// on 284 blocks, each a handful of dependent steps (flags, gathers of the runs' ends, copies).  Both
// passes together take 17 us there; the five kernels before them (serial walks along each run, a
// one-block scan) took 64 us, and with their allocations, copies and waits a call through the
// binding 249 us against 46 us now.
template <bool EMIT>
__global__ __launch_bounds__(IVT_TPB) void ivt_pass(IvtArgs A)
{
    __shared__ uint64_t bits[WORDS + 1];
    __shared__ int64_t s_carry;                              // saccade samples right before the chunk
    __shared__ int64_t s_cnt[IVT_TPB / 64], s_len[IVT_TPB / 64];
    __shared__ int s_kept;
    __shared__ int64_t s_klen;
    __shared__ int k_last[EMIT ? CHUNK / 2 : 1], k_T[EMIT ? CHUNK / 2 : 1], k_off[EMIT ? CHUNK / 2 : 1];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    int64_t cnt = 0, len = 0;  // kept runs and their samples before the chunk: of the tile, or (EMIT) of the stream
    if (EMIT) {
        for (int i = tid; i < (int)blockIdx.x; i += IVT_TPB) { cnt += A.cnt[i]; len += A.len[i]; }
        cnt = wave_sum(cnt);
        len = wave_sum(len);
        if (lane == 0) { s_cnt[wave] = cnt; s_len[wave] = len; }
        __syncthreads();
        cnt = len = 0;
        for (int w = 0; w < IVT_TPB / 64; ++w) { cnt += s_cnt[w]; len += s_len[w]; }
    }
    int64_t out = 0;  // records emitted by this thread
    for (int ch = 0; ch < A.chunks_per_tile; ++ch) {
        const int64_t c0 = ((int64_t)blockIdx.x * A.chunks_per_tile + ch) * CHUNK;
        if (c0 >= A.N) break;
        uint64_t w0 = 0;
#pragma unroll
        for (int i = 0; i < WORDS / (IVT_TPB / 64); ++i) {
            const int w = wave * (WORDS / (IVT_TPB / 64)) + i;
            const uint64_t b = __ballot(fast(A, c0 + 64 * w + lane));
            if (i == 0) w0 = b;
            if (lane == 0) bits[w] = b;
        }
        if (tid == IVT_TPB - 1) bits[WORDS] = fast(A, c0 + CHUNK) ? 1 : 0;
        if (wave == 0) {  // a run may come in from before the chunk: its length so far, up to max_T
            int64_t n = 0;
            if (w0 & 1)
                while (n < A.max_T) {
                    const uint64_t b = __ballot(fast(A, c0 - 1 - n - lane));
                    const int ones = b == ~0ull ? 64 : __builtin_ctzll(~b);
                    n += ones;
                    if (ones < 64) break;
                }
            if (lane == 0) s_carry = n;
        }
        __syncthreads();
        if (wave == 0) {
            uint64_t keep = 0;
            int mine = 0;
            int64_t samples = 0;
            // length of the run that ends at bit j of word `lane`
            auto run_length = [&](int j) {
                const uint64_t inv = ~(bits[lane] << (63 - j));
                int64_t n = inv ? __builtin_clzll(inv) : 64;
                if (n <= j) return n;
                n = j + 1;
                int w = lane - 1;
                for (; w >= 0 && bits[w] == ~0ull; --w) n += 64;
                return n + (w >= 0 ? (int64_t)__builtin_clzll(~bits[w]) : s_carry);
            };
            if (lane < WORDS) {
                uint64_t e = bits[lane] & ~((bits[lane] >> 1) | (bits[lane + 1] << 63));  // last samples of runs
                while (e) {
                    const int j = __builtin_ctzll(e);
                    e &= e - 1;
                    const int64_t T = run_length(j) + 1;  // with the fixation sample before the run
                    if (!((float)(T - 1) * A.dt >= A.min_dur && T <= A.max_T)) continue;
                    const int64_t k1 = c0 + 64 * lane + j;
                    const Sample p = A.g[k1], q = A.g[k1 - T + 1];
                    const float dx = p.x - q.x, dy = p.y - q.y;
                    if (!(sqrtf(dx * dx + dy * dy) >= A.min_amp)) continue;
                    keep |= 1ull << j;
                    ++mine;
                    samples += T;
                }
            }
            int before = mine;
            int64_t sbefore = samples;
#pragma unroll
            for (int o = 1; o < WORDS; o <<= 1) {  // inclusive scan over the words
                const int u = __shfl_up(before, o);
                const int64_t v = (int64_t)__shfl_up((long long)sbefore, o);
                if (lane >= o) { before += u; sbefore += v; }
            }
            if (lane == WORDS - 1) { s_kept = before; s_klen = sbefore; }
            if (EMIT) {
                int i = before - mine;
                int off = (int)(sbefore - samples);
                while (keep) {
                    const int j = __builtin_ctzll(keep);
                    keep &= keep - 1;
                    const int T = (int)run_length(j) + 1;
                    k_last[i] = 64 * lane + j;
                    k_T[i] = T;
                    k_off[i] = off;
                    ++i;
                    off += T;
                }
            }
        }
        __syncthreads();
        const int kept = s_kept;
        const int64_t klen = s_klen;
        if (EMIT) {
            // The output is a prefix of the stream's kept runs: both bounds grow along it.
            auto past = [&](int i) { return cnt + i >= A.max_out || 2 * (len + k_off[i] + k_T[i]) > A.pos_cap; };
            // a record per thread
            for (int i = tid; i < kept && !past(i); i += IVT_TPB) {
                ++out;
                const int64_t o = cnt + i;
                if (o < A.first || o - A.first >= A.n_recs) continue;
                const int T = k_T[i];
                const int64_t k1 = c0 + k_last[i], k = k1 - T + 1;
                const Sample s0 = A.g[k], s1 = A.g[k1];
                const float dx = s1.x - s0.x, dy = s1.y - s0.y;
                float d = atan2f(dy, dx) * (180.0f / 3.14159265358979f);
                if (d < 0.0f) d += 360.0f;
                opmm_saccade s;
                s.pos_offset = 2 * (len + k_off[i]);
                s.T = T;
                s.C = 2;
                s.amp_deg = sqrtf(dx * dx + dy * dy);
                s.dir_deg = d;
                s.dur_ms = (float)(T - 1) * A.dt;
                s.n_cand = 0;
                s.seed = A.seed_base + (uint64_t)k;
                A.recs[o - A.first] = s;
                A.src[o - A.first] = k;
            }
            // a trace sample per thread, its run by bisection.  (A wave per run, its record by one lane, serialised
            // chunks of many short runs: 100 k samples that move in every other one took 386 us a call, 70 now; a
            // recording with one saccade in 290 samples takes the same 40 us either way.)
            if (A.first == 0)
                for (int j = tid; j < klen; j += IVT_TPB) {
                    int i = 0;
                    for (int n = kept; n > 1;) {  // last run that starts at or before j
                        const int h = n >> 1;
                        if (k_off[i + h] <= j) { i += h; n -= h; }
                        else n = h;
                    }
                    if (past(i)) break;
                    const int64_t k = c0 + k_last[i] - k_T[i] + 1;
                    const Sample p = A.g[k + j - k_off[i]], s0 = A.g[k];
                    A.pos[len + j] = Sample{p.x - s0.x, p.y - s0.y};
                }
        }
        cnt += kept;
        len += klen;
        __syncthreads();  // the chunk's words and lists are read; the next chunk may overwrite them
    }
    if (EMIT) {
        out = wave_sum(out);
        if (lane == 0) s_cnt[wave] = out;
        __syncthreads();
        for (int w = 1; w < IVT_TPB / 64; ++w) out += s_cnt[w];
        if (tid == 0) A.emitted[blockIdx.x] = (int32_t)out;
    } else if (tid == 0) {
        A.cnt[blockIdx.x] = (int32_t)cnt;
        A.len[blockIdx.x] = len;
    }
}

}  // namespace

extern "C" {

int opmm_ivt_extract(opmm_ctx* ctx, const float* gaze, int64_t N, float dt_ms, float vel_thresh_deg_s,
                     float min_dur_ms, float min_amp_deg, int32_t max_T, uint64_t seed_base, int32_t max_out,
                     opmm_saccade* sacs_out, float* pos_out, int64_t pos_cap, int64_t* src_start_out,
                     int32_t* n_out, void* stream)
{
    if (!ctx || !n_out) return OPMM_EINVAL;
    *n_out = 0;
    if (N < 0 || (N > 0 && !gaze) || !(dt_ms > 0) || !(vel_thresh_deg_s >= 0) || !(min_dur_ms >= 0) ||
        !(min_amp_deg >= 0) || max_T < 2 || max_T > OPMM_MAX_T || max_out < 0 ||
        (max_out > 0 && (!sacs_out || !pos_out)))
        return opmm_rt::fail(ctx, OPMM_EINVAL, "bad I-VT arguments");
    if (N < 2 || max_out == 0) return OPMM_OK;
    // the staging below is made once and kept: on the context's device, whichever is current now
    const hipError_t dev = hipSetDevice(opmm_rt::ctx_device(ctx));
    if (dev != hipSuccess) return opmm_rt::hip_fail(ctx, dev, "hipSetDevice");
    hipStream_t st = (hipStream_t)stream;
    const float v_per_sample = vel_thresh_deg_s * dt_ms * 1e-3f;  // deg per sample at the threshold
    const int64_t chunks = (N + CHUNK - 1) / CHUNK;
    const int per_tile = (int)((chunks + MAX_TILES - 1) / MAX_TILES);
    const int tiles = (int)((chunks + per_tile - 1) / per_tile);
    // kept runs are separated by a slow sample and hold at least min_dur / dt samples
    const double shortest = std::max(1.0, std::floor((double)min_dur_ms / (double)dt_ms) - 1.0);
    const int64_t cap = std::min<int64_t>(max_out, (int64_t)((double)N / (shortest + 1.0)) + 1);
    const int host_recs = (int)std::min<int64_t>(cap, HOST_RECS);
    int rc = OPMM_OK;
    auto ok = [&](hipError_t e, const char* w) { if (rc == OPMM_OK && e != hipSuccess) rc = opmm_rt::hip_fail(ctx, e, w); };
    // pinned host: emitted [MAX_TILES], first samples, records; kept between calls (every call waits for its
    // kernels before it returns)
    const size_t emitted_bytes = sizeof(int32_t) * MAX_TILES;
    char *hp = nullptr, *tp = nullptr;
    if ((rc = opmm_rt::ctx_ivt_stage(ctx, emitted_bytes + (sizeof(opmm_saccade) + sizeof(int64_t)) * (size_t)host_recs,
                                     &hp, (sizeof(int64_t) + sizeof(int32_t)) * MAX_TILES, &tp)) != OPMM_OK)
        return rc;
    int32_t* h_emitted = (int32_t*)hp;
    int64_t* h_src = (int64_t*)(hp + emitted_bytes);
    opmm_saccade* h_recs = (opmm_saccade*)(h_src + host_recs);
    IvtArgs A;
    A.g = (const Sample*)gaze;
    A.N = N;
    A.thr2 = v_per_sample * v_per_sample;
    A.dt = dt_ms;
    A.min_dur = min_dur_ms;
    A.min_amp = min_amp_deg;
    A.max_T = max_T;
    A.chunks_per_tile = per_tile;
    A.len = (int64_t*)tp;
    A.cnt = (int32_t*)(A.len + MAX_TILES);
    A.seed_base = seed_base;
    A.max_out = (int32_t)cap;
    A.pos_cap = pos_cap;
    A.pos = (Sample*)pos_out;
    A.recs = h_recs;
    A.src = h_src;
    A.first = 0;
    A.n_recs = host_recs;
    A.emitted = h_emitted;
    hipLaunchKernelGGL(ivt_pass<false>, dim3(tiles), dim3(IVT_TPB), 0, st, A);
    ok(hipGetLastError(), "ivt_pass");
    hipLaunchKernelGGL(ivt_pass<true>, dim3(tiles), dim3(IVT_TPB), 0, st, A);
    ok(hipGetLastError(), "ivt_pass");
    ok(hipStreamSynchronize(st), "sync");
    if (rc == OPMM_OK) {
        int64_t n = 0;
        for (int i = 0; i < tiles; ++i) n += h_emitted[i];
        const int64_t nh = std::min<int64_t>(n, host_recs);
        // Device memory for the records past the pinned ones, now that their number is known: max_out only bounds it
        // (allocated for that bound, 580 k samples with 2000 saccades and room for 100000 took 121 us instead of 74,
        // and 4 MB; 20 M samples with 70700 take 488 us instead of 408 with the third pass).
        const size_t more = (size_t)(n - nh);
        char* dp = nullptr;
        if (more > 0) {
            ok(hipMallocAsync((void**)&dp, (sizeof(opmm_saccade) + sizeof(int64_t)) * more, st), "alloc");
            if (rc != OPMM_OK) return rc;
            A.src = (int64_t*)dp;
            A.recs = (opmm_saccade*)(A.src + more);
            A.first = host_recs;
            A.n_recs = (int32_t)more;
            hipLaunchKernelGGL(ivt_pass<true>, dim3(tiles), dim3(IVT_TPB), 0, st, A);
            ok(hipGetLastError(), "ivt_pass");
        }
        std::memcpy(sacs_out, h_recs, sizeof(opmm_saccade) * (size_t)nh);
        if (src_start_out) std::memcpy(src_start_out, h_src, sizeof(int64_t) * (size_t)nh);
        if (more > 0) {
            ok(hipMemcpyAsync(sacs_out + nh, A.recs, sizeof(opmm_saccade) * more, hipMemcpyDeviceToHost, st), "copy");
            if (src_start_out)
                ok(hipMemcpyAsync(src_start_out + nh, A.src, sizeof(int64_t) * more, hipMemcpyDeviceToHost, st), "copy");
            ok(hipStreamSynchronize(st), "sync");
            (void)hipFreeAsync(dp, st);
        }
        if (rc == OPMM_OK) *n_out = (int32_t)n;
    }
    return rc;
}

}  // extern "C"
