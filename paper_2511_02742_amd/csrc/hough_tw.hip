// Time-sliced track finding with track extension (paper Sec. 4: three-hit
// seeds on consecutive vanes extrapolated to neighbouring vanes inside 10 ns
// windows that slide by 5 ns, flagged candidates continued first in the
// next window; Sec. 5: the Hough seeds of each window).
//
// Layout: a batch of independent timelines (CSR offsets over time-sorted
// hits). A timeline's windows are processed in order, those of different
// timelines independently: one workgroup takes a timeline through all its
// windows in one launch (tw::run in hough_tw.h). Per window it
//   1. skips windows that hold nothing to do (no flagged track and fewer unused
//      hits than a candidate needs): one wave, from the hit times it holds;
//   2. continues the tracks flagged in the window before, in track order;
//   3. collects the window's unused hits as one event and runs the library's
//      event finder on it;
//   4. seeds a track from each Hough candidate, in emission order, from three of
//      its unused hits on consecutive vanes, and extends it at both ends.
// Steps 2 and 4 are serial by definition (a hit taken by one track is gone for
// the next) and run in one wave on the window's hits in LDS, sorted by vane: an
// extension step reads one vane's hits and keeps the smallest (distance, index),
// so its choice does not depend on the lane order. A track's hits are a doubly
// linked list over the hit arrays; tracks are written out at the end.
//
// Bound by the chain of dependent steps of a timeline: 64 timelines at 6
// decays/ns take 150 us a window (73 us of it the finder, 52 us the seeds), at
// 0.06 decays/ns 5.6 us (a window in six runs the finder, 19 us). Three launches
// per window step of all timelines, with a wave per timeline scanning device
// memory for every extension, took 590 and 65 us.

#include <hip/hip_runtime.h>

#include <algorithm>
#include <climits>
#include <cmath>
#include <string>

#include "hough_internal.h"
#include "hough_runtime.h"
#include "hough_tf.h"
#include "hough_tw.h"

namespace hough {
namespace {

__device__ __forceinline__ int lane() { return threadIdx.x & 63; }

__device__ __forceinline__ int64_t slot0(const TwArgs &A, int b, int64_t base) { return base / 3 + b; }

// Clears the tracks, and puts the event finder's arguments in device memory (wide:
// a second shape's behind them, or no more).
__global__ void k_tw_init(TwArgs A, FindArgs F, FindArgs wide) {
    const int64_t stride = (int64_t)gridDim.x * blockDim.x;
    for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < A.n_total; i += stride) {
        A.used[i] = -1;
        A.up[i] = -1;
        A.down[i] = -1;
    }
    for (int64_t b = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; b < A.n_tl; b += stride) {
        A.ntr[b] = 0;
        A.tl_hits[b] = 0;
        A.tl_cand[b] = 0;
        A.tl_carry[b] = 0;
    }
    if (blockIdx.x == 0 && threadIdx.x == 0) {
        A.err[0] = 0;
        A.err[1] = LLONG_MAX;
        A.find[0] = F;
        if (A.pick != nullptr) {
            A.find[1] = wide;
            *A.pick = 0;
        }
    }
}

// Offsets, hit fields and the time order of every timeline, and whether a window
// may hold more than pick_hits hits.
__global__ __launch_bounds__(256) void k_tw_validate(TwArgs A) {
    const int b = blockIdx.x;
    const int64_t base = A.offsets[b], end = A.offsets[b + 1];
    if (threadIdx.x == 0) {
        bool bad = base < 0 || end < base || end > A.n_total || (b == 0 && base != 0) ||
                   (b == A.n_tl - 1 && end != A.n_total);
        if (bad) atomicMin(&A.err[0], (long long)HOUGH_ERR_INVALID_ARG);
    }
    if (base < 0 || end < base || end > A.n_total) return;
    for (int64_t i = base + threadIdx.x; i < end; i += blockDim.x) {
        const float ti = A.t[i];
        const int v = A.vane[i];
        const bool bad = v < 0 || v >= A.n_vanes || !(fabsf(A.z[i]) <= HOUGH_Z_LIMIT) || !isfinite(A.r[i]) ||
                         !isfinite(ti) || ti < 0.0f || (i > base && ti < A.t[i - 1]);
        if (bad) {
            atomicMin(&A.err[0], (long long)HOUGH_ERR_DATA);
            atomicMin(&A.err[1], (long long)i);
        }
        if (A.pick != nullptr && i + A.pick_hits < end && A.t[i + A.pick_hits] - ti <= A.window_ns) *A.pick = 1;
    }
}

// Track and hit bases of every timeline, and the counts (one block).
__global__ __launch_bounds__(1024) void k_tw_out_scan(TwArgs A) {
    __shared__ int64_t pt[1024], ph[1024];
    __shared__ int64_t ct, chh, ccand, ccarry;
    const bool ok = A.err[0] == 0;
    if (threadIdx.x == 0) ct = chh = ccand = ccarry = 0;
    __syncthreads();
    for (int32_t b0 = 0; b0 < A.n_tl; b0 += 1024) {
        const int32_t b = b0 + threadIdx.x;
        const int64_t vt = (b < A.n_tl && ok) ? A.ntr[b] : 0, vh = (b < A.n_tl && ok) ? A.tl_hits[b] : 0;
        pt[threadIdx.x] = vt;
        ph[threadIdx.x] = vh;
        if (b < A.n_tl) {
            atomicAdd((unsigned long long *)&ccand, (unsigned long long)A.tl_cand[b]);
            atomicAdd((unsigned long long *)&ccarry, (unsigned long long)A.tl_carry[b]);
        }
        __syncthreads();
        for (int o = 1; o < 1024; o <<= 1) {
            const int64_t at = threadIdx.x >= o ? pt[threadIdx.x - o] : 0;
            const int64_t ah = threadIdx.x >= o ? ph[threadIdx.x - o] : 0;
            __syncthreads();
            pt[threadIdx.x] += at;
            ph[threadIdx.x] += ah;
            __syncthreads();
        }
        if (b < A.n_tl) {
            A.tl_tbase[b] = ct + pt[threadIdx.x] - vt;
            A.tl_hbase[b] = chh + ph[threadIdx.x] - vh;
        }
        __syncthreads();
        if (threadIdx.x == 1023) {
            ct += pt[1023];
            chh += ph[1023];
        }
        __syncthreads();
    }
    if (threadIdx.x == 0) {
        const long long st = A.err[0];
        A.counts[HOUGH_TW_COUNT_TRACKS] = st ? 0 : ct;
        A.counts[HOUGH_TW_COUNT_HITS] = st ? 0 : chh;
        A.counts[HOUGH_TW_COUNT_STATUS] = st;
        A.counts[HOUGH_TW_COUNT_DETAIL] = A.err[1] == LLONG_MAX ? -1 : A.err[1];
        A.counts[HOUGH_TW_COUNT_WINDOWS] = A.n_windows;
        A.counts[HOUGH_TW_COUNT_CANDIDATES] = ccand;
        A.counts[HOUGH_TW_COUNT_CONTINUED] = ccarry;
        for (int i = HOUGH_TW_COUNT_CONTINUED + 1; i < HOUGH_COUNTS; ++i) A.counts[i] = 0;
    }
}

// Track records and hit lists (vane order from each track's lower end).
__global__ __launch_bounds__(64) void k_tw_emit(TwArgs A) {
    if (A.err[0] != 0) return;
    const int b = blockIdx.x;
    const int64_t base = A.offsets[b];
    const int64_t s0 = slot0(A, b, base);
    const int32_t ntr = A.ntr[b];
    int64_t hoff = A.tl_hbase[b];
    const int64_t tbase = A.tl_tbase[b];
    for (int32_t k0 = 0; k0 < ntr; k0 += 64) {
        const int32_t kid = k0 + lane();
        const int64_t nhk = kid < ntr ? A.nh[s0 + kid] : 0;
        // inclusive prefix over the wave
        int64_t incl = nhk;
        for (int o = 1; o < 64; o <<= 1) {
            const int64_t u = __shfl_up(incl, o, 64);
            if (lane() >= o) incl += u;
        }
        if (kid < ntr) {
            const int64_t k = s0 + kid;
            const int64_t off = hoff + incl - nhk;
            hough_track T;
            T.timeline = b;
            T.track = kid;
            T.window = A.win[k];
            T.n_hits = A.nh[k];
            T.hit_offset = off;
            T.vane_first = A.vane[A.end_down[k]];
            T.vane_last = A.vane[A.end_up[k]];
            T.theta_bin = A.tb[k];
            T.rho_bin = A.rb[k];
            T.last_window = A.last_win[k];
            T.carried = A.carried[k];
            A.tracks[tbase + kid] = T;
            int32_t h = A.end_down[k];
            for (int64_t i = 0; h >= 0 && i < T.n_hits; ++i) {
                A.hit_index[off + i] = (int32_t)(h - base);
                h = A.up[h];
            }
        }
        hoff += __shfl(incl, 63, 64);
    }
}

size_t align256(size_t x) { return (x + 255) & ~(size_t)255; }

}  // namespace
}  // namespace hough

using namespace hough;
using namespace hough::rt;

extern "C" {

hough_status hough_tw_config_default(hough_tw_config *tw) {
    if (!tw) return HOUGH_ERR_INVALID_ARG;
    *tw = hough_tw_config{};
    tw->window_ns = 10.0f;
    tw->step_ns = 5.0f;
    tw->gate_r_mm = 10.0f;
    tw->gate_z_mm = 4.0f;
    tw->gate_t_ns = 2.0f;
    tw->max_track_hits = 64;
    return HOUGH_OK;
}

hough_status hough_tw_find(hough_ctx *ctx, void *stream, const hough_tw_config *tw, int32_t n_timelines,
                           int64_t n_hits_total, const int64_t *offsets, const float *r, const float *z,
                           const int16_t *vane, const float *t, int32_t n_windows, hough_track *tracks,
                           int64_t track_capacity, int32_t *hit_index, int64_t hit_capacity, int64_t *counts) {
    Ctx *c = as_ctx(ctx);
    if (!c) return fail(nullptr, HOUGH_ERR_INVALID_ARG, "bad context");
    if (!tw || !counts || n_timelines < 0 || n_hits_total < 0 || n_windows < 0 || !offsets ||
        (n_hits_total > 0 && (!r || !z || !vane || !t)))
        return fail(c, HOUGH_ERR_INVALID_ARG, "bad hough_tw_find arguments");
    if (!(std::isfinite(tw->window_ns) && std::isfinite(tw->step_ns) && tw->step_ns > 0.0f &&
          tw->window_ns >= tw->step_ns) ||
        !(tw->gate_r_mm >= 0.0f && tw->gate_z_mm >= 0.0f && tw->gate_t_ns >= 0.0f) || tw->max_track_hits < 3 ||
        tw->max_track_hits > 1024 || tw->reserved[0] != 0 || tw->reserved[1] != 0)
        return fail(c, HOUGH_ERR_INVALID_ARG, "bad time-window configuration");
    if (c->cfg.n_vanes < 3 || c->cfg.n_vanes > kTwVaneMax)
        return fail(c, HOUGH_ERR_INVALID_ARG, "the time-sliced finder needs 3..1024 vanes");
    if (track_capacity < n_hits_total / 3 || hit_capacity < n_hits_total || (n_hits_total > 0 && (!tracks || !hit_index)))
        return fail(c, HOUGH_ERR_CAPACITY, "outputs need n_hits / 3 tracks and n_hits hit indices");
    if (n_hits_total > INT32_MAX) return fail(c, HOUGH_ERR_CAPACITY, "at most 2^31 - 1 hits per call");
    if (hipSetDevice(c->device) != hipSuccess) return fail(c, HOUGH_ERR_DEVICE, "hipSetDevice failed");
    hipStream_t s = static_cast<hipStream_t>(stream);

    const int64_t N = n_hits_total, B = n_timelines;
    const int64_t nslots = N / 3 + B + 1;
    size_t off = 0;
    auto take = [&](size_t bytes) { size_t o = off; off = align256(off + bytes); return o; };
    const size_t o_used = take(4 * N), o_up = take(4 * N), o_down = take(4 * N), o_widx = take(4 * N);
    const size_t o_wz = take(4 * N), o_wv = take(2 * N);
    const size_t o_ntr = take(4 * B);
    const size_t o_tlc = take(8 * B), o_tlk = take(8 * B), o_tlh = take(8 * B), o_tlt = take(8 * B),
                 o_tlhb = take(8 * B);
    const size_t o_slots = take(40 * (size_t)nslots);
    const size_t o_err = take(8 * 4), o_find = take(2 * sizeof(FindArgs)), o_pick = take(4);
    if (off > c->tw_bytes) {
        if (c->tw_base) {
            if (hipStreamSynchronize(s) != hipSuccess) return fail(c, HOUGH_ERR_DEVICE, "hipStreamSynchronize failed");
            (void)hipFree(c->tw_base);
            c->tw_base = nullptr;
            c->tw_bytes = 0;
        }
        if (hipMalloc(&c->tw_base, off) != hipSuccess) {
            c->tw_base = nullptr;
            return fail(c, HOUGH_ERR_OOM, "time-window workspace allocation failed");
        }
        c->tw_bytes = off;
    }
    hough_status st = ensure_workspace(*c, c->ws, std::max<int64_t>(N, 1), std::max<int64_t>(B, 1), s);
    if (st) return fail(c, st, "workspace allocation failed");

    char *base = static_cast<char *>(c->tw_base);
    TwArgs A{};
    A.n_tl = (int32_t)B;
    A.n_total = N;
    A.offsets = offsets;
    A.r = r;
    A.z = z;
    A.t = t;
    A.vane = vane;
    A.n_vanes = c->cfg.n_vanes;
    A.window_ns = tw->window_ns;
    A.step_ns = tw->step_ns;
    A.gate_r = tw->gate_r_mm;
    A.gate_z = tw->gate_z_mm;
    A.gate_t = tw->gate_t_ns;
    A.max_track_hits = tw->max_track_hits;
    A.used = reinterpret_cast<int32_t *>(base + o_used);
    A.up = reinterpret_cast<int32_t *>(base + o_up);
    A.down = reinterpret_cast<int32_t *>(base + o_down);
    A.widx = reinterpret_cast<int32_t *>(base + o_widx);
    A.wz = reinterpret_cast<float *>(base + o_wz);
    A.wv = reinterpret_cast<int16_t *>(base + o_wv);
    A.ntr = reinterpret_cast<int32_t *>(base + o_ntr);
    A.tl_cand = reinterpret_cast<int64_t *>(base + o_tlc);
    A.tl_carry = reinterpret_cast<int64_t *>(base + o_tlk);
    A.tl_hits = reinterpret_cast<int64_t *>(base + o_tlh);
    A.tl_tbase = reinterpret_cast<int64_t *>(base + o_tlt);
    A.tl_hbase = reinterpret_cast<int64_t *>(base + o_tlhb);
    int32_t *sl = reinterpret_cast<int32_t *>(base + o_slots);
    A.end_up = sl;
    A.end_down = sl + nslots;
    A.nh = sl + 2 * nslots;
    A.win = sl + 3 * nslots;
    A.last_win = sl + 4 * nslots;
    A.carried = sl + 5 * nslots;
    A.flagged = sl + 6 * nslots;
    A.tb = sl + 7 * nslots;
    A.rb = sl + 8 * nslots;
    A.tmax = reinterpret_cast<float *>(sl + 9 * nslots);
    A.err = reinterpret_cast<long long *>(base + o_err);
    A.find = reinterpret_cast<FindArgs *>(base + o_find);
    // hits of a window that fit the LDS beside the vane tables (16-bit positions)
    auto lds_hits = [&](int lds) { return std::max(0, std::min(4096, (lds - tw_vane_bytes(A.n_vanes)) / kTwHitBytes)) & ~63; };
    A.lds_hits = lds_hits(c->tw_lds);
    A.tracks = tracks;
    A.hit_index = hit_index;
    A.counts = counts;
    A.n_windows = n_windows;
    // the windows' events: timeline b's hits from offsets[b] on
    auto window_args = [&](const Shape &f) {
        FindArgs F = find_args(*c, f, c->ws);
        F.n_events = (int32_t)B;
        F.n_total = N;
        F.total_is_bound = 1;
        F.z = A.wz;
        F.vane = A.wv;
        F.g_hs = nullptr;
        return F;
    };
    // long rows: the shape of more waves for calls with a window that outgrows
    // the own shape's list (the device finds out)
    const bool wide = c->wide.max_resident > 0 && N > list_hits(*c);
    if (wide) {
        A.pick = reinterpret_cast<int32_t *>(base + o_pick);
        A.pick_hits = (int32_t)list_hits(*c);
    }

    auto launched = [&](const char *what) -> hough_status {
        const hipError_t e = hipGetLastError();
        if (e != hipSuccess) return fail(c, HOUGH_ERR_DEVICE, std::string(what) + " launch failed: " + hipGetErrorString(e));
        return HOUGH_OK;
    };
    {
        const int64_t m = std::max<int64_t>(std::max<int64_t>(N, B), 1);
        const int grid = (int)std::min<int64_t>((m + 255) / 256, 2048);
        hipLaunchKernelGGL(k_tw_init, dim3(grid), dim3(256), 0, s, A, window_args(*c), window_args(wide ? c->wide : *c));
        if ((st = launched("k_tw_init"))) return st;
    }
    if (B > 0) {
        hipLaunchKernelGGL(k_tw_validate, dim3((unsigned)B), dim3(256), 0, s, A);
        if ((st = launched("k_tw_validate"))) return st;
        hipError_t e = c->cfg.peak_mode == 2 ? launch_tw_run_cf(A, c->wg_threads, c->tw_lds, s)
                                             : launch_tw_run(A, c->wg_threads, c->cfg.peak_mode == 0, c->tw_lds, s);
        if (e == hipSuccess && wide) {
            TwArgs W = A;
            W.mine = 1;
            W.find = A.find + 1;
            W.lds_hits = lds_hits(c->wide.lds_bytes);
            e = launch_tw_run(W, c->wide.wg_threads, c->cfg.peak_mode == 0, c->wide.lds_bytes, s);
        }
        if (e != hipSuccess)
            return fail(c, HOUGH_ERR_DEVICE, std::string("k_tw_run launch failed: ") + hipGetErrorString(e));
    }
    hipLaunchKernelGGL(k_tw_out_scan, dim3(1), dim3(1024), 0, s, A);
    if ((st = launched("k_tw_out_scan"))) return st;
    if (B > 0) {
        hipLaunchKernelGGL(k_tw_emit, dim3((unsigned)B), dim3(64), 0, s, A);
        if ((st = launched("k_tw_emit"))) return st;
    }
    c->last_error.clear();
    return HOUGH_OK;
}

}  // extern "C"
