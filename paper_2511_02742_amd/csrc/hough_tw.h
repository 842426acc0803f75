// Device side of the time-sliced finder: the window loop of one timeline by one
// workgroup, generic in the event finder it calls (hough_kernels.hip and
// hough_cf.hip instantiate it with theirs).
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "hough_internal.h"
#include "hough_tf.h"

namespace hough {

struct TwArgs {
    int32_t n_tl;
    int64_t n_total;
    const int64_t *offsets;
    const float *r, *z, *t;
    const int16_t *vane;
    int32_t n_vanes;
    float window_ns, step_ns, gate_r, gate_z, gate_t;
    int32_t max_track_hits;
    int32_t n_windows;
    int32_t lds_hits;                // largest window staged in LDS
    // per hit (global index)
    int32_t *used;                   // track id (timeline-local) or -1
    int32_t *up, *down;              // neighbour on the next / previous vane in its track, or -1
    // per timeline
    int32_t *ntr;                    // tracks
    int64_t *tl_cand, *tl_carry, *tl_hits, *tl_tbase, *tl_hbase;
    // per track slot: timeline b owns slots [offsets[b] / 3 + b, ...)
    int32_t *end_up, *end_down, *nh, *win, *last_win, *carried, *tb, *rb;
    int32_t *flagged;                // track ids flagged for the next window, ascending (the timeline's slots)
    float *tmax;
    // the window's event: timeline b's at [offsets[b], + its unused hits)
    float *wz;
    int16_t *wv;
    int32_t *widx;                   // global hit index of each window-event hit
    long long *err;                  // [status (min), first bad global hit (min)]
    FindArgs *find;                  // the event finder's arguments, in device memory
    // calls of two shapes: 1 at *pick when a window holds more than pick_hits hits, and
    // then the launch whose `mine` is 1 runs, else the other (NULL: this one does)
    int32_t *pick;
    int32_t mine, pick_hits;
    // outputs
    hough_track *tracks;
    int32_t *hit_index;
    int64_t *counts;
};

// The window loop of every timeline (one workgroup each): hough_kernels.hip
// with the histogram finder, hough_cf.hip with the coarse-to-fine one.
hipError_t launch_tw_run(const TwArgs &t, int wg_threads, bool argmax, int lds_bytes, hipStream_t s);
hipError_t set_tw_lds_limit(int wg_threads, int lds_bytes);
hipError_t launch_tw_run_cf(const TwArgs &t, int wg_threads, int lds_bytes, hipStream_t s);
hipError_t set_tw_cf_lds_limit(int wg_threads, int lds_bytes);

// LDS of a staged window: two ints per vane, and per hit its coordinates and
// four 16-bit indices.
constexpr int kTwVaneMax = 1024;
constexpr int kTwHitBytes = 20;
inline int tw_vane_bytes(int n_vanes) { return (4 * (2 * n_vanes + 1) + 15) & ~15; }

namespace tw {

__device__ __forceinline__ int tid() {
    int t = (int)threadIdx.x;
    asm volatile("" : "+v"(t));   // not hoisted and held across the finder
    return t;
}
__device__ __forceinline__ int lane() { return tid() & 63; }

// *A as constant memory: an earlier kernel wrote it, nothing does now.
__device__ __forceinline__ const FindArgs &const_args(const FindArgs *A) {
    const uint64_t p = (uint64_t)(uintptr_t)A;
    const uint32_t lo = (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)p);
    const uint32_t hi = (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)(p >> 32));
    typedef const __attribute__((address_space(4))) FindArgs *ConstArgs;
    return *(const FindArgs *)(ConstArgs)(((uint64_t)hi << 32) | lo);
}
__device__ __forceinline__ int wave() { return __builtin_amdgcn_readfirstlane(tid() >> 6); }
__device__ __forceinline__ int rl(int v, int l) { return __builtin_amdgcn_readlane(v, l); }
__device__ __forceinline__ float rl(float v, int l) { return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), l)); }
__device__ __forceinline__ void wave_order() { __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront"); }

__device__ __forceinline__ uint32_t wave_min(uint32_t v) {
#define HOUGH_TW_MIN(ctrl, rows) \
    v = min(v, (uint32_t)__builtin_amdgcn_update_dpp((int)0xffffffffu, (int)v, ctrl, rows, 0xf, false))
    HOUGH_TW_MIN(0x111, 0xf);   // row_shr:1, 2, 4, 8
    HOUGH_TW_MIN(0x112, 0xf);
    HOUGH_TW_MIN(0x114, 0xf);
    HOUGH_TW_MIN(0x118, 0xf);
    HOUGH_TW_MIN(0x142, 0xa);   // row_bcast:15, 31
    HOUGH_TW_MIN(0x143, 0xc);
#undef HOUGH_TW_MIN
    return (uint32_t)__builtin_amdgcn_readlane((int)v, 63);
}

// What the workgroup keeps of its timeline between windows.
struct Shared {
    int w;           // window being processed
    int wa, we;      // its hits
    int busy;        // 0: no window is left
    int ntr, nflag;  // tracks; of them flagged in the previous window
    int hits;        // hits in tracks
    int ncarry;      // (track, window) continuations
    int ncand;       // candidates over the windows
    int wtot[16];
};

// Hits are 32-bit positions below 2^31 - 1. A lane's position or the next round's
// may pass the end by up to a workgroup's width, so scans count unsigned.

// A window's hits in LDS, by vane (in hit order inside a vane is not kept: the
// choice of a hit does not depend on the order). Position p holds hit q = bq[p]
// of the window; r is NaN once the hit is in a track (no gate takes it).
struct Window {
    int wa, m;       // first hit and number of hits
    int *vst;        // [n_vanes + 1] first position of each vane
    int *first;      // [n_vanes] the seed's table
    float *r, *z, *t;
    uint16_t *bq, *bv, *qpos;   // hit and vane of a position; position of a hit
    uint16_t *fq;    // the event finder's hit lists as hits of the window
};

__device__ __forceinline__ Window window_lds(const TwArgs &A, uint32_t *lds) {
    Window W;
    W.vst = reinterpret_cast<int *>(lds);
    W.first = W.vst + A.n_vanes + 1;
    W.r = reinterpret_cast<float *>(lds + ((2 * A.n_vanes + 1 + 3) & ~3));
    W.z = W.r + A.lds_hits;
    W.t = W.z + A.lds_hits;
    W.bq = reinterpret_cast<uint16_t *>(W.t + A.lds_hits);
    W.bv = W.bq + A.lds_hits;
    W.qpos = W.bv + A.lds_hits;
    W.fq = W.qpos + A.lds_hits;
    return W;
}

// The window's hits into LDS by the workgroup: a counting sort on the vane.
template <int NT>
__device__ __forceinline__ void stage(const TwArgs &A, const Window &W) {
    const int i0 = tid();
    float r0 = 0.0f, z0 = 0.0f, t0 = 0.0f;
    int v0 = 0;
    bool in0 = i0 < W.m;
    if (in0) {
        const int h = W.wa + i0;
        v0 = A.vane[h];
        r0 = A.used[h] < 0 ? A.r[h] : __int_as_float(0x7fc00000);
        z0 = A.z[h];
        t0 = A.t[h];
    }
    for (int v = i0; v <= A.n_vanes; v += NT) W.vst[v] = 0;
    __syncthreads();
    for (int i = i0; i < W.m; i += NT)
        W.qpos[i] = (uint16_t)atomicAdd(&W.vst[i == i0 ? v0 : (int)A.vane[W.wa + i]], 1);
    __syncthreads();
    if (wave() == 0) {
        int carry = 0;
        for (int vb = 0; vb <= A.n_vanes; vb += 64) {
            const int v = vb + lane();
            const int c = v < A.n_vanes ? W.vst[v] : 0;
            int incl = c;
            for (int o = 1; o < 64; o <<= 1) {
                const int u = __shfl_up(incl, o, 64);
                if (lane() >= o) incl += u;
            }
            if (v <= A.n_vanes) W.vst[v] = carry + incl - c;
            carry += rl(incl, 63);
        }
    }
    __syncthreads();
    for (int i = i0; i < W.m; i += NT) {
        const int h = W.wa + i;
        if (i != i0) {
            v0 = A.vane[h];
            r0 = A.used[h] < 0 ? A.r[h] : __int_as_float(0x7fc00000);
            z0 = A.z[h];
            t0 = A.t[h];
        }
        const int p = W.vst[v0] + W.qpos[i];
        W.r[p] = r0;
        W.z[p] = z0;
        W.t[p] = t0;
        W.bq[p] = (uint16_t)i;
        W.bv[p] = (uint16_t)v0;
        W.qpos[i] = (uint16_t)p;
    }
    __syncthreads();
}

// One end of a track: its end hit e and, from the third-last hit to it, the
// coordinates that the extrapolation uses.
struct End {
    int e, v;
    float t, r1, r2, r3, z1, z2, z3;
};

// Extends track kid at one end (D = +1: next vane, -1: previous vane) through
// the window's unused hits; one wave. Among a vane's gated hits the smallest
// (|dr| + |dz|, hit) joins. Returns the hits added. STAGED: the window is in
// LDS, else its hits are scanned in device memory.
template <int D, bool STAGED>
__device__ int extend(const TwArgs &A, const Window &W, int kid, End &E, int &n, float &tmax) {
    int added = 0;
    while (n < A.max_track_hits) {
        int target = E.v + D;
        target = target < 0 ? A.n_vanes - 1 : target == A.n_vanes ? 0 : target;
        const float r_hat = (E.r1 - 3.0f * E.r2) + 3.0f * E.r3;
        const float z_hat = (E.z1 - 3.0f * E.z2) + 3.0f * E.z3;
        // this lane's best: score bits (>= 0, so they order like the values), hit, position
        uint32_t score = 0xffffffffu, q = 0xffffffffu;
        int pos = 0;
        float rb = 0.0f, zb = 0.0f, tb = 0.0f;
        const uint32_t s = STAGED ? W.vst[target] : 0, e = STAGED ? W.vst[target + 1] : W.m;
        for (uint32_t i = s + lane(); i < e; i += 64) {
            if (!STAGED && (A.used[W.wa + i] >= 0 || A.vane[W.wa + i] != target)) continue;
            const float r = STAGED ? W.r[i] : A.r[W.wa + i];
            const float z = STAGED ? W.z[i] : A.z[W.wa + i];
            const float t = STAGED ? W.t[i] : A.t[W.wa + i];
            const float dr = fabsf(r - r_hat), dz = fabsf(z - z_hat), dt = fabsf(t - E.t);
            if (dr <= A.gate_r && dz <= A.gate_z && dt <= A.gate_t) {
                const uint32_t sc = __float_as_uint(dr + dz);
                const uint32_t qi = STAGED ? (uint32_t)W.bq[i] : i;
                if (sc < score || (sc == score && qi < q)) {
                    score = sc;
                    q = qi;
                    pos = (int)i;
                    rb = r;
                    zb = z;
                    tb = t;
                }
            }
        }
        unsigned long long win = __ballot(q != 0xffffffffu);
        if (win == 0ull) break;
        if ((win & (win - 1)) != 0ull) {
            const uint32_t top = wave_min(score);
            win = __ballot(q != 0xffffffffu && score == top);
            if ((win & (win - 1)) != 0ull) {
                const uint32_t qt = wave_min(score == top ? q : 0xffffffffu);
                win = __ballot(score == top && q == qt);
            }
        }
        const int l = __builtin_ctzll(win);
        const int hb = W.wa + rl((int)q, l);
        if (STAGED) {
            if (lane() == l) W.r[pos] = __int_as_float(0x7fc00000);
            wave_order();
        }
        E.r1 = E.r2;
        E.r2 = E.r3;
        E.r3 = rl(rb, l);
        E.z1 = E.z2;
        E.z2 = E.z3;
        E.z3 = rl(zb, l);
        E.t = rl(tb, l);
        tmax = E.t > tmax ? E.t : tmax;
        if (lane() == 0) {
            A.used[hb] = kid;
            if (D > 0) {
                A.up[E.e] = hb;
                A.down[hb] = E.e;
            } else {
                A.down[E.e] = hb;
                A.up[hb] = E.e;
            }
        }
        // the next scan reads `used` back
        if (!STAGED) __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "workgroup");
        E.e = hb;
        E.v = target;
        ++n;
        ++added;
    }
    return added;
}

// Continues the tracks flagged in the previous window into window w, in track
// order (one wave). Their ends are read 64 tracks at a time (a track's ends
// depend on no other track); the list of those still flagged replaces the list
// in place (it never outruns the reading).
template <bool STAGED>
__device__ void carry(const TwArgs &A, const Window &W, Shared &T, int w, float next_lo, int64_t s0) {
    const int nf = T.nflag;
    int keep = 0, hits = 0, carried = 0;
    for (int k0 = 0; k0 < nf; k0 += 64) {
        const int cnt = min(64, nf - k0);
        const int i = k0 + min(lane(), cnt - 1);
        const int kid_l = A.flagged[s0 + i];
        const int64_t k_l = s0 + kid_l;
        const int nh_l = A.nh[k_l], car_l = A.carried[k_l];
        const float tmax_l = A.tmax[k_l];
        const int eu = A.end_up[k_l], ed = A.end_down[k_l];
        const int eu2 = A.down[eu], ed2 = A.up[ed];
        const int eu1 = A.down[eu2], ed1 = A.up[ed2];
        const End U{eu, (int)A.vane[eu], A.t[eu], A.r[eu1], A.r[eu2], A.r[eu], A.z[eu1], A.z[eu2], A.z[eu]};
        const End L{ed, (int)A.vane[ed], A.t[ed], A.r[ed1], A.r[ed2], A.r[ed], A.z[ed1], A.z[ed2], A.z[ed]};
        for (int j = 0; j < cnt; ++j) {
            const int kid = rl(kid_l, j);
            const int64_t k = s0 + kid;
            int n = rl(nh_l, j);
            float tmax = rl(tmax_l, j);
            End E{rl(U.e, j), rl(U.v, j), rl(U.t, j), rl(U.r1, j), rl(U.r2, j), rl(U.r3, j), rl(U.z1, j), rl(U.z2, j), rl(U.z3, j)};
            const int up = extend<1, STAGED>(A, W, kid, E, n, tmax);
            if (up > 0 && lane() == 0) A.end_up[k] = E.e;
            E = End{rl(L.e, j), rl(L.v, j), rl(L.t, j), rl(L.r1, j), rl(L.r2, j), rl(L.r3, j), rl(L.z1, j), rl(L.z2, j), rl(L.z3, j)};
            const int down = extend<-1, STAGED>(A, W, kid, E, n, tmax);
            if (down > 0 && lane() == 0) A.end_down[k] = E.e;
            if (up + down == 0) continue;
            hits += up + down;
            ++carried;
            const int car = rl(car_l, j) + 1;
            if (lane() == 0) {
                A.nh[k] = n;
                A.tmax[k] = tmax;
                A.carried[k] = car;
                A.last_win[k] = w;
            }
            if (tmax >= next_lo) {
                if (lane() == 0) A.flagged[s0 + keep] = kid;
                ++keep;
            }
        }
    }
    if (lane() == 0) {
        T.nflag = keep;
        T.hits += hits;
        T.ncarry += carried;
    }
}

// Seeds and extends a track from each of the window event's nc candidates, in
// emission order (one wave): per vane the candidate's unused hit of lowest
// index, then the first three consecutive vanes whose hits are near in time.
template <bool STAGED>
__device__ void seed(const TwArgs &A, const FindArgs &F, const Window &W, Shared &T, int w, float next_lo, int64_t s0,
                     int64_t base, int nc) {
    const int nv = A.n_vanes;
    const hough_candidate *const cb = F.cand_ws + base / (int64_t)F.min_votes;
    int ntr = T.ntr, nflag = T.nflag, hits = 0;
    for (int c0 = 0; c0 < nc; c0 += 64) {
        const int cnt = min(64, nc - c0);
        const hough_candidate *const mine = cb + c0 + min(lane(), cnt - 1);
        const int n_l = (int)mine->n_hits, off_l = (int)mine->hit_offset;
        const int tb_l = mine->theta_bin, rb_l = mine->rho_bin;
        for (int j = 0; j < cnt; ++j) {
            const int n_hits = rl(n_l, j), off = rl(off_l, j);
            for (int v = lane(); v < nv; v += 64) W.first[v] = 0x7fffffff;
            wave_order();
            for (int i = off + lane(); i < off + n_hits; i += 64) {
                if (STAGED) {
                    const int q = W.fq[i], p = W.qpos[q];
                    if (W.r[p] == W.r[p]) atomicMin(&W.first[W.bv[p]], q);
                } else {
                    const int h = A.widx[base + F.hits_ws[base + i]];
                    if (A.used[h] < 0) atomicMin(&W.first[A.vane[h]], h - W.wa);
                }
            }
            wave_order();
            auto time_of = [&](int q) { return STAGED ? W.t[W.qpos[q]] : A.t[W.wa + q]; };
            int v0 = -1;
            for (int vb = 0; vb < nv && v0 < 0; vb += 64) {
                const int v = vb + lane();
                bool ok = false;
                if (v < nv) {
                    const int v1 = v + 1 == nv ? 0 : v + 1, v2 = v1 + 1 == nv ? 0 : v1 + 1;
                    const int fa = W.first[v], fb = W.first[v1], fc = W.first[v2];
                    if (fa != 0x7fffffff && fb != 0x7fffffff && fc != 0x7fffffff) {
                        const float tb = time_of(fb);
                        ok = fabsf(tb - time_of(fa)) <= A.gate_t && fabsf(time_of(fc) - tb) <= A.gate_t;
                    }
                }
                const unsigned long long m = __ballot(ok);
                if (m != 0ull) v0 = vb + __builtin_ctzll(m);
            }
            if (v0 < 0) continue;
            const int v1 = v0 + 1 == nv ? 0 : v0 + 1, v2 = v1 + 1 == nv ? 0 : v1 + 1;
            const int qa = __builtin_amdgcn_readfirstlane(W.first[v0]), qb = __builtin_amdgcn_readfirstlane(W.first[v1]),
                      qc = __builtin_amdgcn_readfirstlane(W.first[v2]);
            const int ha = W.wa + qa, hb = W.wa + qb, hc = W.wa + qc;
            float ra, rb, rc, za, zb, zc, ta, tb, tc;
            if (STAGED) {
                const int pa = W.qpos[qa], pb = W.qpos[qb], pc = W.qpos[qc];
                ra = W.r[pa], rb = W.r[pb], rc = W.r[pc];
                za = W.z[pa], zb = W.z[pb], zc = W.z[pc];
                ta = W.t[pa], tb = W.t[pb], tc = W.t[pc];
                wave_order();
                if (lane() < 3) W.r[lane() == 0 ? pa : lane() == 1 ? pb : pc] = __int_as_float(0x7fc00000);
                wave_order();
            } else {
                ra = A.r[ha], rb = A.r[hb], rc = A.r[hc];
                za = A.z[ha], zb = A.z[hb], zc = A.z[hc];
                ta = A.t[ha], tb = A.t[hb], tc = A.t[hc];
            }
            const int kid = ntr++;
            const int64_t k = s0 + kid;
            float tmax = ta;
            tmax = tb > tmax ? tb : tmax;
            tmax = tc > tmax ? tc : tmax;
            if (lane() == 0) {
                A.up[ha] = hb;
                A.down[hb] = ha;
                A.up[hb] = hc;
                A.down[hc] = hb;
                A.used[ha] = kid;
                A.used[hb] = kid;
                A.used[hc] = kid;
            }
            if (!STAGED) __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "workgroup");
            int n = 3;
            End E{hc, v2, tc, ra, rb, rc, za, zb, zc};
            extend<1, STAGED>(A, W, kid, E, n, tmax);
            const int top = E.e;
            E = End{ha, v0, ta, rc, rb, ra, zc, zb, za};
            extend<-1, STAGED>(A, W, kid, E, n, tmax);
            hits += n;
            const bool flag = tmax >= next_lo;
            const int theta_bin = rl(tb_l, j), rho_bin = rl(rb_l, j);
            if (lane() == 0) {
                A.end_down[k] = E.e;
                A.end_up[k] = top;
                A.nh[k] = n;
                A.win[k] = w;
                A.last_win[k] = w;
                A.carried[k] = 0;
                A.tb[k] = theta_bin;
                A.rb[k] = rho_bin;
                A.tmax[k] = tmax;
                if (flag) A.flagged[s0 + nflag] = kid;
            }
            nflag += flag ? 1 : 0;
        }
    }
    if (lane() == 0) {
        T.ntr = ntr;
        T.nflag = nflag;
        T.hits += hits;
    }
}

// First index in [from, end) whose time is >= x, scanning forward 64 hits at a
// time (one wave).
__device__ __forceinline__ int advance_lb(const float *t, int from, int end, float x) {
    for (;;) {
        const uint32_t i = (uint32_t)from + lane();
        const int c = __popcll(__ballot(i < (uint32_t)end && t[i] < x));
        from += c;
        if (c < 64) return from;
    }
}

// From window T.w on, the next window with work: flagged tracks and a hit that
// could continue them, or at least T unused hits (one wave). The times of the 64
// hits from the last window's first one on are held one per lane, so a window
// with neither costs two ballots, and a run of empty ones a division.
__device__ __forceinline__ void next_window(const TwArgs &A, uint32_t min_votes, Shared &T, int end) {
    int w = T.w, cb = T.wa, we = 0, wa = 0, nflag = T.nflag, busy = 0;
    float tl = 0.0f;
    bool unused = false, load = true;
    while (w < A.n_windows) {
        if (load) {
            const uint32_t i = (uint32_t)cb + lane();
            tl = i < (uint32_t)end ? A.t[i] : __int_as_float(0x7f800000);
            unused = i < (uint32_t)end && A.used[i] < 0;
            load = false;
        }
        const float lo = (float)w * A.step_ns, hi = lo + A.window_ns;
        const unsigned long long mlo = __ballot(tl < lo), mhi = __ballot(tl < hi);
        const int a = __popcll(mlo), z = __popcll(mhi);
        if (a == 64 || (z == 64 && a > 0)) {
            cb += a;
            load = true;
            continue;
        }
        wa = cb + a;
        we = cb + z;
        if (z == 64) {
            we = advance_lb(A.t, we, end, hi);
            busy = 1;
            break;
        }
        if (a == z) {
            // no hit: nothing stays flagged, and the windows that end before
            // the next hit are as empty (lo and hi grow with w)
            nflag = 0;
            if (wa >= end) {
                w = A.n_windows;
                break;
            }
            const float tn = rl(tl, a);
            const float est = fminf((tn - A.window_ns) / A.step_ns, 2.0e9f);
            int to = est > 0.0f ? (int)est - 2 - ((int)est >> 20) : 0;
            while (to > w + 1 && (float)(to - 1) * A.step_ns + A.window_ns > tn) --to;
            w = max(w + 1, min(to, A.n_windows));
            continue;
        }
        if (nflag > 0 || (uint32_t)__popcll(__ballot(unused) & mhi & ~mlo) >= min_votes) {
            busy = 1;
            break;
        }
        ++w;
    }
    if (lane() == 0) {
        T.w = w;
        T.wa = busy ? wa : cb;
        T.we = we;
        T.nflag = nflag;
        T.busy = busy;
    }
}

// The window's unused hits, in hit order, as the event at `base`; their number.
template <int NT>
__device__ __forceinline__ int collect(const TwArgs &A, Shared &T, int wa, int we, int64_t base) {
    int n = 0;
    for (uint32_t h0 = wa; h0 < (uint32_t)we; h0 += NT) {
        const uint32_t h = h0 + tid();
        const bool take = h < (uint32_t)we && A.used[h] < 0;
        const unsigned long long m = __ballot(take);
        if (lane() == 0) T.wtot[wave()] = __popcll(m);
        __syncthreads();
        int before = 0, all = 0;
        for (int u = 0; u < NT / 64; ++u) {
            const int x = T.wtot[u];
            before += u < wave() ? x : 0;
            all += x;
        }
        if (take) {
            const int64_t o = base + n + before + __popcll(m & ((1ull << lane()) - 1ull));
            A.wz[o] = A.z[h];
            A.wv[o] = A.vane[h];
            A.widx[o] = (int)h;
        }
        n += all;
        __syncthreads();
    }
    return n;
}

// All windows of timeline b by the workgroup. `find(b, base, n)` runs the event
// finder on the n hits at wz, wv + base as event b (results in F's workspace).
// `lds` is the finder's dynamic LDS, used between its calls.
template <int NT, class Find>
__device__ __forceinline__ void run(const TwArgs &A, const FindArgs &F, uint32_t *lds, Shared &T, const Find &find) {
    // one thread's look at the status: another workgroup may set it meanwhile
    if (tid() == 0) T.busy = A.err[0] == 0 && (A.pick == nullptr || *A.pick == A.mine) ? 1 : 0;
    __syncthreads();
    if (!T.busy) return;
    const int b = blockIdx.x;
    const int64_t base = A.offsets[b];
    const int end = (int)A.offsets[b + 1];
    const int64_t s0 = base / 3 + b;
    __syncthreads();
    if (tid() == 0) {
        T.w = 0;
        T.wa = (int)base;
        T.ntr = T.nflag = T.hits = T.ncarry = T.ncand = 0;
    }
    __syncthreads();
    for (;;) {
        if (wave() == 0) next_window(A, F.min_votes, T, end);
        __syncthreads();
        if (!T.busy) break;
        const int w = __builtin_amdgcn_readfirstlane(T.w);
        const int nflag = __builtin_amdgcn_readfirstlane(T.nflag);
        Window W = window_lds(A, lds);
        W.wa = __builtin_amdgcn_readfirstlane(T.wa);
        const int we = __builtin_amdgcn_readfirstlane(T.we);
        W.m = we - W.wa;
        const bool staged = W.m <= A.lds_hits;
        const float next_lo = (float)(w + 1) * A.step_ns;
        __syncthreads();   // T is read by every wave before wave 0 changes it
        if (nflag > 0) {
            if (staged) stage<NT>(A, W);
            if (wave() == 0) {
                if (staged)
                    carry<true>(A, W, T, w, next_lo, s0);
                else
                    carry<false>(A, W, T, w, next_lo, s0);
            }
            __syncthreads();
        }
        const int n = collect<NT>(A, T, W.wa, we, base);
        if (n > HOUGH_MAX_EVENT_HITS) {
            if (tid() == 0) atomicMin(&A.err[0], (long long)HOUGH_ERR_CAPACITY);
            return;
        }
        if ((uint32_t)n >= F.min_votes) {
            find(b, base, (int64_t)n);
            __syncthreads();
            const int nc = __builtin_amdgcn_readfirstlane(F.ev_ncand[b]);
            if (nc > 0) {
                if (staged) {
                    const int nh = F.ev_nhits[b];
                    stage<NT>(A, W);
                    for (int i = tid(); i < nh; i += NT)
                        W.fq[i] = (uint16_t)(A.widx[base + F.hits_ws[base + i]] - W.wa);
                    __syncthreads();
                }
                if (wave() == 0) {
                    if (staged)
                        seed<true>(A, F, W, T, w, next_lo, s0, base, nc);
                    else
                        seed<false>(A, F, W, T, w, next_lo, s0, base, nc);
                    if (lane() == 0) T.ncand += nc;
                }
            }
        }
        __syncthreads();
        if (tid() == 0) T.w = w + 1;
        __syncthreads();
    }
    if (tid() == 0) {
        A.ntr[b] = T.ntr;
        A.tl_hits[b] = T.hits;
        A.tl_cand[b] = T.ncand;
        A.tl_carry[b] = T.ncarry;
    }
}

}  // namespace tw
}  // namespace hough
