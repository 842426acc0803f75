// Helix refit of track candidates: initial parameters, the chi^2 of the hit
// residuals, its adjoint (gradient) and damped Gauss-Newton steps.
//
// One wave takes a few consecutive candidates:
// what a hit needs (its model, its float64 angles) runs one lane per hit over
// the candidates' hits laid end to end, what a candidate needs (the sums over
// its hits, the 3 x 3 and 5 x 5 systems) one lane per sum, candidate or matrix
// column. The sums run over a candidate's hits in their order, one after the
// other: the results do not depend on how candidates are dealt to waves. The
// initial fit runs in float64 (it takes discrete decisions: the order of the
// hits along the track and the root of each vane crossing); the chi^2, the
// adjoint and the Gauss-Newton steps run in float32.
//
// Model (perigee parameters p = (kappa, phi0, d0, z0, tan_lambda)): signed
// radius rs = 1 / kappa, normal n = (sin phi0, -cos phi0), centre
// c = (d0 + rs) n. Hit i on vane k (unit ray u_k) is predicted at the ray's
// crossing t = b + s_i sqrt(b^2 - d0 (d0 + 2 rs)), b = u_k . c (square root 0
// when the ray misses the circle), and at z = z0 + |rs| a tan_lambda with a the
// crossing's turning angle past the perigee, unwrapped against a_ref_i. The
// residuals (r - t) / sigma and (z - z_hat) / sigma make the chi^2.

#include <hip/hip_runtime.h>

#include <cmath>
#include <cstdint>

#include "hough_tf.h"

namespace hough {
namespace {

constexpr int kRefitThreads = 256;   // k_refit_gather
constexpr int kLanes = 64;           // one wave per workgroup everywhere else
constexpr int kMaxRefitHits = 128;   // hits per candidate the initial fit orders
constexpr double kTwoPi = 6.283185307179586476925286766559;
constexpr double kZOrderMM = 1.0;    // z spread above which hits are ordered by z
constexpr double kRMaxMM = 1.0e4;    // larger initial circles are lines, not helices

struct RefitHits {
    int32_t n_cand;
    const int64_t *off;   // [n_cand + 1]
    const float *r, *z;
    const int16_t *vane;
    int32_t n_vanes;
};

// ---------------------------------------------------------------------------
// initial parameters (float64)
// ---------------------------------------------------------------------------

__device__ double wrap_2pi(double x) {   // into [0, 2 pi)
    double y = fmod(x, kTwoPi);
    return y < 0.0 ? y + kTwoPi : y;
}

// Candidates per wave and hits (of candidates it fits) the wave holds at once.
// Eight candidates of a pileup batch (about 13 hits each) are two rounds of
// everything that is done per hit.
constexpr int kInitCand = 8;
constexpr int kInitHits = 256;

struct InitShared {
    double ux[kInitHits], uy[kInitHits];   // the hit's vane direction
    double x[kInitHits], y[kInitHits];     // its position; later the turning steps of the two z orders
    double al[kInitHits];                  // its turning angle; later unwrapped along the track
    float r[kInitHits], z[kInitHits];
    int16_t vane[kInitHits];
    uint8_t cand[kInitHits];               // its candidate (of the wave's)
    uint8_t ord[2][kInitHits];             // the candidate's hits by ascending key, per direction
    double cx[kInitCand], cy[kInitCand], R[kInitCand], nx[kInitCand], ny[kInitCand], d0[kInitCand];
    double a_start[kInitCand];
    int64_t b0[kInitCand];                 // its first hit in the call's arrays
    int start[kInitCand], n[kInitCand];    // its hits here
    int how[kInitCand];                    // kNone, kGap, kWalk or kWalkNan
};

enum InitHow { kNone = 0, kGap, kWalk, kWalkNan };

// Solves the 3 x 3 system A[.][0..2] v = A[.][3] by Gaussian elimination with
// partial pivoting; false when a pivot is 0.
__device__ bool solve3(double (&A)[3][4], double &D, double &E, double &F) {
#pragma unroll
    for (int col = 0; col < 3; ++col) {
        int piv = col;
        double top = fabs(A[col][col]);
#pragma unroll
        for (int row = col + 1; row < 3; ++row)
            if (fabs(A[row][col]) > top) {
                piv = row;
                top = fabs(A[row][col]);
            }
#pragma unroll
        for (int row = col + 1; row < 3; ++row)
            if (piv == row)
#pragma unroll
                for (int k = 0; k < 4; ++k) {
                    const double t = A[col][k];
                    A[col][k] = A[row][k];
                    A[row][k] = t;
                }
        if (A[col][col] == 0.0) return false;
#pragma unroll
        for (int row = col + 1; row < 3; ++row) {
            const double f = A[row][col] / A[col][col];
#pragma unroll
            for (int k = col; k < 4; ++k) A[row][k] -= f * A[col][k];
        }
    }
    F = A[2][3] / A[2][2];
    E = (A[1][3] - A[1][2] * F) / A[1][1];
    D = (A[0][3] - A[0][1] * E - A[0][2] * F) / A[0][0];
    return true;
}

// Stable insertion sort of a candidate's hits by +-z, one lane: the order of
// hits among which a z is NaN depends on how the sort compares.
__device__ void insert_by_z(const float *z, int n, bool down, uint8_t *ord) {
    for (int i = 0; i < n; ++i) {
        const float zk = down ? -z[i] : z[i];
        int j = i - 1;
        while (j >= 0) {
            const float zj = down ? -z[ord[j]] : z[ord[j]];
            if (zj <= zk) break;
            ord[j + 1] = ord[j];
            --j;
        }
        ord[j + 1] = (uint8_t)i;
    }
}

// Initial parameters. Bound by the latency of one wave's float64 work: the
// vane angles, turning angles and unwrapping steps of a hit are independent
// of the others' (a lane each), the order along the track is a rank count
// instead of a serial sort, and only the sums and the small systems are left
// to one lane per candidate. The arrays of a hit are in LDS: one thread per
// candidate had them in scratch memory (4 KB a lane), its 330 waves ran
// 920 us for 20 571 candidates of 12.9 hits; this form takes 49 us.
__global__ __launch_bounds__(kLanes) void k_refit_init(RefitHits H, float *params, float *sign, float *aref,
                                                       int32_t *status) {
    __shared__ InitShared S;
    const int lane = threadIdx.x;
    const int c0 = blockIdx.x * kInitCand;
    const int nc = min(kInitCand, H.n_cand - c0);
    const bool own = lane < nc;   // lane c: candidate c0 + c
    const int64_t first = own ? H.off[c0 + lane] : 0;
    const int n = own ? (int)(H.off[c0 + lane + 1] - first) : 0;
    // a helix needs 3 hits, and more than kMaxRefitHits are refused
    const bool takes = own && n >= 3 && n <= kMaxRefitHits;
    int before = takes ? n : 0;   // hits of the candidates up to this one (then: before it)
    for (int o = 1; o < kInitCand; o <<= 1) {
        const int u = __shfl_up(before, o, kLanes);
        if (lane >= o) before += u;
    }
    const int upto = before;
    before -= takes ? n : 0;
    float *P = params + 5 * (size_t)(c0 + (own ? lane : 0));
    if (own && !takes) {
        for (int q = 0; q < 5; ++q) P[q] = 0.0f;
        status[c0 + lane] = n < 3 ? 1 : 2;
    }
    for (unsigned long long m = __ballot(own && !takes); m != 0ull; m &= m - 1) {
        const int c = __builtin_ctzll(m);
        const int64_t b = __shfl(first, c, kLanes);
        const int nn = __shfl(n, c, kLanes);
        for (int i = lane; i < nn; i += kLanes) {
            sign[b + i] = 1.0f;
            aref[b + i] = 0.0f;
        }
    }
    // as many candidates at a time as their hits fit here (each one does)
    for (int cs = 0; cs < nc;) {
        const int base = __shfl(before, cs, kLanes);
        const unsigned long long over = __ballot(lane >= cs && lane < nc && upto - base > kInitHits);
        const int ce = over != 0ull ? __builtin_ctzll(over) : nc;
        const int total = __shfl(upto, ce - 1, kLanes) - base;
        const bool mine = takes && lane >= cs && lane < ce;
        const int st = before - base;
        __syncthreads();
        if (lane >= cs && lane < ce) {
            S.b0[lane] = first;
            S.start[lane] = st;
            S.n[lane] = takes ? n : 0;
            S.how[lane] = kNone;
        }
        __syncthreads();
        for (int c = cs; c < ce; ++c)
            for (int i = lane; i < S.n[c]; i += kLanes) {
                S.cand[S.start[c] + i] = (uint8_t)c;
                S.ord[0][S.start[c] + i] = S.ord[1][S.start[c] + i] = (uint8_t)i;
            }
        __syncthreads();
        for (int i = lane; i < total; i += kLanes) {
            const int c = S.cand[i];
            const int64_t g = S.b0[c] + (i - S.start[c]);
            const int v = H.vane[g];
            const float rf = H.r[g];
            const double ph = kTwoPi * (double)v / (double)H.n_vanes;
            const double rr = (double)rf;
            const double ux = cos(ph), uy = sin(ph);
            S.vane[i] = (int16_t)v;
            S.r[i] = rf;
            S.z[i] = H.z[g];
            S.ux[i] = ux;
            S.uy[i] = uy;
            S.x[i] = rr * ux;
            S.y[i] = rr * uy;
        }
        __syncthreads();
        double R = 0.0, d0 = 0.0, nx = 0.0, ny = 0.0;
        bool helix = false;
        if (mine) {
            // hits on at least three vanes
            const int va = S.vane[st];
            int vb = va;
            bool three = false;
            for (int i = 1; i < n; ++i) {
                const int v = S.vane[st + i];
                if (v != va) {
                    three = three || (vb != va && v != vb);
                    vb = vb == va ? v : vb;
                }
            }
            double xm = 0.0, ym = 0.0;
            for (int i = 0; i < n; ++i) {
                xm += S.x[st + i];
                ym += S.y[st + i];
            }
            xm /= n;
            ym /= n;
            // algebraic circle fit: least squares of u^2 + v^2 + D u + E v + F = 0
            double suu = 0, suv = 0, svv = 0, su = 0, sv = 0, suw = 0, svw = 0, sw = 0;
            double zmin = 1e300, zmax = -1e300;
            bool nan = false;
            for (int i = 0; i < n; ++i) {
                const double u = S.x[st + i] - xm, v = S.y[st + i] - ym, w = u * u + v * v;
                suu += u * u;
                suv += u * v;
                svv += v * v;
                su += u;
                sv += v;
                suw += u * w;
                svw += v * w;
                sw += w;
                const double zz = (double)S.z[st + i];
                zmin = fmin(zmin, zz);
                zmax = fmax(zmax, zz);
                nan = nan || zz != zz;
            }
            double A[3][4] = {{suu, suv, su, -suw}, {suv, svv, sv, -svw}, {su, sv, (double)n, -sw}};
            double D = 0.0, E = 0.0, F = 0.0;
            if (three && solve3(A, D, E, F)) {
                const double cx = xm - D / 2.0, cy = ym - E / 2.0;
                const double R2 = D * D / 4.0 + E * E / 4.0 - F;
                const double cn = sqrt(cx * cx + cy * cy);
                if (!(!(R2 > 0.0) || !(cn > 0.0) || sqrt(R2) > kRMaxMM)) {
                    helix = true;
                    R = sqrt(R2);
                    nx = cx / cn;
                    ny = cy / cn;
                    d0 = cn - R;
                    S.cx[lane] = cx;
                    S.cy[lane] = cy;
                    S.R[lane] = R;
                    S.nx[lane] = nx;
                    S.ny[lane] = ny;
                    S.d0[lane] = d0;
                    S.how[lane] = !(zmax - zmin >= kZOrderMM) ? kGap : nan ? kWalkNan : kWalk;
                }
            }
        }
        __syncthreads();
        // turning angles of the measured points past the perigee (clockwise)
        for (int i = lane; i < total; i += kLanes) {
            const int c = S.cand[i];
            if (S.how[c] == kNone) continue;
            const double v0x = -S.R[c] * S.nx[c], v0y = -S.R[c] * S.ny[c];
            const double vx = S.x[i] - S.cx[c], vy = S.y[i] - S.cy[c];
            S.al[i] = -atan2(v0x * vy - v0y * vx, v0x * vx + v0y * vy);
        }
        __syncthreads();
        // the candidate's hits in z order, ascending and descending, equal z in
        // hit order; or, for a flat track, by angle
        for (int i = lane; i < total; i += kLanes) {
            const int c = S.cand[i], s0 = S.start[c], s1 = s0 + S.n[c];
            const int how = S.how[c];
            if (how == kWalk) {
                const float zi = S.z[i];
                int up = 0, down = 0;
                for (int j = s0; j < s1; ++j) {
                    const float zj = S.z[j];
                    const bool tie = zj == zi && j < i;
                    up += zj < zi || tie ? 1 : 0;
                    down += zj > zi || tie ? 1 : 0;
                }
                S.ord[0][s0 + up] = (uint8_t)(i - s0);
                S.ord[1][s0 + down] = (uint8_t)(i - s0);
            } else if (how == kGap) {
                const double ai = S.al[i];
                int up = 0;
                for (int j = s0; j < s1; ++j) {
                    const double aj = S.al[j];
                    up += aj < ai || (aj == ai && j < i) ? 1 : 0;
                }
                S.ord[0][s0 + up] = (uint8_t)(i - s0);
            }
        }
        if (helix && S.how[lane] == kWalkNan) {
            insert_by_z(S.z + st, n, false, S.ord[0] + st);
            insert_by_z(S.z + st, n, true, S.ord[1] + st);
        }
        __syncthreads();
        // the turn from each hit to the next one in either z order
        for (int i = lane; i < total; i += kLanes) {
            const int c = S.cand[i], s0 = S.start[c];
            if (S.how[c] < kWalk || i == s0) continue;
            S.x[i] = wrap_2pi(S.al[s0 + S.ord[0][i]] - S.al[s0 + S.ord[0][i - 1]]);
            S.y[i] = wrap_2pi(S.al[s0 + S.ord[1][i]] - S.al[s0 + S.ord[1][i - 1]]);
        }
        __syncthreads();
        if (helix) {
            if (S.how[lane] >= kWalk) {
                // the hits walked in z order, ascending or descending,
                // whichever turns less in total
                double up = 0.0, down = 0.0;
                for (int i = 1; i < n; ++i) {
                    up += S.x[st + i];
                    down += S.y[st + i];
                }
                const bool dir = down < up;
                const uint8_t *ord = S.ord[dir ? 1 : 0] + st;
                const double *step = (dir ? S.y : S.x) + st;
                double acc = S.al[st + ord[0]];
                for (int i = 1; i < n; ++i) {
                    acc += step[i];
                    S.al[st + ord[i]] = acc;
                }
            } else {
                // the arc between the two sides of the largest angular gap
                const uint8_t *ord = S.ord[0] + st;
                const double a0 = S.al[st + ord[0]];
                double gmax = -1.0, far = S.al[st + ord[1]], cur = a0;
                for (int i = 0; i < n; ++i) {
                    const double nxt = i + 1 < n ? S.al[st + ord[i + 1]] : a0;
                    const double gap = i + 1 < n ? nxt - cur : a0 + kTwoPi - cur;
                    if (gap > gmax) {
                        gmax = gap;
                        far = nxt;
                    }
                    cur = nxt;
                }
                S.a_start[lane] = far;
            }
        }
        __syncthreads();
        for (int i = lane; i < total; i += kLanes) {
            const int c = S.cand[i];
            if (S.how[c] != kGap) continue;
            const double a_start = S.a_start[c];
            S.al[i] = a_start + wrap_2pi(S.al[i] - a_start);
        }
        __syncthreads();
        if (mine) {
            if (helix) {
                // z against the arc length R a
                double sm = 0.0, zm = 0.0;
                for (int i = 0; i < n; ++i) {
                    sm += R * S.al[st + i];
                    zm += (double)S.z[st + i];
                }
                sm /= n;
                zm /= n;
                double sxz = 0.0, sxx = 0.0;
                for (int i = 0; i < n; ++i) {
                    const double ds = R * S.al[st + i] - sm;
                    sxz += ds * ((double)S.z[st + i] - zm);
                    sxx += ds * ds;
                }
                const double tl = sxx > 0.0 ? sxz / sxx : 0.0;
                P[0] = (float)(1.0 / R);
                P[1] = (float)atan2(nx, -ny);
                P[2] = (float)d0;
                P[3] = (float)(zm - tl * sm);
                P[4] = (float)tl;
            } else {
                for (int q = 0; q < 5; ++q) P[q] = 0.0f;
            }
            status[c0 + lane] = helix ? 0 : 3;
        }
        // root of each hit at the initial circle: the one nearest the measured r
        for (int i = lane; i < total; i += kLanes) {
            const int c = S.cand[i];
            const int64_t g = S.b0[c] + (i - S.start[c]);
            float sg = 1.0f, ar = 0.0f;
            if (S.how[c] != kNone) {
                const double cd0 = S.d0[c], cR = S.R[c];
                const double bb = S.ux[i] * (cd0 + cR) * S.nx[c] + S.uy[i] * (cd0 + cR) * S.ny[c];
                const double disc = bb * bb - cd0 * (cd0 + 2.0 * cR);
                const double sq = sqrt(fmax(disc, 0.0));
                const double rr = (double)S.r[i];
                sg = fabs(bb + sq - rr) <= fabs(bb - sq - rr) ? 1.0f : -1.0f;
                ar = (float)S.al[i];
            }
            sign[g] = sg;
            aref[g] = ar;
        }
        cs = ce;
    }
}

// ---------------------------------------------------------------------------
// residuals and their derivatives (float32)
// ---------------------------------------------------------------------------

struct HitModel {
    float er, ez;          // residuals / sigma
    float jr[5], jz[5];    // d(er)/dp, d(ez)/dp
};

// A candidate's parameters as its hits' models use them.
struct __align__(16) Helix {
    float kappa, d0, z0, tl;
    float rs, sn, cs, pad;   // 1 / kappa, sin and cos of phi0
};

__device__ __forceinline__ Helix make_helix(const float p[5]) {
    Helix x;
    x.kappa = p[0];
    x.d0 = p[2];
    x.z0 = p[3];
    x.tl = p[4];
    x.rs = 1.0f / p[0];
    sincosf(p[1], &x.sn, &x.cs);
    x.pad = 0.0f;
    return x;
}

// A hit as its model uses it.
struct HitIn {
    float r, z, ux, uy, s, aref;   // ux, uy: its vane's direction
};

__device__ __forceinline__ HitIn load_hit(const RefitHits &H, const float *sign, const float *aref, int64_t i) {
    HitIn h;
    h.r = H.r[i];
    h.z = H.z[i];
    h.s = sign[i];
    h.aref = aref[i];
    sincosf(6.28318530717958647692f * (float)H.vane[i] / (float)H.n_vanes, &h.uy, &h.ux);
    return h;
}

// Residuals of one hit and, with DERIV, their derivatives in p.
template <bool DERIV>
__device__ __forceinline__ void hit_model(const Helix &x, const HitIn &h, float inv_sigma, HitModel &m) {
    const float kappa = x.kappa, d0 = x.d0, z0 = x.z0, tl = x.tl, rs = x.rs, sn = x.sn, cs = x.cs;
    const float r = h.r, z = h.z, ux = h.ux, uy = h.uy, s = h.s, aref = h.aref;
    const float nx = sn, ny = -cs;          // normal
    const float ox = cs, oy = sn;           // direction at the perigee
    const float mm = d0 + rs;
    const float cx = mm * nx, cy = mm * ny;
    const float bb = ux * cx + uy * cy;
    const float q = d0 * (d0 + 2.0f * rs);
    const float disc = bb * bb - q;
    const bool in = disc > 0.0f;
    const float sq = in ? sqrtf(disc) : 0.0f;
    const float t = bb + s * sq;
    const float v0x = -rs * nx, v0y = -rs * ny;
    const float vx = t * ux - cx, vy = t * uy - cy;
    const float X = v0x * vy - v0y * vx;
    const float Y = v0x * vx + v0y * vy;
    const float sg = kappa > 0.0f ? 1.0f : -1.0f;
    const float alpha = -sg * atan2f(X, Y);
    const float twopi = 6.28318530717958647692f;
    const float da = alpha - aref;
    const float a = aref + (da - twopi * rintf(da / twopi));
    const float R = fabsf(rs);
    m.er = (r - t) * inv_sigma;
    m.ez = (z - (z0 + R * a * tl)) * inv_sigma;
    if (!DERIV) return;
    const float rs2 = rs * rs;
    // d c / d (kappa, phi0, d0)
    const float dcx[3] = {-rs2 * nx, mm * ox, nx};
    const float dcy[3] = {-rs2 * ny, mm * oy, ny};
    const float dq[3] = {-2.0f * d0 * rs2, 0.0f, 2.0f * d0 + 2.0f * rs};
    // d v0 / d (kappa, phi0, d0)
    const float dv0x[3] = {rs2 * nx, -rs * ox, 0.0f};
    const float dv0y[3] = {rs2 * ny, -rs * oy, 0.0f};
    const float den = X * X + Y * Y;
    const float dR = -sg * rs2;   // d |rs| / d kappa
#pragma unroll
    for (int k = 0; k < 3; ++k) {
        const float db = ux * dcx[k] + uy * dcy[k];
        const float dsq = in ? (2.0f * bb * db - dq[k]) / (2.0f * sq) : 0.0f;
        const float dt = db + s * dsq;
        const float dvx = dt * ux - dcx[k], dvy = dt * uy - dcy[k];
        const float dX = dv0x[k] * vy + v0x * dvy - dv0y[k] * vx - v0y * dvx;
        const float dY = dv0x[k] * vx + v0x * dvx + dv0y[k] * vy + v0y * dvy;
        const float dal = -sg * (Y * dX - X * dY) / den;
        float dz = R * tl * dal;
        if (k == 0) dz += dR * a * tl;
        m.jr[k] = -dt * inv_sigma;
        m.jz[k] = -dz * inv_sigma;
    }
    m.jr[3] = 0.0f;
    m.jr[4] = 0.0f;
    m.jz[3] = -inv_sigma;
    m.jz[4] = -R * a * inv_sigma;
}

// Candidates per wave of the chi^2, gradient and Gauss-Newton kernels: eight
// (about 100 hits of a pileup batch) fill two rounds of 64 lanes with hits and
// leave eight lanes for each candidate's normal system. Few enough that 20 571
// candidates make 2.5 waves per SIMD: with 24 per wave (one wave per SIMD) an
// instruction took 10.8 cycles and 20 Gauss-Newton steps 593 us.
constexpr int kCands = 8;
constexpr int kGroup = kLanes / kCands;   // lanes per candidate
constexpr int kPer = 2;                   // hits a lane takes at a time
constexpr int kRound = kPer * kLanes;
constexpr int kKeep = 2;                  // rounds whose hits stay in registers over the Gauss-Newton steps
constexpr int kTermPitch = kRound + 1;

// The hits of a wave's candidates: any number, taken kRound at a time.
struct WaveHits {
    int64_t base;   // the first one in the call's arrays
    int total;
};

// Candidates c0 .. c0 + kCands - 1: where each one's hits start (relative to
// the wave's first) goes to off[0 .. kCands]; those past the last candidate are
// empty.
__device__ __forceinline__ WaveHits wave_hits(const RefitHits &H, int c0, int *off) {
    WaveHits W;
    W.base = H.off[c0];
    if (threadIdx.x <= kCands) off[threadIdx.x] = (int)(H.off[min(c0 + (int)threadIdx.x, H.n_cand)] - W.base);
    __syncthreads();
    W.total = off[kCands];
    return W;
}

// The candidate (of the wave's) that holds position i.
__device__ __forceinline__ int cand_of(const int *off, int i) {
    int c = 0;
#pragma unroll
    for (int step = kCands / 2; step > 0; step >>= 1)
        if (off[c + step] <= i) c += step;
    return c;
}

// Adds to acc[r] the terms of the round at position h0 that belong to sum
// t = 64 r + lane: quantity t % Q of candidate t / Q, over the candidate's hits
// in order. term[q * kTermPitch + j]: quantity q of the round's hit j.
template <int Q>
constexpr int kSums = (kCands * Q + kLanes - 1) / kLanes;

template <int Q>
__device__ __forceinline__ void add_terms(const int *off, const float *term, int h0, float (&acc)[kSums<Q>]) {
#pragma unroll
    for (int r = 0; r < kSums<Q>; ++r) {
        const int t = r * kLanes + (int)threadIdx.x;
        const int c = t < kCands * Q ? t / Q : 0;
        const int hi = t < kCands * Q ? min(off[c + 1] - h0, kRound) : 0;
        const float *const row = term + (t < kCands * Q ? t - c * Q : 0) * kTermPitch;
        int j = max(off[c] - h0, 0);
        for (; j + 4 <= hi; j += 4) {
            const float a = row[j], b = row[j + 1], x = row[j + 2], y = row[j + 3];
            acc[r] = (((acc[r] + a) + b) + x) + y;
        }
        for (; j < hi; ++j) acc[r] += row[j];
    }
}

template <int Q>
__device__ __forceinline__ void put_sums(const float (&acc)[kSums<Q>], float *sum) {
#pragma unroll
    for (int r = 0; r < kSums<Q>; ++r)
        if (r * kLanes + (int)threadIdx.x < kCands * Q) sum[r * kLanes + threadIdx.x] = acc[r];
}

// chi^2 of the wave's candidates at hx[]: sum_i er^2 + ez^2, in LDS sum[kCands].
__device__ __forceinline__ void wave_chi2(const RefitHits &H, const WaveHits &W, const int *off, const Helix *hx,
                                          const float *sign, const float *aref, float inv_sigma, float *term,
                                          float *sum) {
    float acc[kSums<1>] = {0.0f};
    for (int h0 = 0; h0 < W.total; h0 += kRound) {
        for (int j = threadIdx.x; j < min(kRound, W.total - h0); j += kLanes) {
            HitModel m;
            hit_model<false>(hx[cand_of(off, h0 + j)], load_hit(H, sign, aref, W.base + h0 + j), inv_sigma, m);
            term[j] = m.er * m.er + m.ez * m.ez;
        }
        __syncthreads();
        add_terms<1>(off, term, h0, acc);
        __syncthreads();
    }
    put_sums<1>(acc, sum);
    __syncthreads();
}

__global__ __launch_bounds__(kLanes) void k_refit_chi2(RefitHits H, const float *sign, const float *aref,
                                                       const float *params, float inv_sigma, float *chi2) {
    __shared__ int off[kCands + 1];
    __shared__ Helix hx[kCands];
    __shared__ float term[kTermPitch], sum[kCands];
    const int c = blockIdx.x * kCands + threadIdx.x;
    const bool own = threadIdx.x < kCands && c < H.n_cand;
    if (own) hx[threadIdx.x] = make_helix(params + 5 * (size_t)c);
    const WaveHits W = wave_hits(H, blockIdx.x * kCands, off);
    wave_chi2(H, W, off, hx, sign, aref, inv_sigma, term, sum);
    if (own) chi2[c] = sum[threadIdx.x];
}

// grad[c] = upstream[c] * d chi^2_c / d p_c = upstream[c] * 2 sum_i (er jr + ez jz)
__global__ __launch_bounds__(kLanes) void k_refit_grad(RefitHits H, const float *sign, const float *aref,
                                                       const float *params, const float *upstream,
                                                       float inv_sigma, float *grad) {
    __shared__ int off[kCands + 1];
    __shared__ Helix hx[kCands];
    __shared__ float term[5 * kTermPitch], sum[5 * kCands];
    const int c0 = blockIdx.x * kCands;
    const int c = c0 + threadIdx.x;
    if (threadIdx.x < kCands && c < H.n_cand) hx[threadIdx.x] = make_helix(params + 5 * (size_t)c);
    const WaveHits W = wave_hits(H, c0, off);
    float acc[kSums<5>] = {0.0f};
    for (int h0 = 0; h0 < W.total; h0 += kRound) {
        for (int j = threadIdx.x; j < min(kRound, W.total - h0); j += kLanes) {
            HitModel m;
            hit_model<true>(hx[cand_of(off, h0 + j)], load_hit(H, sign, aref, W.base + h0 + j), inv_sigma, m);
#pragma unroll
            for (int q = 0; q < 5; ++q) term[q * kTermPitch + j] = m.er * m.jr[q] + m.ez * m.jz[q];
        }
        __syncthreads();
        add_terms<5>(off, term, h0, acc);
        __syncthreads();
    }
    put_sums<5>(acc, sum);
    __syncthreads();
    if ((int)threadIdx.x < 5 * min(kCands, H.n_cand - c0)) {
        const float w = upstream != nullptr ? 2.0f * upstream[c0 + threadIdx.x / 5] : 2.0f;
        grad[5 * (size_t)c0 + threadIdx.x] = w * sum[threadIdx.x];
    }
}

// The value that lane K of this lane's group of eight holds.
template <int K>
__device__ __forceinline__ float group_lane(float v) {
    static_assert(kGroup == 8, "the swizzle keeps the upper two of five lane bits");
    return __int_as_float(__builtin_amdgcn_ds_swizzle(__float_as_int(v), (K << 5) | 0x18));
}

// Whether `ok` holds in the first five lanes of this lane's group.
__device__ __forceinline__ bool group_all5(bool ok) {
    const unsigned long long m = __ballot(ok) >> (threadIdx.x & ~(kGroup - 1));
    return (m & 0x1full) == 0x1full;
}

// Stage A of the factorisation: row A of the columns the lanes hold.
template <int A>
__device__ __forceinline__ void factor_row(int k, float (&col)[5], bool &ok) {
    float t = col[A];
    if constexpr (A > 0) t -= group_lane<A>(col[0]) * col[0];
    if constexpr (A > 1) t -= group_lane<A>(col[1]) * col[1];
    if constexpr (A > 2) t -= group_lane<A>(col[2]) * col[2];
    if constexpr (A > 3) t -= group_lane<A>(col[3]) * col[3];
    const float ua = group_lane<A>(sqrtf(fmaxf(t, 1e-30f)));
    if (k == A) ok = t > 0.0f;
    col[A] = k == A ? ua : t / ua;
}

// One damped, scaled Gauss-Newton step of the group's candidate: with
// hg[0..14] the upper triangle of H = J^T J (row-major) and hg[15..19]
// g = J^T e, solves (S H S + mu I) y = -S g, S = diag(H)^-1/2, by Cholesky
// (U^T U) and returns lane k's p_k + y_k / d_k (p when the step is not taken:
// a pivot is not positive or a parameter would not be finite). Lane b < 5 holds
// column b of U, lane 5 the right-hand side, whose forward substitution is the
// same recurrence; `u` is LDS for U's rows and the right-hand side.
__device__ __forceinline__ float gn_step(const float *hg, float mu, float p, float *u, bool &fit) {
    const int k = threadIdx.x & (kGroup - 1);
    const int b = min(k, 4);
    constexpr int kRow[5] = {0, 5, 9, 12, 14};   // index of (a, a)
    const float hv = hg[b == 0 ? 0 : b == 1 ? 5 : b == 2 ? 9 : b == 3 ? 12 : 14];
    const float db = hv > 0.0f ? sqrtf(hv) : 1.0f;
    const float d[5] = {group_lane<0>(db), group_lane<1>(db), group_lane<2>(db), group_lane<3>(db),
                        group_lane<4>(db)};
    float col[5];
#pragma unroll
    for (int a = 0; a < 5; ++a) {
        // lanes below a hold nothing in row a: any finite or other value
        const float num = k >= 5 ? -hg[15 + a] : hg[kRow[a] + max(b - a, 0)];
        const float den = k >= 5 ? d[a] : d[a] * db;
        const float q = num / den;
        col[a] = k >= 5 ? q : q + (a == b ? mu : 0.0f);
    }
    bool ok = true;
    factor_row<0>(k, col, ok);
    factor_row<1>(k, col, ok);
    factor_row<2>(k, col, ok);
    factor_row<3>(k, col, ok);
    factor_row<4>(k, col, ok);
    const bool solved = group_all5(ok);
    __syncthreads();
    if (k < 6)
#pragma unroll
        for (int a = 0; a < 5; ++a) u[a * 6 + k] = col[a];
    __syncthreads();
    float y[5];
#pragma unroll
    for (int a = 4; a >= 0; --a) {  // U y = w
        float t = u[a * 6 + 5];
#pragma unroll
        for (int c = a + 1; c < 5; ++c) t -= u[a * 6 + c] * y[c];
        y[a] = t / u[a * 6 + a];
    }
    const float yk = b == 0 ? y[0] : b == 1 ? y[1] : b == 2 ? y[2] : b == 3 ? y[3] : y[4];
    const float next = p + yk / db;
    const bool finite = group_all5(isfinite(next));
    fit = fit && solved && finite;
    return fit ? next : p;
}

// `steps` damped, scaled Gauss-Newton steps; chi2 (optional) at the end.
//
// Bound by VALU issue: per step a wave takes about 330 instructions per 64 hits
// (the model: seven correctly rounded divisions, an arc tangent, two square
// roots), about 500 for its eight normal systems and 200 for the sums. The hits'
// inputs and their vanes' directions stay in registers over the steps while
// the wave's hits fit kKeep rounds, the LDS holds one round's terms (12 KB, so
// that every wave of such a batch is resident: with 17 KB a tenth of them ran
// in a second turn, 262 us); each of the 160 sums is one lane's; eight
// lanes share a candidate's solve. One thread per candidate took 960 us for
// 20 571 candidates of 12.9 hits and 20 steps; this form takes 202 us.
__global__ __launch_bounds__(kLanes) void k_refit_gn(RefitHits H, const float *sign, const float *aref,
                                                     float *params, int steps, float mu, float inv_sigma,
                                                     const int32_t *status, float *chi2) {
    __shared__ int off[kCands + 1];
    __shared__ Helix hx[kCands];
    __shared__ float term[20 * kTermPitch], sum[20 * kCands], rows[30 * kCands];
    const int lane = threadIdx.x;
    const int c0 = blockIdx.x * kCands;
    const int g = lane / kGroup, k = lane & (kGroup - 1);   // lane k of candidate c0 + g
    const bool own = c0 + g < H.n_cand;
    // lane k < 5 holds parameter k
    float p = own && k < 5 ? params[5 * (size_t)(c0 + g) + k] : 0.0f;
    bool fit = own && (status == nullptr || status[c0 + g] == 0);
    const WaveHits W = wave_hits(H, c0, off);
    const bool keep = W.total <= kKeep * kRound;
    HitIn hit[kKeep * kPer];
    int cand[kKeep * kPer];
    if (keep) {
#pragma unroll
        for (int u = 0; u < kKeep * kPer; ++u) {
            const int i = u * kLanes + lane;
            hit[u] = HitIn{};
            cand[u] = 0;
            if (i < W.total) {
                hit[u] = load_hit(H, sign, aref, W.base + i);
                cand[u] = cand_of(off, i);
            }
        }
    }
    // the 20 quantities that hit j of a round adds to its candidate's sums
    auto put_terms = [&](const Helix &x, const HitIn &h, int j) {
        HitModel m;
        hit_model<true>(x, h, inv_sigma, m);
        int o = 0;
#pragma unroll
        for (int a = 0; a < 5; ++a) {
            term[(15 + a) * kTermPitch + j] = m.jr[a] * m.er + m.jz[a] * m.ez;
#pragma unroll
            for (int b = a; b < 5; ++b) term[o++ * kTermPitch + j] = m.jr[a] * m.jr[b] + m.jz[a] * m.jz[b];
        }
    };
    for (int it = 0;; ++it) {
        const float v[5] = {group_lane<0>(p), group_lane<1>(p), group_lane<2>(p), group_lane<3>(p),
                            group_lane<4>(p)};
        const Helix x = make_helix(v);
        if (k == 0) hx[g] = x;
        __syncthreads();
        if (it >= steps || __ballot(fit) == 0ull) break;
        float acc[kSums<20>] = {0.0f};
        if (keep) {
#pragma unroll
            for (int rd = 0; rd < kKeep; ++rd) {
                const int h0 = rd * kRound;
                if (h0 >= W.total) break;
#pragma unroll
                for (int u = 0; u < kPer; ++u)
                    if (h0 + u * kLanes + lane < W.total)
                        put_terms(hx[cand[rd * kPer + u]], hit[rd * kPer + u], u * kLanes + lane);
                __syncthreads();
                add_terms<20>(off, term, h0, acc);
                __syncthreads();
            }
        } else {
            for (int h0 = 0; h0 < W.total; h0 += kRound) {
                for (int j = lane; j < min(kRound, W.total - h0); j += kLanes)
                    put_terms(hx[cand_of(off, h0 + j)], load_hit(H, sign, aref, W.base + h0 + j), j);
                __syncthreads();
                add_terms<20>(off, term, h0, acc);
                __syncthreads();
            }
        }
        put_sums<20>(acc, sum);
        __syncthreads();
        p = gn_step(sum + 20 * g, mu, p, rows + 30 * g, fit);
    }
    if (own && k < 5) params[5 * (size_t)(c0 + g) + k] = p;
    if (chi2 != nullptr) {
        wave_chi2(H, W, off, hx, sign, aref, inv_sigma, term, sum);
        if (lane < kCands && c0 + lane < H.n_cand) chi2[c0 + lane] = sum[lane];
    }
}

// Gathers each candidate's hits (event-local indices in hit_index) from the
// batch's hit arrays: candidate c's hits land at [hit_offset_c, + n_hits_c).
__global__ __launch_bounds__(kRefitThreads) void k_refit_gather(int32_t n_cand, const hough_candidate *cand,
                                                               const int32_t *hit_index, const int64_t *ev_off,
                                                               const float *r, const float *z,
                                                               const int16_t *vane, int64_t *off, float *ro,
                                                               float *zo, int16_t *vo) {
    const int c = blockIdx.x * blockDim.x + threadIdx.x;
    if (c > n_cand) return;
    if (c == n_cand) {
        off[c] = n_cand > 0 ? cand[c - 1].hit_offset + cand[c - 1].n_hits : 0;
        return;
    }
    const hough_candidate cd = cand[c];
    off[c] = cd.hit_offset;
    const int64_t base = ev_off[cd.event];
    for (uint32_t j = 0; j < cd.n_hits; ++j) {
        const int64_t g = base + hit_index[cd.hit_offset + j];
        ro[cd.hit_offset + j] = r[g];
        zo[cd.hit_offset + j] = z[g];
        vo[cd.hit_offset + j] = vane[g];
    }
}

int grid(int n, int per) { return (n + per - 1) / per; }

hough_status check(int32_t n_cand, const int64_t *off, const float *r, const float *z, const int16_t *vane,
                   int32_t n_vanes) {
    if (n_cand < 0 || n_vanes < 1) return HOUGH_ERR_INVALID_ARG;
    if (n_cand > 0 && (!off || !r || !z || !vane)) return HOUGH_ERR_INVALID_ARG;
    return HOUGH_OK;
}

hough_status launched() { return hipGetLastError() == hipSuccess ? HOUGH_OK : HOUGH_ERR_DEVICE; }

}  // namespace
}  // namespace hough

using namespace hough;

extern "C" {

hough_status hough_refit_gather(void *stream, int32_t n_cand, const hough_candidate *cand, const int32_t *hit_index,
                                const int64_t *event_offsets, const float *r, const float *z, const int16_t *vane,
                                int64_t *hit_offsets, float *r_out, float *z_out, int16_t *vane_out) {
    if (n_cand < 0 || !hit_offsets || (n_cand > 0 && (!cand || !hit_index || !event_offsets || !r || !z || !vane ||
                                                      !r_out || !z_out || !vane_out)))
        return HOUGH_ERR_INVALID_ARG;
    hipLaunchKernelGGL(k_refit_gather, dim3(grid(n_cand + 1, kRefitThreads)), dim3(kRefitThreads), 0,
                       static_cast<hipStream_t>(stream), n_cand, cand, hit_index, event_offsets, r, z, vane,
                       hit_offsets, r_out, z_out, vane_out);
    return launched();
}

hough_status hough_refit_init(void *stream, int32_t n_cand, const int64_t *hit_offsets, const float *r,
                              const float *z, const int16_t *vane, int32_t n_vanes, float *params, float *hit_sign,
                              float *hit_aref, int32_t *status) {
    hough_status st = check(n_cand, hit_offsets, r, z, vane, n_vanes);
    if (st) return st;
    if (n_cand > 0 && (!params || !hit_sign || !hit_aref || !status)) return HOUGH_ERR_INVALID_ARG;
    if (n_cand == 0) return HOUGH_OK;
    RefitHits H{n_cand, hit_offsets, r, z, vane, n_vanes};
    hipLaunchKernelGGL(k_refit_init, dim3(grid(n_cand, kInitCand)), dim3(kLanes), 0,
                       static_cast<hipStream_t>(stream), H, params, hit_sign, hit_aref, status);
    return launched();
}

hough_status hough_refit_chi2(void *stream, int32_t n_cand, const int64_t *hit_offsets, const float *r,
                              const float *z, const int16_t *vane, int32_t n_vanes, const float *hit_sign,
                              const float *hit_aref, const float *params, float sigma, float *chi2) {
    hough_status st = check(n_cand, hit_offsets, r, z, vane, n_vanes);
    if (st) return st;
    if (!(sigma > 0.0f) || (n_cand > 0 && (!hit_sign || !hit_aref || !params || !chi2))) return HOUGH_ERR_INVALID_ARG;
    if (n_cand == 0) return HOUGH_OK;
    RefitHits H{n_cand, hit_offsets, r, z, vane, n_vanes};
    hipLaunchKernelGGL(k_refit_chi2, dim3(grid(n_cand, kCands)), dim3(kLanes), 0,
                       static_cast<hipStream_t>(stream), H, hit_sign, hit_aref, params, 1.0f / sigma, chi2);
    return launched();
}

hough_status hough_refit_grad(void *stream, int32_t n_cand, const int64_t *hit_offsets, const float *r,
                              const float *z, const int16_t *vane, int32_t n_vanes, const float *hit_sign,
                              const float *hit_aref, const float *params, const float *grad_chi2, float sigma,
                              float *grad_params) {
    hough_status st = check(n_cand, hit_offsets, r, z, vane, n_vanes);
    if (st) return st;
    if (!(sigma > 0.0f) || (n_cand > 0 && (!hit_sign || !hit_aref || !params || !grad_params)))
        return HOUGH_ERR_INVALID_ARG;
    if (n_cand == 0) return HOUGH_OK;
    RefitHits H{n_cand, hit_offsets, r, z, vane, n_vanes};
    hipLaunchKernelGGL(k_refit_grad, dim3(grid(n_cand, kCands)), dim3(kLanes), 0,
                       static_cast<hipStream_t>(stream), H, hit_sign, hit_aref, params, grad_chi2, 1.0f / sigma,
                       grad_params);
    return launched();
}

hough_status hough_refit_gauss_newton(void *stream, int32_t n_cand, const int64_t *hit_offsets, const float *r,
                                      const float *z, const int16_t *vane, int32_t n_vanes, const float *hit_sign,
                                      const float *hit_aref, const int32_t *status, float *params, int32_t steps,
                                      float damping, float sigma, float *chi2) {
    hough_status st = check(n_cand, hit_offsets, r, z, vane, n_vanes);
    if (st) return st;
    if (!(sigma > 0.0f) || steps < 0 || !(damping >= 0.0f) ||
        (n_cand > 0 && (!hit_sign || !hit_aref || !params)))
        return HOUGH_ERR_INVALID_ARG;
    if (n_cand == 0) return HOUGH_OK;
    RefitHits H{n_cand, hit_offsets, r, z, vane, n_vanes};
    hipLaunchKernelGGL(k_refit_gn, dim3(grid(n_cand, kCands)), dim3(kLanes), 0,
                       static_cast<hipStream_t>(stream), H, hit_sign, hit_aref, params, steps, damping,
                       1.0f / sigma, status, chi2);
    return launched();
}

}  // extern "C"
