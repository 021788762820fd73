// Device building blocks shared by the projection kernels (plain, fused and
// time-of-flight): wave helpers, the per-lane ray and per-wave beam, the FP64
// pair core of Eq. 7, the binary and 64-wide traversals with beam tests, and
// packet location in a launch table. Everything here is inline device code.
#pragma once

#include <float.h>
#include <math.h>

#include "gr_launch.h"

namespace gr {

constexpr float kHalfLog2e = 0.72134752044448170f;  // log2(e) / 2
constexpr float kSqrt2Pi = 2.5066282746310002f;
constexpr float kBeamAbs = 1e-2f;   // absolute margin of the beam test (mm)
constexpr float kBeamRel = 1e-4f;   // relative margin on the beam's intervals
constexpr float kShadowRel = 1e-6f; // relative margin on the terms of a shadow width (FP32 rounding)
constexpr float kAxisShare = 0.25f; // a run's rays keep this share of |d|_1 along the run's axis
constexpr float kWideRun = 0.125f;  // a run this wide against the scene is looked over for a split
constexpr float kShadowPad = 0.0625f;  // shadow size, as a share of the scene, in the split's cost
constexpr float kSplitGain = 0.8f;  // a split has to cut the estimated candidates below this share

// ---------------------------------------------------------------------------
// wave helpers
// ---------------------------------------------------------------------------

template <int CTRL, int ROW_MASK = 0xF>
__device__ inline float dpp(float old, float v) {
    return __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(__builtin_bit_cast(int, old),
                                                                  __builtin_bit_cast(int, v), CTRL,
                                                                  ROW_MASK, 0xF, false));
}

__device__ inline float lane63(float v) {
    return __builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, v), 63));
}

// Sum over the 64 lanes: quad butterflies, row rotations, then row broadcasts
// 15 and 31 carry the row sums into lane 63. All lanes must be active.
__device__ inline float wave_sum(float v) {
    v += dpp<0xB1>(0.0f, v);         // quad_perm [1,0,3,2]
    v += dpp<0x4E>(0.0f, v);         // quad_perm [2,3,0,1]
    v += dpp<0x124>(0.0f, v);        // row_ror:4
    v += dpp<0x128>(0.0f, v);        // row_ror:8
    v += dpp<0x142, 0xA>(0.0f, v);   // row_bcast:15 into rows 1, 3
    v += dpp<0x143, 0xC>(0.0f, v);   // row_bcast:31 into rows 2, 3
    return lane63(v);
}

__device__ inline float wave_min(float v) {
    const float I = INFINITY;
    v = fminf(v, dpp<0xB1>(I, v));
    v = fminf(v, dpp<0x4E>(I, v));
    v = fminf(v, dpp<0x124>(I, v));
    v = fminf(v, dpp<0x128>(I, v));
    v = fminf(v, dpp<0x142, 0xA>(I, v));
    v = fminf(v, dpp<0x143, 0xC>(I, v));
    return lane63(v);
}

__device__ inline float wave_max(float v) { return -wave_min(-v); }

__device__ inline float lane_value(float v, int l) {
    return __builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, v), l));
}

__device__ inline float bcast0(float v) {
    return __builtin_bit_cast(float, __builtin_amdgcn_readfirstlane(__builtin_bit_cast(int, v)));
}

__device__ inline uint64_t ballot(bool p) { return __ballot(p); }

// Read-only data at a wave-uniform address, through the constant address
// space so that the compiler emits scalar loads into SGPRs.
template <class T>
using const_ptr = const __attribute__((address_space(4))) T *;
template <class T>
__device__ inline T sload(const T *p, int64_t i) {
#if defined(__HIP_DEVICE_COMPILE__)
    return ((const_ptr<T>)p)[i];
#else
    return p[i];  // host pass only parses device code
#endif
}

// Inclusive prefix sum over the wave (lane k gets the sum of lanes 0..k):
// shifts by 1, 2, 4, 8 within each row of 16 lanes, then the row totals
// (row_bcast:15 into rows 1 and 3, row_bcast:31 into rows 2 and 3).
__device__ inline int wave_incl_scan(int v) {
    v += __builtin_amdgcn_update_dpp(0, v, 0x111, 0xF, 0xF, true);
    v += __builtin_amdgcn_update_dpp(0, v, 0x112, 0xF, 0xF, true);
    v += __builtin_amdgcn_update_dpp(0, v, 0x114, 0xF, 0xF, true);
    v += __builtin_amdgcn_update_dpp(0, v, 0x118, 0xF, 0xF, true);
    v += __builtin_amdgcn_update_dpp(0, v, 0x142, 0xA, 0xF, false);
    v += __builtin_amdgcn_update_dpp(0, v, 0x143, 0xC, 0xF, false);
    return v;
}

// The record's density loaded with the rest of it.
__device__ inline void load_whole(const AxisRec &a) { asm volatile("" ::"s"(a.rho_c)); }

// Both records of a traversal step held in scalar registers before either is
// used, so that the step waits for memory once: the compiler otherwise issues
// each record's loads at its first use, and the density's inside the branch
// of the lanes within the cutoff, each followed by its own wait.
__device__ inline void hold_records(const AxisRec &a, const AxisRec &b) {
    asm volatile("" ::"s"(a.m1), "s"(a.rho_c), "s"(b.m1), "s"(b.rho_c));
}

// ---------------------------------------------------------------------------
// per-lane ray and per-wave beam
// ---------------------------------------------------------------------------

struct Ray {
    float o[3], d[3];
};

// The lane's ray as the pair evaluation takes it along a run's axis k: the
// line (X1 + z S1, X2 + z S2, z) and its direction.
struct RunRay {
    double X1, X2, S1, S2;
    double d1, d2, dk, dk2;  // dk2 = dk^2
    float cut;               // kappa^2, or for lanes outside the run -1, which no D >= 0 passes
};

// A run of a packet's rays as seen along one coordinate axis `ax` (t1, t2 the
// two others, cyclic): every ray is x(z) = X + z S in the planes of depth z
// across that axis, and at depth z all rays of the run lie within C +- W along
// t1 and t2, with C and W linear in z on either side of the plane zm (slopes Ca,
// Wa before it, Cb, Wb behind). All fields are wave-uniform.
struct BeamSide {
    float C, Ca, Cb, W, Wa, Wb;
    float box;               // largest |dC| + |dW|, for boxes (a depth range)
};
struct Beam {
    int ax;
    const AxisRec *rec;      // the scene's records along ax
    float zm;
    BeamSide s1, s2;         // along t1, t2
    float k11, k1k, k1kk;    // shadow half width^2 along t1: k11 s11 + k1k s1k + k1kk skk
    float k22, k2k, k2kk;    // along t2
};

__device__ inline void load_ray(const float *__restrict__ ro, const float *__restrict__ rd,
                                int64_t nr_total, int64_t idx, Ray &R) {
    for (int k = 0; k < 3; ++k) {
        R.o[k] = ro[k * nr_total + idx];
        R.d[k] = rd[k * nr_total + idx];
    }
}

// v[i] with a wave-uniform i (selects, so that v stays in registers).
template <class T>
__device__ inline T pick(const T v[3], int i) {
    return i == 0 ? v[0] : i == 1 ? v[1] : v[2];
}

// Interval of a run's rays in the planes z0, zm and z1.
struct RunSpan {
    float lo[6], hi[6];  // t1 at z0, t1 at z1, t2 at z0, t2 at z1; t1 at zm, t2 at zm
};

__device__ inline void span_of(RunSpan &r, const float *x, int from, int to, bool in) {
    for (int k = from; k < to; ++k) {
        r.lo[k] = wave_min(in ? x[k] : INFINITY);
        r.hi[k] = wave_max(in ? x[k] : -INFINITY);
    }
}

// Candidates a run is expected to meet, up to a constant: its cross-section
// widened by a typical shadow, at both ends of the scene.
__device__ inline float span_cost(const RunSpan &r, float pad) {
    return (r.hi[0] - r.lo[0] + pad) * (r.hi[2] - r.lo[2] + pad) +
           (r.hi[1] - r.lo[1] + pad) * (r.hi[3] - r.lo[3] + pad);
}

// The scene's box, from the header (one scalar load, issued beside the rays').
struct Extent {
    int32_t lo[3], hi[3];  // FP32 bits: integers are selected in scalar registers
};

__device__ inline Extent scene_extent(const SceneView &S) {
    const AccelHeader H = sload(S.hdr, 0);
    Extent E;
    for (int k = 0; k < 3; ++k) {
        E.lo[k] = __builtin_bit_cast(int32_t, H.root_box[k]);
        E.hi[k] = __builtin_bit_cast(int32_t, H.root_box[3 + k]);
    }
    return E;
}

// Takes the next run off the packet's rays still to do (todo, not empty) and
// builds its beam; returns the run's lanes, or 0 when the first ray is not a
// line (zero or non-finite: it meets nothing) and was dropped.
//
// A run is a stretch of consecutive rays that one beam bounds well. The axis
// is the largest component of the first ray's direction; a ray that is not
// mostly along it ends the run. A run that is wide against the scene is cut at
// the largest jump between neighbouring rays when the two parts' beams together
// are clearly smaller than its own: packets that straddle two detector rows or
// two views (detectors that are no multiple of the packet tile) otherwise meet
// a whole slab of the scene, or all of it, on every lane. An ordinary packet is
// one run. Measured against one general beam per packet: 7 views of 61 x 47 with
// 3,001 Gaussians, forward and backward 1196 -> 488 us; 7 views of 262 x 31 with
// 44,430 Gaussians 17.4 -> 3.0 ms; ordinary packets (500k Gaussians, 16 views of
// 512 x 512) 9.29 -> 8.54 ms through the cheaper leaf test; a single small view,
// which waits for each step of one wave, 26.0 -> 28.1 us.
//
// The bounds: min and max over the rays of the linear x(z) lie inside the
// chords between their values in two planes. Three planes are used, the scene's
// two ends z0, z1 and zm at the first ray's origin (the foot from the
// isocentre in the generators' rays): a cone's rays spread evenly, so one chord
// would do, but the views of a PET packet cross near their feet and spread to
// both ends. A Gaussian's
// shadow along a ray of slope S has half width sqrt(v^T M v) with v = (1, -S)
// in the (t, ax) plane and M = kappa^2 Sigma; over slopes S +- D it is at most
// h(S) + D sqrt(Mkk), and (h + y)^2 <= (1 + 2D) h^2 + (1 + 1/(2D)) y^2 makes
// that one quadratic form (the split 2D is near the best for shadows of about
// the Gaussian's depth). kShadowRel covers the form's FP32 cancellation.
__device__ inline uint64_t next_run(const Extent &E, const Ray &R, uint64_t &todo, int lane, Beam &B,
                                    RunRay &Q) {
    const int first = __builtin_ctzll(todo);
    const float f0 = fabsf(lane_value(R.d[0], first)), f1 = fabsf(lane_value(R.d[1], first)),
                f2 = fabsf(lane_value(R.d[2], first));
    const int ax = __builtin_amdgcn_readfirstlane(f0 >= f1 && f0 >= f2 ? 0 : f1 >= f2 ? 1 : 2);
    const int t1 = ax == 2 ? 0 : ax + 1, t2 = ax == 0 ? 2 : ax - 1;
    const float dk = pick(R.d, ax);
    Q.dk = dk;
    Q.d1 = pick(R.d, t1);
    Q.d2 = pick(R.d, t2);
    Q.dk2 = Q.dk * Q.dk;
    const double inv = 1.0 / Q.dk;
    Q.S1 = Q.d1 * inv;
    Q.S2 = Q.d2 * inv;
    const double ok = double(pick(R.o, ax));
    Q.X1 = fma(-ok, Q.S1, double(pick(R.o, t1)));
    Q.X2 = fma(-ok, Q.S2, double(pick(R.o, t2)));
    const float S1 = float(Q.S1), S2 = float(Q.S2);
    const bool good = fabsf(dk) >= kAxisShare * (fabsf(R.d[0]) + fabsf(R.d[1]) + fabsf(R.d[2])) && dk != 0.0f &&
                      fabsf(float(Q.X1)) < FLT_MAX && fabsf(float(Q.X2)) < FLT_MAX;
    const uint64_t ends = ballot(!good) & todo;
    if ((ends >> first) & 1ull) {
        todo &= todo - 1;
        return 0;
    }
    uint64_t run = ends ? todo & ((1ull << __builtin_ctzll(ends)) - 1ull) : todo;
    auto lo = [&](int k) { return __builtin_bit_cast(float, pick(E.lo, k)); };
    auto hi = [&](int k) { return __builtin_bit_cast(float, pick(E.hi, k)); };
    const float z0 = lo(ax), z1 = hi(ax);
    const float scene = fmaxf(hi(t1) - lo(t1), hi(t2) - lo(t2));
    const float depth = z1 - z0;
    const float zm = fminf(fmaxf(lane_value(pick(R.o, ax), first), z0 + 0.125f * depth), z1 - 0.125f * depth);
    float x[6];
    {
        const double z[3] = {z0, z1, zm};
        for (int k = 0; k < 3; ++k) {
            x[k < 2 ? k : 4] = float(fma(z[k], Q.S1, Q.X1));
            x[k < 2 ? 2 + k : 5] = float(fma(z[k], Q.S2, Q.X2));
        }
    }
    RunSpan r;
    for (;;) {
        const bool in = (run >> lane) & 1ull;
        span_of(r, x, 0, 4, in);
        float wide = 0.0f;
        for (int k = 0; k < 4; ++k) wide = fmaxf(wide, r.hi[k] - r.lo[k]);
        if (!(wide > kWideRun * scene)) break;
        float jump = 0.0f;
        for (int k = 0; k < 4; ++k) jump = fmaxf(jump, fabsf(x[k] - __shfl(x[k], (lane + 63) & 63, 64)));
        if (!in || lane == __builtin_ctzll(run)) jump = -1.0f;
        const float most = wave_max(jump);
        if (!(most > 0.0f)) break;
        const uint64_t low = run & ((1ull << __builtin_ctzll(ballot(jump == most))) - 1ull);
        const bool in_low = (low >> lane) & 1ull;
        const float pad = kShadowPad * scene;
        RunSpan a, b;
        span_of(a, x, 0, 4, in_low);
        span_of(b, x, 0, 4, in && !in_low);
        if (!(span_cost(a, pad) + span_cost(b, pad) < kSplitGain * span_cost(r, pad))) break;
        run = low;
    }
    todo &= ~run;
    const bool in = (run >> lane) & 1ull;
    const float s1lo = wave_min(in ? S1 : INFINITY), s1hi = wave_max(in ? S1 : -INFINITY);
    const float s2lo = wave_min(in ? S2 : INFINITY), s2hi = wave_max(in ? S2 : -INFINITY);
    span_of(r, x, 4, 6, in);
    for (int k = 0; k < 6; ++k) {
        const float m = kBeamAbs + kBeamRel * fmaxf(fabsf(r.lo[k]), fabsf(r.hi[k]));
        r.lo[k] -= m;
        r.hi[k] += m;
    }
    // the values are the same on all lanes: keep them in scalar registers
    const float ia = 0.5f / (zm - z0), ib = 0.5f / (z1 - zm);
    auto side = [&](int e0, int e1, int m) {
        const float c0 = r.hi[e0] + r.lo[e0], c1 = r.hi[e1] + r.lo[e1], cm = r.hi[m] + r.lo[m];
        const float w0 = r.hi[e0] - r.lo[e0], w1 = r.hi[e1] - r.lo[e1], wm = r.hi[m] - r.lo[m];
        BeamSide s;
        s.C = bcast0(0.5f * cm);
        s.Ca = bcast0((cm - c0) * ia);
        s.Cb = bcast0((c1 - cm) * ib);
        s.W = bcast0(0.5f * wm);
        s.Wa = bcast0((wm - w0) * ia);
        s.Wb = bcast0((w1 - wm) * ib);
        s.box = bcast0(fmaxf(fabsf(s.Ca), fabsf(s.Cb)) + fmaxf(fabsf(s.Wa), fabsf(s.Wb)));
        return s;
    };
    B.ax = ax;
    B.zm = bcast0(zm);
    B.s1 = side(0, 1, 4);
    B.s2 = side(2, 3, 5);
    const float c1 = 0.5f * (s1lo + s1hi), c2 = 0.5f * (s2lo + s2hi);
    const float D1 = 0.5f * (s1hi - s1lo) + 1e-6f * (1.0f + fabsf(c1));
    const float D2 = 0.5f * (s2hi - s2lo) + 1e-6f * (1.0f + fabsf(c2));
    const float q1 = 1.0f + 2.0f * D1, q2 = 1.0f + 2.0f * D2;
    B.k11 = bcast0(q1 * (1.0f + kShadowRel));
    B.k1k = bcast0(-2.0f * c1 * q1);
    B.k1kk = bcast0(q1 * c1 * c1 * (1.0f + kShadowRel) + D1 * D1 + 0.5f * D1);
    B.k22 = bcast0(q2 * (1.0f + kShadowRel));
    B.k2k = bcast0(-2.0f * c2 * q2);
    B.k2kk = bcast0(q2 * c2 * c2 * (1.0f + kShadowRel) + D2 * D2 + 0.5f * D2);
    return run;
}

// Slab test of an infinite line against a box (min xyz, max xyz). An empty
// box (min > max) never hits.
struct RayInv {
    float inv[3], oinv[3];  // reciprocal direction and o * inv
};

__device__ inline RayInv ray_inv(const Ray &R) {
    RayInv v;
    for (int k = 0; k < 3; ++k) {
        v.inv[k] = R.d[k] != 0.0f ? 1.0f / R.d[k] : copysignf(1e30f, R.d[k]);
        v.oinv[k] = R.o[k] * v.inv[k];
    }
    return v;
}

__device__ inline bool slab(const float *b, const RayInv &R) {
    const float tx0 = fmaf(b[0], R.inv[0], -R.oinv[0]), tx1 = fmaf(b[3], R.inv[0], -R.oinv[0]);
    const float ty0 = fmaf(b[1], R.inv[1], -R.oinv[1]), ty1 = fmaf(b[4], R.inv[1], -R.oinv[1]);
    const float tz0 = fmaf(b[2], R.inv[2], -R.oinv[2]), tz1 = fmaf(b[5], R.inv[2], -R.oinv[2]);
    const float tmin = fmaxf(fmaxf(fminf(tx0, tx1), fminf(ty0, ty1)), fminf(tz0, tz1));
    const float tmax = fminf(fminf(fmaxf(tx0, tx1), fmaxf(ty0, ty1)), fmaxf(tz0, tz1));
    return tmin <= tmax && b[0] <= b[3];
}

// ---------------------------------------------------------------------------
// the closed form for one (ray, Gaussian) pair
// ---------------------------------------------------------------------------

// Core of Eq. 7 for one pair, in FP64: A and the numerator N = C A - B^2 of
// D = N / A, along a run's axis. Eq. 7 does not change when the origin slides
// along the line; with the origin in the plane z = mk, e its offset
// from the mean there and g the direction less its conditional part, whitened
// to (a, b) and (c, d): C = a^2 + b^2, A = c^2 + d^2 + h dk^2, B = a c + b d and,
// by Lagrange's identity, N = C A - B^2 = (a d - b c)^2 + h dk^2 C. 21 FP64
// operations instead of the 26 of A, B, C from P, from a record of the same size
// and 16 instead of 24 registers of ray, and sums of squares in place of the
// cancelling C A - B^2. The scale is Eq. 7's own, so A and N round to the same
// FP32 values and the cutoff takes the same decisions. The forward is bound by
// the issue of these instructions: 500k Gaussians, 16 views of 512 x 512,
// 8.54 -> 8.11 ms; 50k, 50 views of 256 x 256, 2.03 -> 1.83 ms (with the leaf
// fields laid together).
struct AxisCore {
    double a, b, c, d, A, N;
};

__device__ inline void axis_core(const AxisRec &G, const RunRay &Q, AxisCore &k) {
    const double e1 = fma(G.mk, Q.S1, Q.X1 - G.m1), e2 = fma(G.mk, Q.S2, Q.X2 - G.m2);
    const double g1 = fma(-G.s1, Q.dk, Q.d1), g2 = fma(-G.s2, Q.dk, Q.d2);
    k.a = fma(G.l21, e2, G.l11 * e1);
    k.b = G.l22 * e2;
    k.c = fma(G.l21, g2, G.l11 * g1);
    k.d = G.l22 * g2;
    const double hk = G.h * Q.dk2;
    const double w = fma(k.a, k.d, -(k.b * k.c));
    k.A = fma(k.d, k.d, fma(k.c, k.c, hk));
    k.N = fma(w, w, hk * fma(k.b, k.b, k.a * k.a));
}

// D = N / A and r = 1/sqrt(A) in FP32 (one transcendental serves both).
template <class Core>
__device__ inline void pair_D(const Core &c, float &D, float &r) {
    r = __builtin_amdgcn_rsqf(float(c.A));
    D = (float(c.N) * r) * r;
}

__device__ inline float gauss_exp(float D) { return __builtin_amdgcn_exp2f(-kHalfLog2e * D); }

// ---------------------------------------------------------------------------
// traversal
// ---------------------------------------------------------------------------

// Candidates of leaf l for this run, as a 64-bit mask over its Gaussians: the
// mean's offset from the beam at the mean's depth against the beam's and the
// shadow's half widths, along both transverse axes. 8 loads and about 33
// instruction slots per leaf (two of them square roots); the general frame it
// replaced took three quadratic forms of six terms and 30 reloads of spilled
// scalars per leaf. A leaf's fields lie together (arrays of `leaf` floats), so
// their addresses are the leaf's and small offsets; all eight loads go out
// before the first is used.
__device__ inline uint64_t leaf_candidates(const SceneView &S, const Beam &B, int l, int lane,
                                           int64_t &start) {
    const int leaf = S.leaf;
    start = int64_t(l) * leaf;
    const int64_t rem = S.n - start;
    const int cnt = rem < leaf ? int(rem) : leaf;
    bool cand = false;
    if (lane < cnt) {
        const int ax = B.ax, t1 = ax == 2 ? 0 : ax + 1, t2 = ax == 0 ? 2 : ax - 1;
        const float *c = S.cull + start * kCullFields;  // xy xz yz sit at 6, 7, 8: field 5 + i + j
        auto field = [&](int f) { return (c + f * leaf)[lane]; };
        const float z = field(ax), m1 = field(t1), m2 = field(t2);
        const float skk = field(3 + ax), s11 = field(3 + t1), s22 = field(3 + t2);
        const float s1k = field(5 + t1 + ax), s2k = field(5 + t2 + ax);
        const float v1 = fmaf(B.k1kk, skk, fmaf(B.k1k, s1k, B.k11 * s11));
        const float v2 = fmaf(B.k2kk, skk, fmaf(B.k2k, s2k, B.k22 * s22));
        // the hardware square root (about 1 ulp) is well inside the margins
        const float u = z - B.zm, ua = fminf(u, 0.0f), ub = fmaxf(u, 0.0f);
        const float h1 = __builtin_amdgcn_sqrtf(fmaxf(v1, 0.0f)) + fmaf(ub, B.s1.Wb, fmaf(ua, B.s1.Wa, B.s1.W));
        const float h2 = __builtin_amdgcn_sqrtf(fmaxf(v2, 0.0f)) + fmaf(ub, B.s2.Wb, fmaf(ua, B.s2.Wa, B.s2.W));
        const bool in1 = fabsf(fmaf(ub, B.s1.Cb, fmaf(ua, B.s1.Ca, B.s1.C - m1))) <= h1;
        const bool in2 = fabsf(fmaf(ub, B.s2.Cb, fmaf(ua, B.s2.Ca, B.s2.C - m2))) <= h2;
        cand = in1 & in2;
    }
    return ballot(cand);
}

template <class LeafFn>
__device__ inline void traverse(const SceneView &S, const Ray &R, bool active, int lane,
                                LeafFn &&leaf_fn) {
    const AccelHeader *hdr = S.hdr;
    const AccelHeader H = sload(hdr, 0);
    const int root = H.root;
    const RayInv V = ray_inv(R);
    float rb[6];
    for (int k = 0; k < 6; ++k) rb[k] = H.root_box[k];
    if (ballot(active && slab(rb, V)) == 0) return;
    if (root < 0) {
        if (~root < S.n_leaves) leaf_fn(~root);
        return;
    }
    int stack = 0;  // lane k holds stack slot k
    int sp = 0;
    int node = root;
    int32_t err = 0;
    // every node is entered at most once per packet, so this cap is never
    // reached on a well-formed tree; it bounds the loop if the tree is corrupt
    const int64_t cap = 2 * int64_t(S.n_nodes) + 2;
    for (int64_t it = 0;; ++it) {
        if (it >= cap || node < 0 || node >= S.n_nodes) {
            err |= it >= cap ? kFlagTraversalCap : kFlagTreeCorrupt;
            break;
        }
        const Node nd = sload(S.nodes, node);
        const bool h0 = active && slab(nd.b, V);
        const bool h1 = active && slab(nd.b + 6, V);
        const uint64_t m0 = ballot(h0), m1 = ballot(h1);
        const int c0 = nd.child[0];
        const int c1 = nd.child[1];
        int next = -1;
        bool have = false;
        int lv0 = -1, lv1 = -1;  // leaves to visit from this node
        if (m0) {
            if (c0 < 0) {
                if (~c0 < S.n_leaves) lv0 = ~c0; else err |= kFlagTreeCorrupt;
            } else {
                next = c0;
                have = true;
            }
        }
        if (m1) {
            if (c1 < 0) {
                if (~c1 < S.n_leaves) lv1 = ~c1; else err |= kFlagTreeCorrupt;
            } else if (!have) {
                next = c1;
                have = true;
            } else if (sp < 64) {
                stack = (lane == sp) ? c1 : stack;
                ++sp;
            } else {
                err |= kFlagStackOverflow;
            }
        }
        for (int k = 0; k < 2; ++k) {
            const int lf = k == 0 ? lv0 : lv1;
            if (lf >= 0) leaf_fn(lf);
        }
        if (!have) {
            if (sp == 0) break;
            --sp;
            next = __builtin_amdgcn_readlane(stack, sp);
        }
        node = next;
    }
    if (err && lane == 0) atomicOr(const_cast<int32_t *>(&hdr->flags), err);
}

// Node count and offset of level lv of the wide hierarchy (level 0 = leaves;
// each level above has ceil(count / 64) nodes), from wave-uniform scalars.
__device__ inline void level_info(int n_leaves, int lv, int &cnt, int &off) {
    cnt = n_leaves;
    off = 0;
    for (int k = 0; k < lv; ++k) {
        off += cnt;
        cnt = (cnt + kWide - 1) / kWide;
    }
}

// Ballot over up to 64 consecutive nodes [first, first + cnt) of one level of
// the wide hierarchy: lane k tests node first + k against the beam, whose
// centre and half width are taken at the box's middle depth and widened by
// what they change over its depth. An empty box (lo > hi) never hits.
__device__ inline uint64_t wide_children(const SceneView &S, const Beam &B, int level_off, int first,
                                         int cnt, int lane) {
    bool hit = false;
    if (lane < cnt) {
        const int ax = B.ax, t1 = ax == 2 ? 0 : ax + 1, t2 = ax == 0 ? 2 : ax - 1;
        const float *w = S.wbox + level_off + first;
        const int64_t t = S.wide_total;
        const float lok = (w + ax * t)[lane], lo1 = (w + t1 * t)[lane], lo2 = (w + t2 * t)[lane];
        const float hik = (w + (3 + ax) * t)[lane], hi1 = (w + (3 + t1) * t)[lane], hi2 = (w + (3 + t2) * t)[lane];
        const float z = 0.5f * (lok + hik), hz = 0.5f * (hik - lok);
        const float u = z - B.zm, ua = fminf(u, 0.0f), ub = fmaxf(u, 0.0f);
        auto meets = [&](const BeamSide &s, float lo, float hi) {
            const float w = fmaf(ub, s.Wb, fmaf(ua, s.Wa, s.W));
            return fabsf(fmaf(ub, s.Cb, fmaf(ua, s.Ca, s.C)) - 0.5f * (lo + hi)) <=
                   fmaf(0.5f, hi - lo, fmaf(hz, s.box, w));
        };
        hit = meets(B.s1, lo1, hi1) && meets(B.s2, lo2, hi2);
    }
    return ballot(hit);
}

// per-wave LDS stack entries: a popped node pushes at most 64 children, so the
// depth never exceeds 64 per level below the top
constexpr int kWideStack = 64 * (kMaxLevels - 1);

// Packet traversal of the wide hierarchy with beam tests, 64 boxes per wave
// step. Pending internal nodes wait on a per-wave LDS stack (entry = level in
// the top 4 bits, node index below); leaves are handed to leaf_fn as soon as
// their parent's ballot names them, from a single call site.
template <class LeafFn>
__device__ inline void traverse_wide(const SceneView &S, const Beam &B, int lane, uint32_t *stack,
                                     LeafFn &&leaf_fn) {
    const int top = S.n_levels - 1;
    int n_top, top_off;
    level_info(S.n_leaves, top, n_top, top_off);
    int sp = 0;          // wave-uniform stack depth
    int next_root = 0;   // next chunk of top-level nodes (children of a virtual root)
    int32_t err = 0;
    while (true) {
        int lv, first, cnt, off;
        if (sp > 0) {
            --sp;
            const uint32_t e = uint32_t(__builtin_amdgcn_readfirstlane(int(stack[sp])));
            lv = int(e >> 28) - 1;  // children of a node at level (e >> 28)
            first = int(e & 0x0FFFFFFFu) * kWide;
            int lc;
            level_info(S.n_leaves, lv, lc, off);
            cnt = min(kWide, lc - first);
        } else if (next_root < n_top) {
            lv = top;
            off = top_off;
            first = next_root;
            cnt = min(kWide, n_top - next_root);
            next_root += kWide;
        } else {
            break;
        }
        uint64_t mask = wide_children(S, B, off, first, cnt, lane);
        if (lv == 0) {
            while (mask) {
                const int c = first + __builtin_ctzll(mask);
                mask &= mask - 1;
                leaf_fn(c);
            }
        } else {
            const int nh = __builtin_popcountll(mask);
            if (sp + nh > kWideStack) {
                err |= kFlagStackOverflow;
                continue;
            }
            // lowest child on top of the stack, so children are visited in order
            if ((mask >> lane) & 1ull) {
                const int above = __builtin_popcountll(mask >> lane) - 1;
                stack[sp + above] = (uint32_t(lv) << 28) | uint32_t(first + lane);
            }
            __builtin_amdgcn_wave_barrier();
            sp += nh;
        }
    }
    if (err && lane == 0) atomicOr(const_cast<int32_t *>(&S.hdr->flags), err);
}

// The leaves of a traversal that part `part` of `parts` (a power of 2) takes:
// every parts-th, in the order they come.
struct Part {
    int mask, part;
};

// Walks the scene for one run: mode 2 = wide hierarchy (default), 1 = binary
// LBVH with slab tests of the run's rays (`in`).
template <class LeafFn>
__device__ inline void traverse_run(int mode, const SceneView &S, const Ray &R, const Beam &B, bool in, int lane,
                                    uint32_t *stack, Part part, LeafFn &&leaf_fn) {
    int ord = 0;
    auto leaf = [&](int l) {
        if ((ord++ & part.mask) == part.part) leaf_fn(l);
    };
    if (mode == 1)
        traverse(S, R, in, lane, leaf);
    else
        traverse_wide(S, B, lane, stack, leaf);
}

// Takes the rays of `todo` run by run: f(in, Q, B) is called for each run, with
// `in` true on its lanes and Q the lane's ray (whose cut lets no lane outside
// the run count).
template <class RunFn>
__device__ inline void for_runs(const SceneView &S, const Ray &R, uint64_t todo, int lane, RunFn &&run_fn) {
    if (S.n == 0) return;
    const Extent E = scene_extent(S);
    while (todo) {
        Beam B;
        RunRay Q;
        const uint64_t run = next_run(E, R, todo, lane, B, Q);
        if (!run) continue;
        const bool in = (run >> lane) & 1ull;
        Q.cut = in ? S.kappa2 : -1.0f;
        B.rec = axis_rec_of(S, B.ax);
        run_fn(in, Q, B);
    }
}

__device__ inline int64_t logical_block(int xcd_remap) {
    const int64_t b = blockIdx.x;
    if (xcd_remap == 2) return b;
    const int64_t G = gridDim.x, nx = 8;
    const int64_t per = G / nx, rem = G % nx;
    const int64_t x = b % nx, k = b / nx;
    return x < rem ? x * (per + 1) + k : rem * (per + 1) + (x - rem) * per + k;
}

// Locates this wave's packet: its segment, and the lane's ray and output.
struct PacketRef {
    int seg;
    int64_t ray;   // index of this lane's ray in the segment's arrays (the packet's first
                   // ray when the lane is past the segment's end)
    int64_t out;   // output index of this lane
    bool active;
};

__device__ inline bool locate_packet(const LaunchTable &T, int64_t packet, int lane, PacketRef &P) {
    if (packet >= T.n_packets) return false;
    int s = 0;
    for (int k = 1; k < T.n_segs; ++k)
        if (packet >= T.segs[k].first_packet) s = k;
    const Segment &sg = T.segs[s];
    const int64_t local0 = (packet - sg.first_packet) * 64;
    const int64_t local = local0 + lane;
    P.seg = s;
    P.active = local < sg.n_rays;
    P.ray = sg.ray_offset + (P.active ? local : local0);
    P.out = sg.out_offset + local;
    return true;
}

// Next packet of a persistent launch: lane 0 takes a ticket from the work
// counter and the wave shares it.
__device__ inline int64_t next_packet(uint32_t *counter, int lane) {
    uint32_t t = 0;
    if (lane == 0) t = atomicAdd(counter, 1u);
    return int64_t(uint32_t(__builtin_amdgcn_readfirstlane(int(t))));
}

}  // namespace gr
