// Replay of a run's hits for the gradients, shared by the plain and the
// time-of-flight backward: a window of hit entries (a Gaussian and the mask of
// the rays inside its cutoff) evaluated with its pairs spread evenly over the
// lanes, the ten sums of each Gaussian kept in its whitened frame and added to
// the accumulators in coordinates.
#pragma once

#include "gr_trace.h"

namespace gr {

// v_writelane_b32: returns old with lane `lane` replaced by the wave-uniform
// value (the LLVM intrinsic; this compiler has no builtin for it).
__device__ int lane_write(int value, int lane, int old) __asm("llvm.amdgcn.writelane.i32");

// m without its r lowest set bits (0 <= r < popcount(m)): the position of the
// r-th set bit by halving, then a mask.
__device__ inline uint64_t drop_low_bits(uint64_t m, int r) {
    uint64_t x = m;
    int pos = 0;
    for (int w = 32; w >= 1; w >>= 1) {
        const int low = __builtin_popcountll(x & ((1ull << w) - 1ull));
        const bool up = r >= low;
        r = up ? r - low : r;
        x = up ? x >> w : x;
        pos = up ? pos + w : pos;
    }
    return m & (~0ull << pos);
}

__device__ inline double gather_f64(double v, int byte) {
    const uint64_t u = __builtin_bit_cast(uint64_t, v);
    const uint32_t lo = uint32_t(__builtin_amdgcn_ds_bpermute(byte, int(uint32_t(u))));
    const uint32_t hi = uint32_t(__builtin_amdgcn_ds_bpermute(byte, int(uint32_t(u >> 32))));
    return __builtin_bit_cast(double, (uint64_t(hi) << 32) | lo);
}

// One window of up to kWin hit entries being replayed (non-empty ones only, in
// list order): the run's axis records, masks, Gaussian indices, inclusive
// prefix sums of the pair counts, and the per-entry gradient sums (SoA,
// res[k][entry]).
template <int kWin>
struct HitWindow {
    union {
        AxisRec rec[kWin];
        float part[10][64];  // lanes' closing sums, once the window's pairs are done
    };
    float res[10][kWin];
    uint64_t m[kWin];
    int32_t g[kWin];
    int32_t incl[kWin];
};

// Closing step of a replay window whose pairs are split over the lanes in
// consecutive ranges (the hit-list and TOF replays). A lane that moved on from
// an entry inside its range has stored that entry's sums already; what is left
// is each lane's sums c for the entry fe its range ends in (fe < 0: the lane
// had no pairs). Lanes ending in the same entry are consecutive, since their
// last pairs increase with the lane, so the first lane of each run adds the
// run's sums to res[.][fe] with one read-modify-write and no LDS atomics;
// part (10 x 64 floats, free by now) carries the other lanes' sums.
template <int kSlots>
__device__ inline void close_window(float (*part)[64], float (*res)[kSlots], float c[10], int fe, int lane) {
    const int fe_prev = __shfl(fe, (lane + 63) & 63, 64);
    const bool head = fe >= 0 && (lane == 0 || fe_prev != fe);
    const uint64_t heads = ballot(head);
    const int n_closing = __builtin_popcountll(ballot(fe >= 0));  // a prefix of the lanes
    __builtin_amdgcn_wave_barrier();
    if (fe >= 0 && !head)
        for (int k = 0; k < 10; ++k) part[k][lane] = c[k];
    __builtin_amdgcn_wave_barrier();
    if (head) {
        const uint64_t later = lane < 63 ? heads >> (lane + 1) : 0ull;
        const int run_end = later ? lane + 1 + __builtin_ctzll(later) : n_closing;
        for (int l = lane + 1; l < run_end; ++l)
            for (int k = 0; k < 10; ++k) c[k] += part[k][l];
        for (int k = 0; k < 10; ++k) res[k][fe] += c[k];
    }
    __builtin_amdgcn_wave_barrier();
}

// The ten sums of one Gaussian added to its accumulators, from the whitened
// frame to coordinates: x1 = a / l11 - l21 b / (l11 l22) + s1 u,
// x2 = b / l22 + s2 u, xk = u, with (x1, x2, xk) along (t1, t2, ax).
__device__ inline void unwhiten_sums(const AxisRec &G, int ax, const float c[10], float *acc, int64_t n, int64_t g) {
    const int t1 = ax == 2 ? 0 : ax + 1, t2 = ax == 0 ? 2 : ax - 1;
    const double i11 = 1.0 / G.l11, i22 = 1.0 / G.l22, i12 = -G.l21 * i11 * i22;
    const double m0 = c[1], m1 = c[2], m2 = c[3];
    const double Maa = c[4], Mbb = c[5], Muu = c[6], Mab = c[7], Mau = c[8], Mbu = c[9];
    // rows of T M for T = [[i11, i12, s1], [0, i22, s2], [0, 0, 1]]
    const double ra = fma(G.s1, Mau, fma(i12, Mab, i11 * Maa)), rb = fma(G.s1, Mbu, fma(i12, Mbb, i11 * Mab)),
                 ru = fma(G.s1, Muu, fma(i12, Mbu, i11 * Mau));
    const double sb = fma(G.s2, Mbu, i22 * Mbb), su = fma(G.s2, Muu, i22 * Mbu);
    auto add = [&](int row, double v) { atomicAdd(&acc[row * n + g], float(v)); };
    add(0, double(c[0]));
    add(1 + t1, fma(G.s1, m2, fma(i12, m1, i11 * m0)));
    add(1 + t2, fma(G.s2, m2, i22 * m1));
    add(1 + ax, m2);
    add(4 + t1, fma(G.s1, ru, fma(i12, rb, i11 * ra)));
    add(4 + t2, fma(G.s2, su, i22 * sb));
    add(4 + ax, Muu);
    add(6 + t1 + t2, fma(G.s2, ru, i22 * rb));  // xy, xz, yz at 7, 8, 9
    add(6 + t1 + ax, ru);
    add(6 + t2 + ax, su);
}

// One window of a run's hit entries: lane j holds entry j (Gaussian gj, mask mj
// of its rays; 0 = none). The T included pairs of the window, each entry's
// rounded up to a multiple of kGroup, are split evenly over the lanes (lane k
// takes [k s, k s + s) in list order), so every lane is busy however unequal the
// entries' ray counts are. With some 24 pairs per entry a few lanes come to the
// end of theirs at every step; the rounding lets them all move on at the same
// steps, once per kGroup, for a 2% longer list (fused pass, kGroup 1 / 2 / 4: 500k
// x 24 views 25.0 / 24.7 / 24.7 ms, 50k x 50 views 3.76 / 3.68 / 3.69 ms, PET
// 8.15 / 8.04 / 8.09 ms; the time-of-flight pairs are long enough to take 1:
// 13.9 / 14.0 ms). A lane that moves on from an entry stores its sums into the
// window's LDS slot for it; the sums for the entry it is in when its range ends
// are added per run of lanes ending in that entry, with no LDS atomics. At the
// end of the window lane j adds entry j's sums to the global accumulators, so
// those atomics cover consecutive Gaussians of the same leaves. `mine` is the
// lane's ray (gather_ray hands it on), pair(G, rho, h, ray, i, c) adds ray i's
// terms for record G (density rho, h in FP32) to the sums c.
template <int kWin, int kGroup, class LaneRay, class PairFn>
__device__ inline void replay_window(const AxisRec *rec, int ax, int64_t n, HitWindow<kWin> &W, int64_t gj,
                                     uint64_t mj, const LaneRay &mine, int lane, float *acc, PairFn &&pair) {
    const uint64_t below = lane ? (~0ull >> (64 - lane)) : 0ull;
    const int cj = (__builtin_popcountll(mj) + kGroup - 1) & ~(kGroup - 1);
    const int incl = wave_incl_scan(cj);
    const int T = __builtin_amdgcn_readlane(incl, 63);
    if (T == 0) return;
    // compact the entries with pairs into slots 0..nq-1
    const uint64_t nonempty = ballot(cj > 0);
    const int nq = __builtin_popcountll(nonempty);
    if (cj > 0) {
        const int q = __builtin_popcountll(nonempty & below);
        W.rec[q] = rec[gj];
        W.m[q] = mj;
        W.g[q] = int32_t(gj);
        W.incl[q] = incl;
    }
    if (lane < kWin)
        for (int k = 0; k < 10; ++k) W.res[k][lane] = 0.0f;
    __builtin_amdgcn_wave_barrier();
    const int inclq = lane < nq ? W.incl[lane] : T;
    // this lane's pairs: [p, p + left) of the window's T pairs
    const int s = (T / kGroup + 63) / 64 * kGroup;
    const int p = lane * s;
    const int left = max(0, min(s, T - p));
    // first slot whose inclusive count exceeds p (binary search over lanes)
    int lo = 0, hi = 63;
    for (int step = 0; step < 6; ++step) {
        const int mid = (lo + hi) >> 1;
        const int v = __shfl(inclq, mid, 64);
        if (v > p) hi = mid; else lo = mid + 1;
    }
    int e = left > 0 ? lo : 0;
    uint64_t m = W.m[e];
    // skip the entry's first (p - exclusive prefix) rays
    if (left > 0) m = drop_low_bits(m, p - (e > 0 ? W.incl[e - 1] : 0));
    AxisRec G = W.rec[e];
    float rho = G.rho_c * (1.0f / kSqrt2Pi), h = float(G.h);
    float c[10];
    for (int k = 0; k < 10; ++k) c[k] = 0.0f;
    for (int it = 0; it < s; it += kGroup) {
        if (it < left && m == 0) {
            // Entry e ends inside this lane's range, so no other lane
            // leaves it inside the loop: the lanes that also hold part of
            // it hold its start and add their sums after the loop. Its
            // slot is still zero here, and a plain store replaces the
            // LDS float atomic.
            for (int k = 0; k < 10; ++k) {
                W.res[k][e] = c[k];
                c[k] = 0.0f;
            }
            e = min(e + 1, nq - 1);
            m = W.m[e];
            G = W.rec[e];
            rho = G.rho_c * (1.0f / kSqrt2Pi);
            h = float(G.h);
        }
#pragma unroll
        for (int q = 0; q < kGroup; ++q) {
            const bool act = it < left && m != 0;
            // the gather runs on every lane (bpermute needs its sources active)
            const int i = act ? __builtin_ctzll(m) : lane;
            const LaneRay Rr = gather_ray(mine, i);
            if (act) {
                m &= m - 1;
                pair(G, rho, h, Rr, i, c);
            }
        }
    }
    // the closing sums take the records' place: each lane keeps its own entry's
    const AxisRec Gq = W.rec[min(lane, nq - 1)];
    close_window<kWin>(W.part, W.res, c, left > 0 ? e : -1, lane);
    if (lane < nq) {
        for (int k = 0; k < 10; ++k) c[k] = W.res[k][lane];
        unwhiten_sums(Gq, ax, c, acc, n, W.g[lane]);
    }
    __builtin_amdgcn_wave_barrier();
}

}  // namespace gr
