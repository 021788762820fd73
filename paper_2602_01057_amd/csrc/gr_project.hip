// Ray-packet projection kernels: forward (Eq. 12 with the kappa cutoff),
// backward (gradient of a per-ray loss) and the fused forward -> loss ->
// backward pass.
//
// One wave64 owns one packet of 64 consecutive rays (one lane per ray):
//  1. the packet's rays are taken in runs that one "beam" bounds well (an
//     ordinary packet is one run, next_run in gr_trace.h): every line as
//     x(z) = X + z S across the coordinate axis it mostly follows, and the
//     run's [min, max] of x in three planes, reduced with DPP;
//  2. the wave walks the 64-wide box hierarchy over the Morton-ordered leaves
//     (64 child boxes tested against the beam per wave step, pending nodes on
//     a per-wave LDS stack), or the binary LBVH with per-ray slab tests;
//  3. at a leaf, up to 64 Gaussians are tested lane-parallel against the beam
//     (the mean's offset at its depth against the beam's and the kappa
//     ellipsoid's shadow's half widths), giving a 64-bit candidate mask;
//  4. for each candidate the 80-byte record of the run's axis is fetched with scalar
//     loads and every lane evaluates the closed form for its ray.
//
// Closed form (Sec. 3.2-3.3, Eq. 7-11). With delta = o - mu, the literal
// A = d^T P d, B = d^T P delta, C = delta^T P delta and D = C - B^2/A are
// evaluated in FP64, which runs at the full non-packed FP32 rate on CDNA4, from
// records of the Gaussians as seen along the run's axis (axis_core in
// gr_trace.h: the same A and C A - B^2 as sums of squares, 21 operations). Only
// the transcendentals run in FP32: r = rsqrt(A), D = (C A - B^2) r^2,
// T = rho sqrt(2 pi) r exp2(-D log2(e)/2) when D <= kappa^2; the per-ray sum
// accumulates in FP64.
//
// Gradient (not in the paper; derived from Eq. 11): with t* = -B/A and
// p = delta + t* d (the line's closest point to mu in the metric P),
//   dT/drho = T/rho, dT/dmu = T P p, dT/dP = -(T/2)(p p^T + d d^T/A)
// (the last by the envelope theorem on D = min_t). Per Gaussian the backward
// sums, in FP32,
//   g_rho = sum w T/rho, m = sum w T p, M = sum w T (p p^T + d d^T / A)
// (10 floats) and adds them to the Gaussian's accumulators with float
// atomics; k_epilogue maps them to mean, scale and quaternion gradients. The
// fused pass records each run's (Gaussian, ray mask) hit list in its forward
// half and replays it with the pairs spread evenly over the lanes; with dL/dI
// given, or for a list that outgrew its region, the traversal runs again with
// the cutoff test alone and its hits are replayed window by window.
#include <algorithm>

#include "gr_replay.h"

namespace gr {

// ---------------------------------------------------------------------------
// kernels
// ---------------------------------------------------------------------------

// Forward sum over up to 64 candidate Gaussians (mask, at(bit) their position),
// two records per step. The compiler issues each record's scalar loads at its first use; the 8
// waves per SIMD of k_forward hide that latency. The density is taken with the
// record (load_whole): inside the branch of the lanes within the cutoff, where
// the compiler would put it, it is a second wait per pair (50k Gaussians, 50
// views of 256 x 256: 1819 -> 1781 us, one small view 14.3 -> 13.7 us, the 500k
// scene the same). Holding both records before the first evaluation
// (hold_records, as the recording loop of the fused pass does) is slower here:
// 1873 us, more scalar registers spill at 8 waves.
template <bool kStats, class At>
__device__ inline void leaf_forward(const AxisRec *rec, const RunRay &Q, uint64_t mask, At &&at, double &acc,
                                    uint32_t &n_inc, uint32_t &n_hitc) {
    const float k2 = Q.cut;
    while (mask) {
        const int j0 = __builtin_ctzll(mask);
        mask &= mask - 1;
        const bool two = mask != 0;
        const int j1 = two ? __builtin_ctzll(mask) : j0;
        if (two) mask &= mask - 1;
        const AxisRec G0 = sload(rec, at(j0));
        const AxisRec G1 = sload(rec, at(j1));
        AxisCore c;
        float D, r;
        load_whole(G0);
        axis_core(G0, Q, c);
        pair_D(c, D, r);
        if (kStats) n_hitc += ballot(D <= k2) != 0 ? 1u : 0u;
        if (D <= k2) {
            acc += double(G0.rho_c * r * gauss_exp(D));
            if (kStats) ++n_inc;
        }
        if (two) {
            load_whole(G1);
            axis_core(G1, Q, c);
            pair_D(c, D, r);
            if (kStats) n_hitc += ballot(D <= k2) != 0 ? 1u : 0u;
            if (D <= k2) {
                acc += double(G1.rho_c * r * gauss_exp(D));
                if (kStats) ++n_inc;
            }
        }
    }
}

// Eq. 7 for one pair in FP32 from the compact record (the forward's FP32
// precision mode). The offset o - mu is kept exactly as hi + lo (TwoSum), the
// origin slides along the line to the point nearest mu (t0 = -hi.d / d.d;
// sliding does not change the integral), and with u = W delta', v = W d
// (P = W^T W): A = v.v, B = u.v and D = |u - (B/A) v|^2, which loses far less
// to cancellation than C - B^2/A. r = 1/sqrt(A).
__device__ inline void pair_core32(const GaussRec32 &G, const Ray &R, float inv_dd, float &D, float &r) {
    float hi[3], lo[3];
    for (int k = 0; k < 3; ++k) {
        const float a = R.o[k], b = -G.mu[k];
        const float s = a + b;
        const float bv = s - a;
        lo[k] = (a - (s - bv)) + (b - bv);
        hi[k] = s;
    }
    const float t0 = -(hi[0] * R.d[0] + hi[1] * R.d[1] + hi[2] * R.d[2]) * inv_dd;
    float dl[3];
    for (int k = 0; k < 3; ++k) dl[k] = fmaf(t0, R.d[k], hi[k]) + lo[k];
    float u[3], v[3];
    for (int a = 0; a < 3; ++a) {
        u[a] = G.W[3 * a] * dl[0] + G.W[3 * a + 1] * dl[1] + G.W[3 * a + 2] * dl[2];
        v[a] = G.W[3 * a] * R.d[0] + G.W[3 * a + 1] * R.d[1] + G.W[3 * a + 2] * R.d[2];
    }
    const float A = v[0] * v[0] + v[1] * v[1] + v[2] * v[2];
    const float B = u[0] * v[0] + u[1] * v[1] + u[2] * v[2];
    r = __builtin_amdgcn_rsqf(A);
    const float tB = B * (r * r);
    const float p0 = fmaf(-tB, v[0], u[0]), p1 = fmaf(-tB, v[1], u[1]), p2 = fmaf(-tB, v[2], u[2]);
    D = p0 * p0 + p1 * p1 + p2 * p2;
}

// leaf_forward in the FP32 precision mode (compact records, two per step).
template <bool kStats, class At>
__device__ inline void leaf_forward32(const SceneView &S, const Ray &R, float inv_dd, uint64_t mask, At &&at,
                                      float k2, double &acc, uint32_t &n_inc, uint32_t &n_hitc) {
    while (mask) {
        const int j0 = __builtin_ctzll(mask);
        mask &= mask - 1;
        const bool two = mask != 0;
        const int j1 = two ? __builtin_ctzll(mask) : j0;
        if (two) mask &= mask - 1;
        const GaussRec32 *rec32 = rec32_of(S);
        const GaussRec32 G0 = sload(rec32, at(j0));
        const GaussRec32 G1 = sload(rec32, at(j1));
        float D, r;
        pair_core32(G0, R, inv_dd, D, r);
        if (kStats) n_hitc += ballot(D <= k2) != 0 ? 1u : 0u;
        if (D <= k2) {
            acc += double(G0.rho_c * r * gauss_exp(D));
            if (kStats) ++n_inc;
        }
        if (two) {
            pair_core32(G1, R, inv_dd, D, r);
            if (kStats) n_hitc += ballot(D <= k2) != 0 ? 1u : 0u;
            if (D <= k2) {
                acc += double(G1.rho_c * r * gauss_exp(D));
                if (kStats) ++n_inc;
            }
        }
    }
}

// One packet of the forward pass. kStats adds work counters (atomics once per
// packet) for measurement runs; the production instantiation has none.
// kCompact selects the FP32 precision mode. With kTeam the workgroup's waves
// take one part of the leaves each and meet in `team`.
//
// Where a wave has few leaves, its own can hold a multiple of another's
// candidates, and the packet waits for it: then the waves list their candidates
// and evaluate the packet's in equal shares, in an order that does not depend on
// timing. With many leaves per wave the shares are even by themselves and only
// the phases' barriers are felt, likewise for a packet of several runs. Measured,
// own leaves / shared, us: 3,001 Gaussians, one view of 64 x 64 29.2 / 23.4, of
// 61 x 47 (several runs) 47.4 / 52.0; 5,000, 64 packets 39.7 / 33.1, 1,024 64.4 /
// 53.4; 20,000, six views of 200 x 152 (8 parts) 168 / 157, 64 packets (16 parts)
// 73.7 / 76.3; 50,000, 256 packets 146 / 158.
constexpr int kTeamList = 512;  // candidates a wave lists; past it, it evaluates its own
inline bool share_candidates(int parts, int32_t n_leaves) { return n_leaves <= (parts == kMaxParts ? 128 : 512); }
struct TeamLds {
    double *sums;     // [waves][64]
    uint32_t *list;   // [waves][kTeamList]
    uint32_t *count;  // [waves]
};

template <bool kStats, bool kCompact, bool kTeam, bool kShare = false>
__device__ inline void packet_forward(const LaunchTable &T, int64_t packet, int lane, int wave, uint32_t *stack,
                                      const TeamLds &team, uint64_t *stats) {
    PacketRef P;
    if (!locate_packet(T, packet, lane, P)) return;
    const Segment &sg = T.segs[P.seg];
    const SceneView &S = T.scenes[sg.scene];
    float *out = sg.out;
    Ray R;
    load_ray(sg.ro, sg.rd, sg.stride, P.ray, R);
    double total = 0.0;
    uint32_t n_inc = 0, n_cand = 0, n_leaf = 0, n_hitc = 0;
    const float inv_dd = kCompact ? 1.0f / (R.d[0] * R.d[0] + R.d[1] * R.d[1] + R.d[2] * R.d[2]) : 0.0f;
    const Part part = kTeam ? Part{T.parts - 1, wave} : Part{0, 0};
    const uint64_t active = ballot(P.active);
    for_runs(S, R, active, lane, [&](bool in, const RunRay &Q, const Beam &B) {
        const bool share = kShare && ballot(in) == active;
        auto evaluate = [&](uint64_t mask, auto &&at) {
            if constexpr (kCompact)
                leaf_forward32<kStats>(S, R, inv_dd, mask, at, Q.cut, total, n_inc, n_hitc);
            else
                leaf_forward<kStats>(B.rec, Q, mask, at, total, n_inc, n_hitc);
        };
        int listed = 0;
        traverse_run(T.traversal, S, R, B, in, lane, stack, part, [&](int l) {
            int64_t start;
            const uint64_t mask = leaf_candidates(S, B, l, lane, start);
            if (kStats) {
                ++n_leaf;
                n_cand += __builtin_popcountll(mask);
            }
            const int nc = kShare ? __builtin_popcountll(mask) : 0;
            if (kShare && share && listed + nc <= kTeamList) {
                if ((mask >> lane) & 1ull)
                    team.list[wave * kTeamList + listed + __builtin_popcountll(mask & ((1ull << lane) - 1ull))] =
                        uint32_t(start + lane);
                listed += nc;
            } else {
                evaluate(mask, [&](int j) { return start + j; });
            }
        });
        if (kShare && share) {
            if (lane == 0) team.count[wave] = uint32_t(listed);
            __syncthreads();
            // candidate q of the run is this wave's when q mod parts is the wave
            const int cnt = lane < T.parts ? int(team.count[lane]) : 0;
            int upto = cnt;  // lane p: candidates listed by waves 0 .. p
            for (int o = 1; o < T.parts; o *= 2) {
                const int v = __shfl_up(upto, o, 64);
                if (lane >= o) upto += v;
            }
            const int all = __builtin_amdgcn_readlane(upto, T.parts - 1);
            for (int q0 = wave; q0 < all; q0 += 64 * T.parts) {
                const int q = q0 + lane * T.parts;
                const bool mine = q < all;
                int w = 0;  // the wave that listed q
                for (int p = 0; p < T.parts - 1; ++p) w += __builtin_amdgcn_readlane(upto, p) <= q;
                const int first = __shfl(upto - cnt, w, 64);
                const int idx = mine ? int(team.list[w * kTeamList + q - first]) : 0;
                evaluate(ballot(mine), [&](int j) { return int64_t(__builtin_amdgcn_readlane(idx, j)); });
            }
            __syncthreads();  // the lists are read
        }
    });
    if (kTeam) {
        team.sums[wave * 64 + lane] = total;
        __syncthreads();
        if (wave != 0) return;
        for (int k = 1; k < T.parts; ++k) total += team.sums[k * 64 + lane];
    }
    if (P.active) out[P.out] = float(total);
    if (kStats) {
        const float inc = wave_sum(float(n_inc));
        const uint64_t act = ballot(P.active);
        if (lane == 0) {
            atomicAdd(reinterpret_cast<unsigned long long *>(&stats[0]), (unsigned long long)(inc));
            atomicAdd(reinterpret_cast<unsigned long long *>(&stats[1]),
                      (unsigned long long)(n_cand) * (unsigned long long)(__builtin_popcountll(act)));
            atomicAdd(reinterpret_cast<unsigned long long *>(&stats[2]), (unsigned long long)(n_leaf));
            atomicAdd(reinterpret_cast<unsigned long long *>(&stats[3]), 1ull);
            atomicAdd(reinterpret_cast<unsigned long long *>(&stats[4]), (unsigned long long)(n_cand));
            atomicAdd(reinterpret_cast<unsigned long long *>(&stats[5]), (unsigned long long)(n_hitc));
        }
    }
}

// 8 waves per SIMD (at most 64 VGPRs; the traversal state spills a few
// registers, the pair loop none): the forward waits on its records' loads,
// and more waves hide that latency (16 views of 512 x 512 on 500,000
// Gaussians: 7.85 ms at 8 waves, 8.02 at 7, 8.50 at 6). Bound by VALU issue (0.9
// of the slots there; 36.6 instructions per candidate of which 21 are FP64, at
// 0.38 of the lanes inside the cutoff): 9.28 ms -> 7.81 with runs, beams and
// records along the run's axis in place of the general frame.
template <bool kStats, bool kCompact>
__global__ __launch_bounds__(1024) __attribute__((amdgpu_waves_per_eu(8))) void k_forward(
    LaunchTable T, uint64_t *stats) {
    extern __shared__ uint32_t fwd_stack[];  // kWideStack entries per wave
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(int(threadIdx.x >> 6));
    uint32_t *stack = fwd_stack + wave * kWideStack;
    // persistent: waves pull packets until the table is exhausted
    const bool pull = T.work_counter != nullptr;
    int64_t packet = pull ? next_packet(T.work_counter, lane) : logical_block(T.xcd_remap) * T.waves_per_group + wave;
    while (packet < T.n_packets) {
        packet_forward<kStats, kCompact, false>(T, packet, lane, 0, stack, TeamLds{}, stats);
        packet = pull ? next_packet(T.work_counter, lane) : T.n_packets;
    }
}

// The forward of a launch of few packets: one workgroup per packet, one wave
// per part.
template <bool kCompact, bool kShare>
__global__ __launch_bounds__(1024) void k_forward_team(LaunchTable T) {
    extern __shared__ __align__(16) unsigned char team_lds[];  // per wave 64 sums, kWideStack entries, kTeamList, a count
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(int(threadIdx.x >> 6));
    TeamLds team;
    team.sums = reinterpret_cast<double *>(team_lds);
    uint32_t *stacks = reinterpret_cast<uint32_t *>(team.sums + 64 * T.waves_per_group);
    team.list = stacks + kWideStack * T.waves_per_group;
    team.count = team.list + kTeamList * T.waves_per_group;
    packet_forward<false, kCompact, true, kShare>(T, logical_block(T.xcd_remap), lane, wave, stacks + wave * kWideStack, team,
                                          nullptr);
}

// A ray as its lane holds it for the replay of its run: the line across the
// run's axis and the weight dL/dI over |dk|, which makes the direction (S1, S2, 1).
struct ReplayRay {
    double X1, X2, S1, S2;
    float w;
};

// Ray i from the lane that holds it (ds_bpermute; every lane of the wave must
// execute this). i is per lane.
__device__ inline ReplayRay gather_ray(const ReplayRay &mine, int i) {
    const int a = i << 2;
    ReplayRay r;
    r.X1 = gather_f64(mine.X1, a);
    r.X2 = gather_f64(mine.X2, a);
    r.S1 = gather_f64(mine.S1, a);
    r.S2 = gather_f64(mine.S2, a);
    r.w = __builtin_bit_cast(float, __builtin_amdgcn_ds_bpermute(a, __builtin_bit_cast(int, mine.w)));
    return r;
}

// The replay of a recorded list takes windows of 64 entries: 8.5 KB per wave,
// so the 160 KB of a compute unit hold 18 waves' windows, against the 20 that
// the fused kernel's registers allow. During a re-traversal the traversal
// stack is live as well: 48 entries and the stack take 7.6 KB.
constexpr int kListWin = 64, kTravWin = 48, kGroup = 2;

struct TravLds {
    HitWindow<kTravWin> win;
    uint32_t stack[kWideStack];
};

// Per-wave LDS of the backward kernels.
union WaveLds {
    TravLds t;
    HitWindow<kListWin> win;  // hit-list replay (the traversal is over by then)
};

// Gradient terms of one included (ray, Gaussian) pair added to the ten sums
// c = (sum w E, sum wT p, sum of the symmetric wT (p p^T + d d^T / A)), E the
// unit-density integral sqrt(2 pi / A) exp(-D/2), T = rho E, and p the line's
// closest point to the mean in the metric P. Vectors are in the record's
// whitened frame (a, b, u) (AxisRec): the offset is (a, b, 0), the direction
// (c, d, 1), p = (a + t c, b + t d, t) with t = -B/A, and D = |p|^2 there. The
// whitened sums round with each axis' own size, so a flat Gaussian's short
// axis keeps its digits; unwhiten_sums maps them to coordinates per window.
__device__ inline void pair_grad(const AxisRec &G, float rho, float h, const ReplayRay &R, int, float c[10]) {
    const double e1 = fma(G.mk, R.S1, R.X1 - G.m1), e2 = fma(G.mk, R.S2, R.X2 - G.m2);
    const double g1 = R.S1 - G.s1, g2 = R.S2 - G.s2;
    const double a = fma(G.l21, e2, G.l11 * e1), b = G.l22 * e2;
    const double cc = fma(G.l21, g2, G.l11 * g1), dd = G.l22 * g2;
    const double A = fma(dd, dd, fma(cc, cc, G.h));
    const float r = __builtin_amdgcn_rsqf(float(A));
    // 1/A from the FP32 r^2 (relative error ~1e-7) and one Newton step
    double ra = double(r * r);
    ra = fma(ra, fma(-A, ra, 1.0), ra);
    const double t = -fma(a, cc, b * dd) * ra;
    const float p0 = float(fma(t, cc, a)), p1 = float(fma(t, dd, b)), p2 = float(t);
    const float f0 = float(cc), f1 = float(dd);
    const float D = fmaf(p0, p0, fmaf(p1, p1, h * (p2 * p2)));
    const float wE = R.w * (kSqrt2Pi * r * gauss_exp(D));
    const float wT = wE * rho;
    const float wTA = wT * (r * r);
    const float q0 = wT * p0, q1 = wT * p1, q2 = wT * p2;
    const float v0 = wTA * f0, v1 = wTA * f1;
    c[0] += wE;
    c[1] += q0;
    c[2] += q1;
    c[3] += q2;
    c[4] = fmaf(q0, p0, fmaf(v0, f0, c[4]));
    c[5] = fmaf(q1, p1, fmaf(v1, f1, c[5]));
    c[6] = fmaf(q2, p2, wTA + c[6]);
    c[7] = fmaf(q0, p1, fmaf(v0, f1, c[7]));
    c[8] = fmaf(q0, p2, v0 + c[8]);
    c[9] = fmaf(q1, p2, v1 + c[9]);
}

// Hit list of one packet: (Gaussian, 64-bit mask of the packet's rays with
// D <= kappa^2) for every candidate with at least one such ray, recorded by
// the forward half of the fused pass into this wave's region of the caller's
// scratch (cap entries). Entries collect in registers (lane k holds the k-th
// pending one) and go out 64 at a time as coalesced stores. A packet with
// more than cap entries marks the list overflowed; its backward half then
// falls back to re-traversal.
struct HitList {
    uint32_t *g;
    uint64_t *m;
    int cap;
    int n;        // entries stored (wave-uniform)
    int nbuf;     // entries pending in registers (wave-uniform)
    bool overflow;
    uint32_t bg;  // lane i holds pending entry i: Gaussian index,
    uint32_t blo; // low and
    uint32_t bhi; // high half of its ray mask

    __device__ void flush(int lane) {
        if (nbuf == 0) return;
        if (n + nbuf <= cap) {
            if (lane < nbuf) {
                g[n + lane] = bg;
                m[n + lane] = (uint64_t(bhi) << 32) | blo;
            }
            n += nbuf;
        } else {
            overflow = true;
        }
        nbuf = 0;
    }
    // Appends (gi, mask); both are wave-uniform and mask is non-zero. The
    // entry goes into lane nbuf of the pending registers by lane writes.
    __device__ void record(int lane, int64_t gi, uint64_t mask) {
        if (overflow) return;
        bg = lane_write(int(uint32_t(gi)), nbuf, int(bg));
        blo = lane_write(int(uint32_t(mask)), nbuf, int(blo));
        bhi = lane_write(int(uint32_t(mask >> 32)), nbuf, int(bhi));
        if (++nbuf == 64) flush(lane);
    }
};

// Forward sum over one leaf's candidates (as leaf_forward), also recording the
// packet's hit list.
__device__ inline void leaf_forward_hits(const AxisRec *rec, const RunRay &Q, int64_t start, uint64_t mask,
                                         double &acc, HitList &H, int lane) {
    const float k2a = Q.cut;
    while (mask) {
        const int j0 = __builtin_ctzll(mask);
        mask &= mask - 1;
        const bool two = mask != 0;
        const int j1 = two ? __builtin_ctzll(mask) : j0;
        if (two) mask &= mask - 1;
        const AxisRec G0 = sload(rec, start + j0);
        const AxisRec G1 = sload(rec, start + j1);
        hold_records(G0, G1);
        AxisCore c;
        float D, r;
        axis_core(G0, Q, c);
        pair_D(c, D, r);
        const uint64_t h0 = __builtin_amdgcn_ballot_w64(D <= k2a);
        if (h0) {
            if (D <= k2a) {
                asm volatile("");  // keeps this a branch: if-converted, every lane pays for the exp
                acc += double(G0.rho_c * r * gauss_exp(D));
            }
            H.record(lane, start + j0, h0);
        }
        if (two) {
            axis_core(G1, Q, c);
            pair_D(c, D, r);
            const uint64_t h1 = __builtin_amdgcn_ballot_w64(D <= k2a);
            if (h1) {
                if (D <= k2a) {
                    asm volatile("");
                    acc += double(G1.rho_c * r * gauss_exp(D));
                }
                H.record(lane, start + j1, h1);
            }
        }
    }
}

// Backward half of a run from its recorded hit list, in windows; the next
// window's entries are loaded while the current one runs.
__device__ inline void drain_hits(const SceneView &S, const Beam &B, HitWindow<kListWin> &W, const ReplayRay &mine,
                                  const uint32_t *hg, const uint64_t *hm, int n_ent, uint64_t live, int lane,
                                  float *acc) {
    uint32_t pg = 0;
    uint64_t pm = 0;
    if (lane < min(kListWin, n_ent)) {
        pg = hg[lane];
        pm = hm[lane] & live;
    }
    for (int e0 = 0; e0 < n_ent; e0 += kListWin) {
        const int64_t gj = pg;
        const uint64_t mj = pm;
        const int e1 = e0 + kListWin;
        pm = 0;
        if (lane < min(kListWin, n_ent - e1)) {
            pg = hg[e1 + lane];
            pm = hm[e1 + lane] & live;
        }
        replay_window<kListWin, kGroup>(B.rec, B.ax, S.n, W, gj, mj, mine, lane, acc, pair_grad);
    }
}

// Per-ray loss weight dL/dI and loss term for the fused pass.
__device__ inline float loss_weight(int kind, float I, float y, float b, double &term) {
    if (kind == GR_LOSS_L2) {
        const float e = I - y;
        term = 0.5 * double(e) * double(e);
        return e;
    }
    const double Ib = double(I) + double(b);
    term = Ib - double(y) * log(Ib);
    return float(1.0 - double(y) / Ib);
}

// Backward of a run without a list (dL/dI given, or a list that outgrew its
// region): the traversal takes the cutoff test of every candidate on the run's
// weighted rays and collects the candidates that pass on any, one per lane;
// every full window is replayed on the spot. A Gaussian per lane looping over all
// rays, which it replaced, evaluated every candidate's gradient on every ray:
// 50k Gaussians, 10 views of 256 x 256, 1116 -> 1074 us.
__device__ inline void backward_by_windows(const LaunchTable &T, const SceneView &S, const Ray &R, const Beam &B,
                                           const RunRay &Q, const ReplayRay &mine, bool live, TravLds &L, int lane,
                                           Part part, float *acc) {
    const float cut = live ? S.kappa2 : -1.0f;
    int n = 0;  // pending entries (wave-uniform); lane q holds entry q
    uint32_t pg = 0, plo = 0, phi = 0;
    auto put = [&](int64_t g, uint64_t m) {
        pg = uint32_t(lane_write(int(uint32_t(g)), n, int(pg)));
        plo = uint32_t(lane_write(int(uint32_t(m)), n, int(plo)));
        phi = uint32_t(lane_write(int(uint32_t(m >> 32)), n, int(phi)));
        ++n;
    };
    auto replay = [&]() {
        const uint64_t m = lane < n ? (uint64_t(phi) << 32) | plo : 0ull;
        replay_window<kTravWin, kGroup>(B.rec, B.ax, S.n, L.win, pg, m, mine, lane, acc, pair_grad);
        n = 0;
    };
    traverse_run(T.traversal, S, R, B, live, lane, L.stack, part, [&](int l) {
        int64_t start;
        uint64_t mask = leaf_candidates(S, B, l, lane, start);
        while (mask) {
            const int j0 = __builtin_ctzll(mask);
            mask &= mask - 1;
            const bool two = mask != 0;
            const int j1 = two ? __builtin_ctzll(mask) : j0;
            if (two) mask &= mask - 1;
            const AxisRec G0 = sload(B.rec, start + j0);
            const AxisRec G1 = sload(B.rec, start + j1);
            hold_records(G0, G1);
            AxisCore c;
            float D, r;
            axis_core(G0, Q, c);
            pair_D(c, D, r);
            const uint64_t h0 = ballot(D <= cut);
            if (h0) put(start + j0, h0);
            if (two) {
                axis_core(G1, Q, c);
                pair_D(c, D, r);
                const uint64_t h1 = ballot(D <= cut);
                if (h1) put(start + j1, h1);
            }
            if (n > kTravWin - 2) replay();
        }
    });
    if (n > 0) replay();
}

// One packet of the backward, run by run (each ray is in one run, so its
// projection is complete when its run's traversal is). With kTeam the
// workgroup's waves take a part of the leaves each, meet in `sums` (64 per
// wave) for the projection, and replay the lists of their own parts. With dL/dI
// given the packet's parts are work items of their own.
template <bool kFused, bool kTeam>
__device__ inline void packet_backward(const LaunchTable &T, int64_t packet, int lane, int part, WaveLds *L,
                                       double *sums, const BwdArgs &A, uint32_t *hit_g, uint64_t *hit_m) {
    PacketRef P;
    if (!locate_packet(T, packet, lane, P)) return;
    const Segment &sg = T.segs[P.seg];
    const SceneView &S = T.scenes[sg.scene];
    float *acc = kFused ? sg.acc : A.acc;
    const int parts = kFused && !kTeam ? 1 : T.parts;
    const Part mine_only{parts - 1, part};
    const bool first = !kTeam || part == 0;
    Ray R;
    load_ray(sg.ro, sg.rd, sg.stride, P.ray, R);
    float w = 0.0f;  // dL/dI
    if (!kFused && P.active) w = A.grad_out[P.out];
    double term = 0.0;
    uint64_t todo = ballot(kFused ? P.active : P.active && w != 0.0f);
    const Extent E = scene_extent(S);
    while (todo) {
        const uint64_t before = todo;
        Beam B;
        RunRay Q;
        const uint64_t run = S.n > 0 ? next_run(E, R, todo, lane, B, Q) : (todo = 0);
        const bool in = ((before & ~todo) >> lane) & 1ull;  // the run's rays, or one that is no line
        Q.cut = in && run ? S.kappa2 : -1.0f;
        B.rec = axis_rec_of(S, B.ax);
        HitList H{hit_g, hit_m, T.hit_cap, 0, 0, !hit_g, 0u, 0u, 0u};
        if (kFused) {
            double total = 0.0;
            if (run)
                traverse_run(T.traversal, S, R, B, in, lane, L->t.stack, mine_only, [&](int l) {
                    int64_t start;
                    const uint64_t mask = leaf_candidates(S, B, l, lane, start);
                    leaf_forward_hits(B.rec, Q, start, mask, total, H, lane);
                });
            if (kTeam) {
                // (all waves of the workgroup take the same runs)
                __syncthreads();  // the last run's sums are read
                sums[part * 64 + lane] = total;
                __syncthreads();
                total = sums[lane];
                for (int p = 1; p < parts; ++p) total += sums[p * 64 + lane];
            }
            if (in) {
                const float I = float(total);
                double t;
                w = loss_weight(sg.loss_kind, I, sg.target[P.out], sg.background, t);
                term += t;
                if (first && sg.out) sg.out[P.out] = I;
            }
        }
        const bool live = in && w != 0.0f;
        const uint64_t live_mask = ballot(live);
        if (!run || !live_mask) continue;
        const ReplayRay mine{Q.X1, Q.X2, Q.S1, Q.S2, live ? w / fabsf(float(Q.dk)) : 0.0f};
        if (kFused) {
            H.flush(lane);
            if (!H.overflow) {
                // the list's global stores (other lanes' entries) are visible to
                // this wave's loads after a workgroup-scope release/acquire
                __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");
                __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup");
                drain_hits(S, B, L->win, mine, hit_g, hit_m, H.n, live_mask, lane, acc);
                continue;
            }
        }
        backward_by_windows(T, S, R, B, Q, mine, live, L->t, lane, mine_only, acc);
    }
    if (kFused && first && sg.loss) {
        for (int off = 32; off >= 1; off >>= 1) term += __shfl_xor(term, off);
        if (lane == 0) atomicAdd(sg.loss, term);
    }
}

// 5 waves per SIMD (at most 96 VGPRs; some spill, outside the pair loops): the
// forward half of the fused pass waits on its records' loads, and the extra
// wave hides part of that latency (persistent launches default to 20 waves per
// compute unit to match; LDS holds 18 windows per compute unit, and later
// workgroups start as earlier ones finish). Bound by VALU issue (0.82-0.86 of the
// slots): 24 views of 512 x 512 on 500,000 Gaussians 29.6 -> 24.7 ms with the
// axis records and the whitened replay (4 / 6 waves 26.2 / 26.0 against 25.75 on
// the way there), dL/dI given 1160 -> 884 us on 50,000 Gaussians x
// 10 views of 256 x 256.
template <bool kFused>
__global__ __launch_bounds__(1024) __attribute__((amdgpu_waves_per_eu(5))) void k_backward(LaunchTable T, BwdArgs A) {
    extern __shared__ __align__(16) unsigned char lds_raw[];
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(int(threadIdx.x >> 6));
    WaveLds *L = reinterpret_cast<WaveLds *>(lds_raw + (kFused ? sizeof(WaveLds) : sizeof(TravLds)) * wave);
    const bool pull = T.work_counter != nullptr;
    // hit-list regions belong to persistent waves (one per wave slot)
    const int64_t slot = int64_t(blockIdx.x) * T.waves_per_group + wave;
    const bool lists = pull && T.hit_cap > 0;
    uint32_t *hg = lists ? T.hit_g + slot * T.hit_cap : nullptr;
    uint64_t *hm = lists ? T.hit_m + slot * T.hit_cap : nullptr;
    // with dL/dI given, a packet's parts are work items of their own
    const int parts = kFused ? 1 : T.parts;
    const int64_t n_items = T.n_packets * parts;
    int64_t item = pull ? next_packet(T.work_counter, lane) : logical_block(T.xcd_remap) * T.waves_per_group + wave;
    while (item < n_items) {
        const int64_t packet = kFused ? item : item / parts;
        packet_backward<kFused, false>(T, packet, lane, int(item - packet * parts), L, nullptr, A, hg, hm);
        item = pull ? next_packet(T.work_counter, lane) : n_items;
    }
}

// The fused pass of a launch of few packets: workgroups take packets, their
// waves one part each (with hit lists, so always persistent). Bound by the longest
// packet's chain until the chip is full: a step of 2,048 packets on 512 Gaussians,
// with its build, 239 -> 197 us.
__global__ __launch_bounds__(1024) __attribute__((amdgpu_waves_per_eu(4))) void k_backward_team(LaunchTable T) {
    extern __shared__ __align__(16) unsigned char lds_raw[];
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(int(threadIdx.x >> 6));
    WaveLds *L = reinterpret_cast<WaveLds *>(lds_raw) + wave;
    double *sums = reinterpret_cast<double *>(lds_raw + sizeof(WaveLds) * T.waves_per_group);
    uint32_t *ticket = reinterpret_cast<uint32_t *>(sums + 64 * T.waves_per_group);
    const int64_t slot = int64_t(blockIdx.x) * T.waves_per_group + wave;
    const BwdArgs none{nullptr, nullptr};
    for (;;) {
        if (threadIdx.x == 0) *ticket = atomicAdd(T.work_counter, 1u);
        __syncthreads();
        const int64_t packet = int64_t(uint32_t(__builtin_amdgcn_readfirstlane(int(*ticket))));
        if (packet >= T.n_packets) return;
        packet_backward<true, true>(T, packet, lane, wave, L, sums, none, T.hit_g + slot * T.hit_cap,
                                    T.hit_m + slot * T.hit_cap);
        __syncthreads();  // the ticket and the sums are read
    }
}

// Zero the accumulators, and a launch's ticket counter with them (a fill
// kernel, so the call stays capturable).
__global__ void k_zero_f32(float *p, int64_t count, uint32_t *counter) {
    const int64_t i = int64_t(blockIdx.x) * blockDim.x + threadIdx.x;
    if (i < count) p[i] = 0.0f;
    if (counter && i == 0) *counter = 0u;
}

// Chain rule from the per-Gaussian sums (g_rho, m, M) to the raw
// parameters. P = R L R^T with L = diag(s^-2): dL/dmu = P m,
// dL/dP = -M/2, so dL/ds_k = (r_k^T M r_k) / s_k^3 (r_k the k-th column of R)
// and dL/dR = -M R L. R(q) = (1 - 2|v|^2) I + 2 w [v]x + 2 v v^T for
// q = (w, v); for G = dL/dR:  dL/dw = 2 v . ax(G) and
// dL/dv = -4 tr(G) v + 2 w ax(G) + 2 (G + G^T) v, with
// ax(G) = (G21 - G12, G02 - G20, G10 - G01); finally the projection through
// q/|q|: dL/dq = (g - qh (qh . g)) / |q|.
__global__ __launch_bounds__(256) void k_epilogue(const float *__restrict__ mean,
                                                  const float *__restrict__ scale,
                                                  const float *__restrict__ quat,
                                                  const float *__restrict__ dens, int64_t n,
                                                  const uint32_t *__restrict__ order,
                                                  const float *__restrict__ acc, float *gmean,
                                                  float *gscale, float *gquat, float *gdens) {
    const int64_t g = int64_t(blockIdx.x) * blockDim.x + threadIdx.x;
    if (g >= n) return;
    const int64_t i = order[g];
    if (i >= n) return;
    double s[3], q[4], qq = 0.0;
    bool ok = isfinite(mean[i]) && isfinite(mean[n + i]) && isfinite(mean[2 * n + i]) &&
              isfinite(dens[i]);
    for (int k = 0; k < 3; ++k) {
        s[k] = scale[k * n + i];
        ok = ok && isfinite(s[k]) && s[k] > 0.0;
    }
    for (int k = 0; k < 4; ++k) {
        q[k] = quat[k * n + i];
        ok = ok && isfinite(q[k]);
        qq += q[k] * q[k];
    }
    ok = ok && qq > 0.0;
    if (!ok) {
        for (int k = 0; k < 3; ++k) gmean[k * n + i] = 0.0f, gscale[k * n + i] = 0.0f;
        for (int k = 0; k < 4; ++k) gquat[k * n + i] = 0.0f;
        gdens[i] = 0.0f;
        return;
    }
    double a[10];
    for (int k = 0; k < 10; ++k) a[k] = acc[k * n + g];
    const double qn = sqrt(qq);
    const double w = q[0] / qn, v[3] = {q[1] / qn, q[2] / qn, q[3] / qn};
    const double vv = v[0] * v[0] + v[1] * v[1] + v[2] * v[2];
    double R[3][3];
    const double cx[3][3] = {{0.0, -v[2], v[1]}, {v[2], 0.0, -v[0]}, {-v[1], v[0], 0.0}};
    for (int r = 0; r < 3; ++r)
        for (int c = 0; c < 3; ++c)
            R[r][c] = (r == c ? 1.0 - 2.0 * vv : 0.0) + 2.0 * w * cx[r][c] + 2.0 * v[r] * v[c];
    const double lam[3] = {1.0 / (s[0] * s[0]), 1.0 / (s[1] * s[1]), 1.0 / (s[2] * s[2])};
    const double m[3] = {a[1], a[2], a[3]};
    const double M[3][3] = {{a[4], a[7], a[8]}, {a[7], a[5], a[9]}, {a[8], a[9], a[6]}};
    // dL/dmu = P m = R L R^T m
    double Rtm[3];
    for (int k = 0; k < 3; ++k) Rtm[k] = lam[k] * (R[0][k] * m[0] + R[1][k] * m[1] + R[2][k] * m[2]);
    for (int r = 0; r < 3; ++r) gmean[r * n + i] = float(R[r][0] * Rtm[0] + R[r][1] * Rtm[1] + R[r][2] * Rtm[2]);
    // M R (columns), then dL/ds and dL/dR
    double MR[3][3];
    for (int r = 0; r < 3; ++r)
        for (int c = 0; c < 3; ++c) MR[r][c] = M[r][0] * R[0][c] + M[r][1] * R[1][c] + M[r][2] * R[2][c];
    for (int k = 0; k < 3; ++k) {
        const double rMr = R[0][k] * MR[0][k] + R[1][k] * MR[1][k] + R[2][k] * MR[2][k];
        gscale[k * n + i] = float(rMr / (s[k] * s[k] * s[k]));
    }
    double G[3][3];
    for (int r = 0; r < 3; ++r)
        for (int c = 0; c < 3; ++c) G[r][c] = -MR[r][c] * lam[c];
    const double axg[3] = {G[2][1] - G[1][2], G[0][2] - G[2][0], G[1][0] - G[0][1]};
    const double tr = G[0][0] + G[1][1] + G[2][2];
    double gq[4];
    gq[0] = 2.0 * (v[0] * axg[0] + v[1] * axg[1] + v[2] * axg[2]);
    for (int k = 0; k < 3; ++k) {
        const double Gv = G[k][0] * v[0] + G[k][1] * v[1] + G[k][2] * v[2];
        const double GTv = G[0][k] * v[0] + G[1][k] * v[1] + G[2][k] * v[2];
        gq[1 + k] = -4.0 * tr * v[k] + 2.0 * w * axg[k] + 2.0 * (Gv + GTv);
    }
    const double qh[4] = {w, v[0], v[1], v[2]};
    const double dot = gq[0] * qh[0] + gq[1] * qh[1] + gq[2] * qh[2] + gq[3] * qh[3];
    for (int k = 0; k < 4; ++k) gquat[k * n + i] = float((gq[k] - qh[k] * dot) / qn);
    gdens[i] = float(a[0]);
}

// ---------------------------------------------------------------------------
// host drivers
// ---------------------------------------------------------------------------

__global__ void k_zero_u32(uint32_t *p) {
    if (threadIdx.x == 0 && blockIdx.x == 0) *p = 0u;
}

hipError_t enqueue_forward(LaunchTable &T, const LaunchShape &shape, hipStream_t st, uint64_t *stats) {
    finish_table(T, shape);
    if (T.n_packets == 0) return hipSuccess;
    if (shape.work_counter) k_zero_u32<<<1, 64, 0, st>>>(shape.work_counter);
    const int team = T.parts;
    if (team > 1 && shape.free_waves && !shape.work_counter && !stats) {
        T.waves_per_group = team;
        const bool share = share_candidates(team, most_leaves(T));
        const size_t lds = (sizeof(double) * 64 + sizeof(uint32_t) * (kWideStack + (share ? kTeamList + 1 : 0))) * size_t(team);
        auto kernel = T.precision == 1 ? (share ? k_forward_team<true, true> : k_forward_team<true, false>)
                                       : (share ? k_forward_team<false, true> : k_forward_team<false, false>);
        kernel<<<dim3(unsigned(T.n_packets)), dim3(64 * team), lds, st>>>(T);
        return hipGetLastError();
    }
    const unsigned groups = launch_groups(T.n_packets, shape);
    const int waves = shape.waves;
    const size_t lds = T.traversal == 1 ? 0 : sizeof(uint32_t) * kWideStack * size_t(waves);
    if (T.precision == 1) {
        if (stats)
            k_forward<true, true><<<dim3(groups), dim3(64 * waves), lds, st>>>(T, stats);
        else
            k_forward<false, true><<<dim3(groups), dim3(64 * waves), lds, st>>>(T, nullptr);
    } else {
        if (stats)
            k_forward<true, false><<<dim3(groups), dim3(64 * waves), lds, st>>>(T, stats);
        else
            k_forward<false, false><<<dim3(groups), dim3(64 * waves), lds, st>>>(T, nullptr);
    }
    return hipGetLastError();
}

// (the caller has zeroed the work counter)
static void launch_backward(LaunchTable &T, const BwdArgs &A, const LaunchShape &shape, uint32_t *hit_g,
                            uint64_t *hit_m, hipStream_t st) {
    finish_table(T, shape);
    const bool lists = !A.grad_out && shape.work_counter && shape.hit_cap > 0 && hit_g && hit_m;
    T.hit_cap = lists ? shape.hit_cap : 0;
    T.hit_g = lists ? hit_g : nullptr;
    T.hit_m = lists ? hit_m : nullptr;
    if (T.n_packets == 0) return;
    const int team = T.parts;
    if (team > 1 && lists && shape.free_groups) {
        // as many waves as the lists' regions were sized for
        T.waves_per_group = team;
        const unsigned groups = unsigned(std::min<int64_t>(T.n_packets, shape.persistent_groups / team));
        const size_t lds = (sizeof(WaveLds) + sizeof(double) * 64) * size_t(team) + 16;
        k_backward_team<<<dim3(groups), dim3(64 * team), lds, st>>>(T);
        return;
    }
    const unsigned groups = launch_groups(A.grad_out ? T.n_packets * T.parts : T.n_packets, shape);
    const int waves = shape.waves;
    if (A.grad_out)
        k_backward<false><<<dim3(groups), dim3(64 * waves), sizeof(TravLds) * size_t(waves), st>>>(T, A);
    else
        k_backward<true><<<dim3(groups), dim3(64 * waves), sizeof(WaveLds) * size_t(waves), st>>>(T, A);
}

hipError_t enqueue_backward(LaunchTable &T, const BwdArgs &A, const gr_scene &sc, const uint32_t *order,
                            float *gmean, float *gscale, float *gquat, float *gdens,
                            const LaunchShape &shape, uint32_t *hit_g, uint64_t *hit_m,
                            hipStream_t st) {
    if (sc.n > 0)
        enqueue_zero_f32(A.acc, 10 * sc.n, st, shape.work_counter);
    else if (shape.work_counter)
        enqueue_zero_u32(shape.work_counter, st);
    launch_backward(T, A, shape, hit_g, hit_m, st);
    enqueue_epilogue(sc, order, A.acc, gmean, gscale, gquat, gdens, st);
    return hipGetLastError();
}

hipError_t enqueue_fused_segments(LaunchTable &T, const LaunchShape &shape, uint32_t *hit_g, uint64_t *hit_m,
                                  hipStream_t st) {
    BwdArgs A{nullptr, nullptr};
    if (shape.work_counter) enqueue_zero_u32(shape.work_counter, st);
    launch_backward(T, A, shape, hit_g, hit_m, st);
    return hipGetLastError();
}

void enqueue_zero_u32(uint32_t *p, hipStream_t st) { k_zero_u32<<<1, 64, 0, st>>>(p); }

void enqueue_zero_f32(float *p, int64_t count, hipStream_t st, uint32_t *counter) {
    if (count > 0) k_zero_f32<<<unsigned((count + 255) / 256), 256, 0, st>>>(p, count, counter);
}

void enqueue_epilogue(const gr_scene &sc, const uint32_t *order, const float *acc, float *gmean, float *gscale,
                      float *gquat, float *gdens, hipStream_t st) {
    const int64_t n = sc.n;
    if (n > 0)
        k_epilogue<<<unsigned((n + 255) / 256), 256, 0, st>>>(sc.mean, sc.scale, sc.quat, sc.density, n, order,
                                                              acc, gmean, gscale, gquat, gdens);
}

}  // namespace gr
