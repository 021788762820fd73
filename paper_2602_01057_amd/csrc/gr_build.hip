// Acceleration-structure build: per-Gaussian preprocessing, Morton codes,
// counting or stable LSD radix sort, records and leaf boxes, the wide hierarchy, Karras
// radix-tree LBVH over leaves of L Gaussians. Everything runs on one stream with
// no host round trip.
//
// A build is a chain of short kernels, so it is bound by their number and by
// each one's longest dependent chain, not by bandwidth (500k Gaussians move
// about 0.25 GB, 50 us): up to 12,288 Gaussians are coded and sorted in one
// launch, the boxes of the leaves come out of the record kernel's LDS, the
// upper levels of the hierarchy are one launch, and a binary node's boxes are
// read off the hierarchy's levels by a wave of its own instead of climbing the
// tree leaf by leaf with atomics.
//
// Geometry of one Gaussian (Sec. 3.1, Eq. 2): Sigma = R S S^T R^T with R the
// rotation of the unit quaternion and S = diag(s). Its kappa-sigma ellipsoid
// {x : (x-mu)^T Sigma^-1 (x-mu) <= kappa^2} has axis-aligned half extents
// kappa sqrt(Sigma_jj) and support width kappa sqrt(e^T Sigma e) along any e.
#include <float.h>
#include <math.h>

#include "gr_trace.h"

namespace gr {

namespace {

// Margins that keep the FP32 box and slab tests conservative for lines that
// meet the kappa ellipsoid (absolute part in the scene's length unit, mm).
constexpr float kBoxRel = 1.0f / 65536.0f;
constexpr float kBoxAbs = 1e-3f;

__device__ inline bool load_params(const float *__restrict__ mean, const float *__restrict__ scale,
                                   const float *__restrict__ quat, const float *__restrict__ dens,
                                   int64_t n, int64_t i, double mu[3], double s[3], double q[4],
                                   double &rho) {
    bool ok = true;
    for (int k = 0; k < 3; ++k) {
        mu[k] = mean[k * n + i];
        s[k] = scale[k * n + i];
        ok = ok && isfinite(mu[k]) && isfinite(s[k]) && s[k] > 0.0;
    }
    double qq = 0.0;
    for (int k = 0; k < 4; ++k) {
        q[k] = quat[k * n + i];
        ok = ok && isfinite(q[k]);
        qq += q[k] * q[k];
    }
    rho = dens[i];
    ok = ok && isfinite(rho) && qq > 0.0;
    if (ok) {
        const double inv = 1.0 / sqrt(qq);
        for (int k = 0; k < 4; ++k) q[k] *= inv;
    }
    return ok;
}

// Rotation of a unit quaternion (w, v): R = I + 2 w [v]x + 2 [v]x^2, with
// [v]x^2 = v v^T - |v|^2 I. Columns are the local axes in world coordinates.
__device__ inline void rotation(const double q[4], double R[3][3]) {
    const double w = q[0], v[3] = {q[1], q[2], q[3]};
    const double vv = v[0] * v[0] + v[1] * v[1] + v[2] * v[2];
    const double cx[3][3] = {{0.0, -v[2], v[1]}, {v[2], 0.0, -v[0]}, {-v[1], v[0], 0.0}};
    for (int a = 0; a < 3; ++a)
        for (int b = 0; b < 3; ++b)
            R[a][b] = (a == b ? 1.0 - 2.0 * vv : 0.0) + 2.0 * w * cx[a][b] + 2.0 * v[a] * v[b];
}

__device__ inline uint32_t spread10(uint32_t v) {
    v &= 1023u;
    v = (v | (v << 16)) & 0x030000FFu;
    v = (v | (v << 8)) & 0x0300F00Fu;
    v = (v | (v << 4)) & 0x030C30C3u;
    v = (v | (v << 2)) & 0x09249249u;
    return v;
}

}  // namespace

// ---------------------------------------------------------------------------
// header and bounds
// ---------------------------------------------------------------------------

// Bounds of the valid means (order-preserving encodings) and the number of
// invalid Gaussians.
struct Bounds {
    uint32_t lo[3], hi[3], bad, pad;
};

__device__ inline void bounds_empty(Bounds &b) {
    for (int k = 0; k < 3; ++k) {
        b.lo[k] = 0xFFFFFFFFu;
        b.hi[k] = 0u;
    }
    b.bad = 0;
    b.pad = 0;
}

__device__ inline void bounds_join(Bounds &b, const Bounds &o) {
    for (int k = 0; k < 3; ++k) {
        b.lo[k] = min(b.lo[k], o.lo[k]);
        b.hi[k] = max(b.hi[k], o.hi[k]);
    }
    b.bad += o.bad;
}

// Joins the workgroup's bounds (all threads get the result).
__device__ inline void bounds_of_block(Bounds &b, Bounds *lds) {
    for (int off = 32; off >= 1; off >>= 1) {
        Bounds o;
        for (int k = 0; k < 3; ++k) {
            o.lo[k] = __shfl_xor(b.lo[k], off);
            o.hi[k] = __shfl_xor(b.hi[k], off);
        }
        o.bad = __shfl_xor(b.bad, off);
        bounds_join(b, o);
    }
    const int wave = threadIdx.x >> 6, waves = blockDim.x >> 6;
    if ((threadIdx.x & 63) == 0) lds[wave] = b;
    __syncthreads();
    bounds_empty(b);
    for (int w = 0; w < waves; ++w) bounds_join(b, lds[w]);
    __syncthreads();
}

__device__ inline void bounds_add(Bounds &b, const float *__restrict__ mean, const float *__restrict__ scale,
                                  const float *__restrict__ quat, const float *__restrict__ dens, int64_t n,
                                  int64_t i) {
    double mu[3], s[3], q[4], rho;
    if (load_params(mean, scale, quat, dens, n, i, mu, s, q, rho)) {
        for (int k = 0; k < 3; ++k) {
            const uint32_t u = f2ord(float(mu[k]));
            b.lo[k] = min(b.lo[k], u);
            b.hi[k] = max(b.hi[k], u);
        }
    } else {
        ++b.bad;
    }
}

__device__ inline void write_header(AccelHeader *hdr, int64_t n, int32_t leaf, int32_t n_leaves, float kappa,
                                    const Bounds &b) {
    hdr->magic = kMagic;
    hdr->built = 0;
    hdr->n = n;
    hdr->leaf_size = leaf;
    hdr->n_leaves = n_leaves;
    hdr->kappa = kappa;
    hdr->n_invalid = int32_t(b.bad);
    for (int k = 0; k < 3; ++k) {
        hdr->bmin[k] = b.lo[k];
        hdr->bmax[k] = b.hi[k];
        hdr->root_box[k] = FLT_MAX;
        hdr->root_box[3 + k] = -FLT_MAX;
    }
    hdr->root = n_leaves > 1 ? 0 : ~0;
    hdr->flags = 0;
}

__global__ void k_build_empty(AccelHeader *hdr, int32_t leaf, int32_t n_leaves, float kappa) {
    if (threadIdx.x != 0 || blockIdx.x != 0) return;
    Bounds b;
    bounds_empty(b);
    write_header(hdr, 0, leaf, n_leaves, kappa, b);
    hdr->built = 1;
}

// Refit: keep the Morton order and the tree of the last build, reset what the
// refit recomputes (invalid count, root box, flags). A workspace that
// was not built for this n and leaf size is flagged; the kernels that follow
// only follow indices they check, so the refit stays memory-safe.
__global__ void k_refit_init(AccelHeader *hdr, int64_t n, int32_t leaf, int32_t n_leaves, float kappa) {
    if (threadIdx.x != 0 || blockIdx.x != 0) return;
    int32_t flags = 0;
    if (hdr->magic != kMagic || hdr->built != 1 || hdr->n != n || hdr->leaf_size != leaf ||
        hdr->n_leaves != n_leaves)
        flags = kFlagNotBuilt;
    hdr->magic = kMagic;
    hdr->built = n > 0 ? 0 : 1;
    hdr->n = n;
    hdr->leaf_size = leaf;
    hdr->n_leaves = n_leaves;
    hdr->kappa = kappa;
    hdr->n_invalid = 0;
    for (int k = 0; k < 3; ++k) {
        hdr->root_box[k] = FLT_MAX;
        hdr->root_box[3 + k] = -FLT_MAX;
    }
    if (flags) hdr->root = n_leaves > 1 ? 0 : ~0;
    hdr->flags = flags;
}

// Bounds of each of at most kBoundsBlocks blocks' Gaussians.
__global__ __launch_bounds__(256) void k_bounds(const float *__restrict__ mean,
                                                const float *__restrict__ scale,
                                                const float *__restrict__ quat,
                                                const float *__restrict__ dens, int64_t n,
                                                Bounds *__restrict__ part) {
    __shared__ Bounds lds[4];
    Bounds b;
    bounds_empty(b);
    for (int64_t i = int64_t(blockIdx.x) * 256 + threadIdx.x; i < n; i += int64_t(gridDim.x) * 256)
        bounds_add(b, mean, scale, quat, dens, n, i);
    bounds_of_block(b, lds);
    if (threadIdx.x == 0) part[blockIdx.x] = b;
}

// Morton code of a valid mean inside the bounds.
__device__ inline uint32_t mean_code(const float mu[3], const Bounds &b) {
    uint32_t code = 0;
    for (int k = 0; k < 3; ++k) {
        float lo = ord2f(b.lo[k]), hi = ord2f(b.hi[k]);
        if (!(hi > lo)) hi = lo + 1.0f;
        float t = (mu[k] - lo) / (hi - lo);
        int c = int(t * 1024.0f);
        c = c < 0 ? 0 : (c > 1023 ? 1023 : c);
        code |= spread10(uint32_t(c)) << (2 - k);
    }
    return code;
}

// 30-bit Morton code of the mean inside the valid-mean bounds; invalid
// Gaussians get 0xFFFFFFFF and sort to the end.
__device__ inline uint32_t morton_code(const float *__restrict__ mean, const float *__restrict__ scale,
                                       const float *__restrict__ quat, const float *__restrict__ dens, int64_t n,
                                       int64_t i, const Bounds &b) {
    double mu[3], s[3], q[4], rho;
    if (!load_params(mean, scale, quat, dens, n, i, mu, s, q, rho)) return 0xFFFFFFFFu;
    const float m[3] = {float(mu[0]), float(mu[1]), float(mu[2])};
    return mean_code(m, b);
}

// Codes of one sort tile, its first digit's histogram, and (block 0) the
// header. vals = input index.
__global__ __launch_bounds__(256) void k_codes(const float *__restrict__ mean, const float *__restrict__ scale,
                                               const float *__restrict__ quat, const float *__restrict__ dens,
                                               int64_t n, const Bounds *__restrict__ part, int n_part,
                                               AccelHeader *hdr, int32_t leaf, int32_t n_leaves, float kappa,
                                               uint32_t *__restrict__ keys, uint32_t *__restrict__ vals,
                                               uint32_t *__restrict__ hist) {
    __shared__ Bounds lds[4];
    __shared__ uint32_t h[256];
    h[threadIdx.x] = 0;
    Bounds b;
    bounds_empty(b);
    if (int(threadIdx.x) < n_part) b = part[threadIdx.x];
    bounds_of_block(b, lds);
    if (blockIdx.x == 0 && threadIdx.x == 0) write_header(hdr, n, leaf, n_leaves, kappa, b);
    const int64_t base = int64_t(blockIdx.x) * kSortTile;
    for (int k = 0; k < kSortTile / 256; ++k) {
        const int64_t i = base + k * 256 + threadIdx.x;
        if (i < n) {
            const uint32_t code = morton_code(mean, scale, quat, dens, n, i, b);
            keys[i] = code;
            vals[i] = uint32_t(i);
            atomicAdd(&h[code & 255u], 1u);
        }
    }
    __syncthreads();
    hist[size_t(threadIdx.x) * gridDim.x + blockIdx.x] = h[threadIdx.x];
}

// Up to kSmallSort Gaussians: bounds, header, codes and the sort of (code, input
// index) in one launch. Every workgroup reads all Gaussians for the bounds and
// the codes, and places 64 of them: a key's rank is the number of keys before
// it, counted from LDS (each of the 16 waves counts one key in 16, which all its
// lanes read at once), so nothing waits for another workgroup. Its reads and
// compares grow with n^2 but stay spread over the chip, where sorting inside one
// workgroup is bound by that compute unit's LDS (3,001 keys: this launch 15 us,
// a bitonic sort 40 us, sorted runs merged by binary search 35-39 us).
// A whole build takes, sorted here / by the radix sort's 13 launches:
// 512 Gaussians 22 / 53 us, 3,001 30 / 64, 8,192 46 / 70, 12,000 57 / 71,
// 16,000 66 / 72. The codes have to fit into the default 64 KB of LDS as well.
constexpr uint32_t kLastCode = 0x40000000u;  // of an invalid Gaussian: after all 30-bit codes
__global__ __launch_bounds__(1024) void k_sort_small(const float *__restrict__ mean, const float *__restrict__ scale,
                                                     const float *__restrict__ quat, const float *__restrict__ dens,
                                                     int32_t n, AccelHeader *hdr, int32_t leaf, int32_t n_leaves,
                                                     float kappa, uint32_t *__restrict__ keys,
                                                     uint32_t *__restrict__ vals) {
    extern __shared__ __attribute__((aligned(16))) uint32_t code[];  // n, rounded up to 64
    __shared__ Bounds lds[16];
    __shared__ int before[64];
    const int t = threadIdx.x, lane = t & 63, wave = t >> 6;
    const int rows = (n + 63) >> 6;
    Bounds b;
    bounds_empty(b);
#pragma unroll 4
    for (int i = t; i < n; i += 1024) {
        double mu[3], s[3], q4[4], rho;
        const bool ok = load_params(mean, scale, quat, dens, n, i, mu, s, q4, rho);
        b.bad += ok ? 0 : 1;
        for (int k = 0; k < 3; ++k) {
            const uint32_t u = f2ord(float(mu[k]));
            b.lo[k] = min(b.lo[k], ok ? u : 0xFFFFFFFFu);
            b.hi[k] = max(b.hi[k], ok ? u : 0u);
        }
        code[i] = ok ? 0u : kLastCode;
    }
    if (t < 64) before[t] = 0;
    bounds_of_block(b, lds);
    if (blockIdx.x == 0 && t == 0) write_header(hdr, n, leaf, n_leaves, kappa, b);
#pragma unroll 4
    for (int i = t; i < n; i += 1024) {  // each thread its own again
        const float m[3] = {mean[i], mean[size_t(n) + i], mean[2 * size_t(n) + i]};
        if (code[i] == 0u) code[i] = mean_code(m, b);
    }
    for (int i = n + t; i < rows * 64; i += 1024) code[i] = 0xFFFFFFFFu;
    __syncthreads();
    const int row = int(blockIdx.x), i = row * 64 + lane;
    const uint32_t mine = code[i];
    int c = 0;
    for (int r = wave; r < rows; r += 16) {  // 64 keys of row r: equal ones of earlier rows go first
        const uint32_t first = r < row ? mine + 1u : mine;  // (no overflow where it counts: i < n)
#pragma unroll
        for (int k = 0; k < 64; k += 4) {
            const uint4 v = *reinterpret_cast<const uint4 *>(code + r * 64 + k);
            c += int(v.x < first) + int(v.y < first) + int(v.z < first) + int(v.w < first);
        }
        if (r == row)
            for (int k = 0; k < 64; ++k) c += int(code[r * 64 + k] == mine && k < lane);
    }
    atomicAdd(&before[lane], c);
    __syncthreads();
    if (wave == 0 && i < n) {
        keys[before[lane]] = mine == kLastCode ? 0xFFFFFFFFu : mine;
        vals[before[lane]] = uint32_t(i);
    }
}

// ---------------------------------------------------------------------------
// stable LSD radix sort, 8-bit digits: histogram -> scan -> scatter
// ---------------------------------------------------------------------------

__global__ __launch_bounds__(256) void k_sort_hist(const uint32_t *__restrict__ keys, int64_t n,
                                                   int shift, uint32_t *__restrict__ hist) {
    __shared__ uint32_t h[256];
    h[threadIdx.x] = 0;
    __syncthreads();
    const int64_t base = int64_t(blockIdx.x) * kSortTile;
    for (int k = 0; k < kSortTile / 256; ++k) {
        const int64_t i = base + k * 256 + threadIdx.x;
        if (i < n) atomicAdd(&h[(keys[i] >> shift) & 255u], 1u);
    }
    __syncthreads();
    hist[size_t(threadIdx.x) * gridDim.x + blockIdx.x] = h[threadIdx.x];
}

// Inclusive scan over the 256 threads of a workgroup.
__device__ inline uint32_t scan256(uint32_t v, uint32_t *lds) {
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const uint32_t in = uint32_t(wave_incl_scan(int(v)));
    if (lane == 63) lds[wave] = in;
    __syncthreads();
    uint32_t before = 0;
    for (int w = 0; w < wave; ++w) before += lds[w];
    __syncthreads();
    return in + before;
}

// Digit d's counts over the tiles (a row of the histogram) become its exclusive
// prefix sums, and its total is written: one workgroup per digit. (One
// workgroup over the whole histogram took 48 us per pass at 500k Gaussians.)
__global__ __launch_bounds__(256) void k_sort_rows(uint32_t *__restrict__ hist, int nblocks,
                                                   uint32_t *__restrict__ totals) {
    __shared__ uint32_t lds[4];
    __shared__ uint32_t last;
    uint32_t *row = hist + size_t(blockIdx.x) * nblocks;
    uint32_t run = 0;
    for (int base = 0; base < nblocks; base += 256) {
        const int i = base + int(threadIdx.x);
        const uint32_t v = i < nblocks ? row[i] : 0u;
        const uint32_t in = scan256(v, lds);
        if (i < nblocks) row[i] = run + in - v;
        if (threadIdx.x == 255) last = in;
        __syncthreads();
        run += last;
        __syncthreads();
    }
    if (threadIdx.x == 0) totals[blockIdx.x] = run;
}

// Stable scatter. Each workgroup walks its tile in rounds of 256 keys in
// input order; inside a wave the keys sharing a digit are found with eight
// ballots (one per digit bit), so each key's rank among equal digits is the
// population count of lower lanes with the same digit.
__global__ __launch_bounds__(256) void k_sort_scatter(const uint32_t *__restrict__ kin,
                                                      const uint32_t *__restrict__ vin,
                                                      uint32_t *__restrict__ kout,
                                                      uint32_t *__restrict__ vout, int64_t n,
                                                      int shift, const uint32_t *__restrict__ hist,
                                                      const uint32_t *__restrict__ totals) {
    __shared__ uint32_t run[256];
    __shared__ uint32_t wsl[4][256];
    __shared__ uint32_t lds[4];
    const int t = threadIdx.x, w = t >> 6, lane = t & 63;
    const uint32_t total = totals[t];
    run[t] = scan256(total, lds) - total + hist[size_t(t) * gridDim.x + blockIdx.x];
    const uint64_t lt = (lane == 0) ? 0ull : (~0ull >> (64 - lane));
    const int64_t base = int64_t(blockIdx.x) * kSortTile;
    for (int k = 0; k < kSortTile / 256; ++k) {
        const int64_t i = base + k * 256 + t;
        const bool valid = i < n;
        const uint32_t key = valid ? kin[i] : 0u;
        const uint32_t val = valid ? vin[i] : 0u;
        const uint32_t dig = (key >> shift) & 255u;
        for (int ww = 0; ww < 4; ++ww) wsl[ww][t] = 0;
        __syncthreads();
        uint64_t peers = __ballot(valid);
        for (int b = 0; b < 8; ++b) {
            const bool bit = (dig >> b) & 1u;
            const uint64_t bal = __ballot(valid && bit);
            peers &= bit ? bal : ~bal;
        }
        const uint32_t rank = uint32_t(__popcll(peers & lt));
        if (valid && rank == 0) wsl[w][dig] = uint32_t(__popcll(peers));
        __syncthreads();
        const uint32_t c0 = wsl[0][t], c1 = wsl[1][t], c2 = wsl[2][t], c3 = wsl[3][t];
        const uint32_t g = run[t];
        __syncthreads();
        wsl[0][t] = g;
        wsl[1][t] = g + c0;
        wsl[2][t] = g + c0 + c1;
        wsl[3][t] = g + c0 + c1 + c2;
        run[t] = g + c0 + c1 + c2 + c3;
        __syncthreads();
        if (valid) {
            const uint32_t pos = wsl[w][dig] + rank;
            if (pos < n) {
                kout[pos] = key;
                vout[pos] = val;
            }
        }
        __syncthreads();
    }
}

// ---------------------------------------------------------------------------
// per-Gaussian records in Morton order
// ---------------------------------------------------------------------------

// Records of the Gaussian at Morton position g; its kappa box in `box` (empty
// if it is invalid: returns false).
__device__ inline bool write_records(const float *__restrict__ mean,
                                                const float *__restrict__ scale,
                                                const float *__restrict__ quat,
                                                const float *__restrict__ dens, int64_t n,
                                                float kappa, int32_t leaf, const uint32_t *__restrict__ order,
                                                GaussRec *__restrict__ rec,
                                                GaussRec32 *__restrict__ rec32,
                                                char *__restrict__ axis, size_t axis_stride,
                                                float *__restrict__ cull, int64_t g, float box[6]) {
    for (int k = 0; k < 3; ++k) {
        box[k] = FLT_MAX;
        box[3 + k] = -FLT_MAX;
    }
    const int64_t i = order[g];
    float *leaf_cull = cull + (g / leaf) * leaf * kCullFields + g % leaf;
    double mu[3], s[3], q[4], rho;
    GaussRec r;
    if (i >= n || !load_params(mean, scale, quat, dens, n, i, mu, s, q, rho)) {
        for (int k = 0; k < 3; ++k) r.mu[k] = __builtin_nan("");
        for (int k = 0; k < 6; ++k) r.P[k] = 0.0;
        r.rho_c = 0.0f;
        r.pad = 0.0f;
        rec[g] = r;
        GaussRec32 c;
        for (int k = 0; k < 3; ++k) c.mu[k] = __builtin_nanf("");
        for (int k = 0; k < 9; ++k) c.W[k] = 0.0f;
        c.rho_c = 0.0f;
        c.pad[0] = c.pad[1] = c.pad[2] = 0.0f;
        rec32[g] = c;
        AxisRec a = {};
        a.m1 = a.m2 = a.mk = __builtin_nan("");
        for (int k = 0; k < 3; ++k) reinterpret_cast<AxisRec *>(axis + k * axis_stride)[g] = a;
        for (int f = 0; f < kCullFields; ++f) leaf_cull[f * leaf] = __builtin_nanf("");
        return false;
    }
    double R[3][3];
    rotation(q, R);
    double Sg[3][3];
    for (int a = 0; a < 3; ++a)
        for (int b = 0; b < 3; ++b)
            Sg[a][b] = R[a][0] * R[b][0] * s[0] * s[0] + R[a][1] * R[b][1] * s[1] * s[1] +
                       R[a][2] * R[b][2] * s[2] * s[2];
    // precision matrix P = R diag(s^-2) R^T, the inverse of Sigma
    const double is[3] = {1.0 / s[0], 1.0 / s[1], 1.0 / s[2]};
    const double lam[3] = {1.0 / (s[0] * s[0]), 1.0 / (s[1] * s[1]), 1.0 / (s[2] * s[2])};
    double Pm[3][3];
    for (int a = 0; a < 3; ++a)
        for (int b = 0; b < 3; ++b)
            Pm[a][b] = R[a][0] * R[b][0] * lam[0] + R[a][1] * R[b][1] * lam[1] + R[a][2] * R[b][2] * lam[2];
    for (int k = 0; k < 3; ++k) r.mu[k] = mu[k];
    r.P[0] = Pm[0][0];
    r.P[1] = Pm[1][1];
    r.P[2] = Pm[2][2];
    r.P[3] = Pm[0][1];
    r.P[4] = Pm[0][2];
    r.P[5] = Pm[1][2];
    r.rho_c = float(rho * 2.5066282746310002);  // rho sqrt(2 pi)
    r.pad = 0.0f;
    rec[g] = r;
    // whitening W = diag(1/s) R^T: row a is the a-th local axis over its scale
    GaussRec32 c;
    for (int k = 0; k < 3; ++k) c.mu[k] = float(mu[k]);
    for (int a = 0; a < 3; ++a)
        for (int b = 0; b < 3; ++b) c.W[3 * a + b] = float(R[b][a] * is[a]);
    c.rho_c = r.rho_c;
    c.pad[0] = c.pad[1] = c.pad[2] = 0.0f;
    rec32[g] = c;
    // views along the axes; det P Sigma_kk is the determinant of P's (t1, t2)
    // block, so l22 = sqrt(det / P11) loses nothing to cancellation
    const double iv = 1.0 / (s[0] * s[1] * s[2]);
    for (int k = 0; k < 3; ++k) {
        const int t1 = (k + 1) % 3, t2 = (k + 2) % 3;
        AxisRec a;
        a.m1 = mu[t1];
        a.m2 = mu[t2];
        a.mk = mu[k];
        a.h = 1.0 / Sg[k][k];
        a.s1 = Sg[t1][k] * a.h;
        a.s2 = Sg[t2][k] * a.h;
        a.l11 = sqrt(Pm[t1][t1]);
        const double i11 = 1.0 / a.l11;
        a.l21 = Pm[t1][t2] * i11;
        a.l22 = iv * sqrt(Sg[k][k]) * i11;
        a.rho_c = r.rho_c;
        a.pad = 0.0f;
        reinterpret_cast<AxisRec *>(axis + k * axis_stride)[g] = a;
    }
    const double k2 = double(kappa) * double(kappa);
    leaf_cull[0 * leaf] = float(mu[0]);
    leaf_cull[1 * leaf] = float(mu[1]);
    leaf_cull[2 * leaf] = float(mu[2]);
    leaf_cull[3 * leaf] = float(k2 * Sg[0][0]);
    leaf_cull[4 * leaf] = float(k2 * Sg[1][1]);
    leaf_cull[5 * leaf] = float(k2 * Sg[2][2]);
    leaf_cull[6 * leaf] = float(k2 * Sg[0][1]);
    leaf_cull[7 * leaf] = float(k2 * Sg[0][2]);
    leaf_cull[8 * leaf] = float(k2 * Sg[1][2]);
    for (int k = 0; k < 3; ++k) {
        const float e = float(double(kappa) * sqrt(Sg[k][k])) * (1.0f + kBoxRel) + kBoxAbs;
        box[k] = float(mu[k]) - e;
        box[3 + k] = float(mu[k]) + e;
    }
    return true;
}

// Records of whole leaves (256 / leaf of them per workgroup) and the leaves'
// boxes, joined in LDS (level 0 of the wide hierarchy). count: add the invalid
// Gaussians to the header (a refit; a build counted them with the bounds).
__global__ __launch_bounds__(256) void k_gather(const float *__restrict__ mean, const float *__restrict__ scale,
                                                const float *__restrict__ quat, const float *__restrict__ dens,
                                                int64_t n, float kappa, int32_t leaf,
                                                const uint32_t *__restrict__ order, GaussRec *__restrict__ rec,
                                                GaussRec32 *__restrict__ rec32, char *__restrict__ axis,
                                                size_t axis_stride, float *__restrict__ cull,
                                                float *__restrict__ wbox, int wide_total, int n_leaves,
                                                AccelHeader *hdr, int count) {
    __shared__ float boxes[6][256];
    const int per = 256 / leaf, t = threadIdx.x;
    const int64_t g = int64_t(blockIdx.x) * per * leaf + t;
    float box[6];
    bool bad = false;
    if (t < per * leaf && g < n) {
        bad = !write_records(mean, scale, quat, dens, n, kappa, leaf, order, rec, rec32, axis, axis_stride, cull, g,
                             box);
    } else {
        for (int k = 0; k < 3; ++k) {
            box[k] = FLT_MAX;
            box[3 + k] = -FLT_MAX;
        }
    }
    for (int k = 0; k < 6; ++k) boxes[k][t] = box[k];
    if (count) {
        const int n_bad = __builtin_popcountll(ballot(bad));
        if (n_bad && (t & 63) == 0) atomicAdd(&hdr->n_invalid, n_bad);
    }
    __syncthreads();
    // thread (field, leaf) of the workgroup
    for (int q = t; q < 6 * per; q += 256) {
        const int f = q / per, l = q % per;
        const int64_t id = int64_t(blockIdx.x) * per + l;
        if (id >= n_leaves) continue;
        float v = f < 3 ? FLT_MAX : -FLT_MAX;
        for (int k = 0, j = t % leaf; k < leaf; ++k, j = j + 1 < leaf ? j + 1 : 0) {
            const float o = boxes[f][l * leaf + j];  // (started apart: one bank each)
            v = f < 3 ? fminf(v, o) : fmaxf(v, o);
        }
        wbox[size_t(f) * wide_total + id] = v;
    }
}

// ---------------------------------------------------------------------------
// wide hierarchy above the leaves, and the header's root box
// ---------------------------------------------------------------------------

// Box of up to 64 consecutive nodes [first, first + cnt) joined over a wave.
struct Box {
    float v[6];
};

__device__ inline Box box_empty() {
    Box b;
    for (int k = 0; k < 3; ++k) {
        b.v[k] = FLT_MAX;
        b.v[3 + k] = -FLT_MAX;
    }
    return b;
}

__device__ inline void box_add(Box &b, const float *wbox, int total, int i) {
    for (int k = 0; k < 3; ++k) {
        b.v[k] = fminf(b.v[k], wbox[size_t(k) * total + i]);
        b.v[3 + k] = fmaxf(b.v[3 + k], wbox[size_t(3 + k) * total + i]);
    }
}

__device__ inline void box_of_wave(Box &b) {
    for (int k = 0; k < 3; ++k) {
        b.v[k] = wave_min(b.v[k]);
        b.v[3 + k] = wave_max(b.v[3 + k]);
    }
}

// Node i of a level: the union of children [64 i, 64 i + 64) of the level below,
// one wave per node.
__device__ inline void wide_node(float *wbox, int total, int child_off, int child_count, int off, int i, int lane) {
    Box b = box_empty();
    if (i * kWide + lane < child_count) box_add(b, wbox, total, child_off + i * kWide + lane);
    box_of_wave(b);
    if (lane == 0)
        for (int k = 0; k < 6; ++k) wbox[size_t(k) * total + off + i] = b.v[k];
}

__global__ __launch_bounds__(256) void k_wide_level(float *wbox, int total, int child_off, int child_count, int off,
                                                    int count) {
    const int i = int(blockIdx.x) * 4 + __builtin_amdgcn_readfirstlane(int(threadIdx.x >> 6));
    if (i < count) wide_node(wbox, total, child_off, child_count, off, i, threadIdx.x & 63);
}

struct LevelTable {
    int n_levels;
    int count[kMaxLevels], off[kMaxLevels];
};

// The levels from `first` up in one workgroup, then the root box; marks the
// header built (what still runs on the stream only adds to the binary tree).
__global__ __launch_bounds__(1024) void k_wide_top(float *wbox, int total, LevelTable L, int first, AccelHeader *hdr) {
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(int(threadIdx.x >> 6));
    for (int lv = first; lv < L.n_levels; ++lv) {
        for (int i = wave; i < L.count[lv]; i += 16)
            wide_node(wbox, total, L.off[lv - 1], L.count[lv - 1], L.off[lv], i, lane);
        __threadfence_block();
        __syncthreads();
    }
    if (threadIdx.x < 6) hdr->root_box[threadIdx.x] = wbox[size_t(threadIdx.x) * total + total - 1];
    if (threadIdx.x == 0) hdr->built = 1;
}

// ---------------------------------------------------------------------------
// Karras radix tree over leaves; leaf l holds Morton positions [l L, (l+1) L)
// ---------------------------------------------------------------------------

__device__ inline int prefix_len(const uint32_t *__restrict__ keys, int leaf, int nl, int i, int j) {
    if (j < 0 || j >= nl) return -1;
    const uint32_t a = keys[size_t(i) * leaf], b = keys[size_t(j) * leaf];
    if (a == b) return 32 + __clz(uint32_t(i ^ j));
    return __clz(a ^ b);
}

// Box of leaves [a, b], joined over a wave: ragged ends at this level, the whole
// groups of 64 between them from the level above.
__device__ inline Box leaf_range_box(const float *wbox, int total, const LevelTable &L, int a, int b, int lane) {
    Box r = box_empty();
    int lv = 0;
    for (; b - a >= 2 * kWide && lv + 1 < L.n_levels; ++lv) {
        const int a1 = (a + kWide - 1) / kWide, b1 = (b + 1) / kWide;  // groups [a1, b1)
        if (a + lane < a1 * kWide) box_add(r, wbox, total, L.off[lv] + a + lane);
        if (b1 * kWide + lane <= b) box_add(r, wbox, total, L.off[lv] + b1 * kWide + lane);
        a = a1;
        b = b1 - 1;
    }
    for (int i = a + lane; i <= b; i += kWide) box_add(r, wbox, total, L.off[lv] + i);
    box_of_wave(r);
    return r;
}

// Binary node i, one wave: with kTopology its range of leaves and its children
// (Karras' radix tree; every lane takes the same steps), then its children's
// boxes. A refit keeps the stored ranges.
template <bool kTopology>
__global__ __launch_bounds__(256) void k_nodes(const uint32_t *__restrict__ keys, int leaf, int nl,
                                               Node *__restrict__ nodes, const float *__restrict__ wbox, int total,
                                               LevelTable L, AccelHeader *hdr) {
    const int i = int(blockIdx.x) * 4 + __builtin_amdgcn_readfirstlane(int(threadIdx.x >> 6));
    const int lane = threadIdx.x & 63;
    if (i >= nl - 1) return;
    int lo, hi, gam;
    if constexpr (kTopology) {
        const int d = (prefix_len(keys, leaf, nl, i, i + 1) - prefix_len(keys, leaf, nl, i, i - 1)) >= 0 ? 1 : -1;
        const int dmin = prefix_len(keys, leaf, nl, i, i - d);
        int lmax = 2;
        while (prefix_len(keys, leaf, nl, i, i + lmax * d) > dmin) lmax <<= 1;
        int l = 0;
        for (int t = lmax >> 1; t >= 1; t >>= 1)
            if (prefix_len(keys, leaf, nl, i, i + (l + t) * d) > dmin) l += t;
        const int j = i + l * d;
        const int dnode = prefix_len(keys, leaf, nl, i, j);
        int s = 0, step = l;
        do {
            step = (step + 1) >> 1;
            if (prefix_len(keys, leaf, nl, i, i + (s + step) * d) > dnode) s += step;
        } while (step > 1);
        gam = i + s * d + (d < 0 ? -1 : 0);
        lo = min(i, j);
        hi = max(i, j);
    } else {
        lo = nodes[i].lo;
        hi = nodes[i].hi;
        const int left = nodes[i].child[0];
        gam = left < 0 ? ~left : left;
    }
    if (lo < 0 || hi >= nl || gam < lo || gam >= hi) {
        if (lane == 0) {
            nodes[i].child[0] = nodes[i].child[1] = nl;  // no node and no leaf: the traversal stops there
            atomicOr(&hdr->flags, kFlagTreeCorrupt);
        }
        return;
    }
    const Box l = leaf_range_box(wbox, total, L, lo, gam, lane), r = leaf_range_box(wbox, total, L, gam + 1, hi, lane);
    if (lane == 0) {
        Node nd;
        for (int k = 0; k < 6; ++k) {
            nd.b[k] = l.v[k];
            nd.b[6 + k] = r.v[k];
        }
        nd.child[0] = lo == gam ? ~gam : gam;
        nd.child[1] = hi == gam + 1 ? ~(gam + 1) : gam + 1;
        nd.lo = lo;
        nd.hi = hi;
        nodes[i] = nd;
    }
}

// ---------------------------------------------------------------------------
// host driver
// ---------------------------------------------------------------------------

static inline unsigned blocks_for(int64_t count, int threads) {
    return unsigned((count + threads - 1) / threads);
}

// Records, leaf boxes, the wide hierarchy and the binary tree's nodes, from the
// Morton order.
static void enqueue_structure(const gr_scene &sc, const Layout &L, bool refit, hipStream_t st) {
    char *base = static_cast<char *>(sc.accel);
    AccelHeader *hdr = reinterpret_cast<AccelHeader *>(base);
    const int64_t n = sc.n;
    const uint32_t *order = reinterpret_cast<const uint32_t *>(base + L.vals0);
    float *wbox = reinterpret_cast<float *>(base + L.wbox);
    const int per = 256 / L.leaf;  // leaves per workgroup
    k_gather<<<blocks_for(L.n_leaves, per), 256, 0, st>>>(
        sc.mean, sc.scale, sc.quat, sc.density, n, sc.kappa, L.leaf, order,
        reinterpret_cast<GaussRec *>(base + L.rec), reinterpret_cast<GaussRec32 *>(base + L.rec32), base + L.axis,
        align256(size_t(n) * sizeof(AxisRec)), reinterpret_cast<float *>(base + L.cull), wbox, L.wide_total,
        L.n_leaves, hdr, refit ? 1 : 0);
    LevelTable T{};
    T.n_levels = L.n_levels;
    for (int k = 0; k < kMaxLevels; ++k) {
        T.count[k] = L.level_count[k];
        T.off[k] = L.level_off[k];
    }
    int lv = 1;
    for (; lv < L.n_levels && L.level_count[lv] > 1024; ++lv)
        k_wide_level<<<blocks_for(L.level_count[lv], 4), 256, 0, st>>>(
            wbox, L.wide_total, L.level_off[lv - 1], L.level_count[lv - 1], L.level_off[lv], L.level_count[lv]);
    k_wide_top<<<1, 1024, 0, st>>>(wbox, L.wide_total, T, lv, hdr);
    if (L.n_nodes > 0) {
        Node *nodes = reinterpret_cast<Node *>(base + L.nodes);
        const uint32_t *keys = reinterpret_cast<const uint32_t *>(base + L.keys0);
        if (refit)
            k_nodes<false><<<blocks_for(L.n_nodes, 4), 256, 0, st>>>(keys, L.leaf, L.n_leaves, nodes, wbox,
                                                                     L.wide_total, T, hdr);
        else
            k_nodes<true><<<blocks_for(L.n_nodes, 4), 256, 0, st>>>(keys, L.leaf, L.n_leaves, nodes, wbox,
                                                                    L.wide_total, T, hdr);
    }
}

hipError_t enqueue_refit(const gr_scene &sc, const Layout &L, hipStream_t st) {
    AccelHeader *hdr = static_cast<AccelHeader *>(sc.accel);
    k_refit_init<<<1, 64, 0, st>>>(hdr, sc.n, L.leaf, L.n_leaves, sc.kappa);
    if (sc.n > 0) enqueue_structure(sc, L, true, st);
    return hipGetLastError();
}

hipError_t enqueue_build(const gr_scene &sc, const Layout &L, hipStream_t st) {
    char *base = static_cast<char *>(sc.accel);
    AccelHeader *hdr = reinterpret_cast<AccelHeader *>(base);
    const int64_t n = sc.n;
    if (n == 0) {
        k_build_empty<<<1, 64, 0, st>>>(hdr, L.leaf, L.n_leaves, sc.kappa);
        return hipGetLastError();
    }
    uint32_t *k0 = reinterpret_cast<uint32_t *>(base + L.keys0);
    uint32_t *k1 = reinterpret_cast<uint32_t *>(base + L.keys1);
    uint32_t *v0 = reinterpret_cast<uint32_t *>(base + L.vals0);
    uint32_t *v1 = reinterpret_cast<uint32_t *>(base + L.vals1);
    if (n <= kSmallSort) {
        const unsigned rows = unsigned((n + 63) / 64);
        k_sort_small<<<rows, 1024, rows * 64 * sizeof(uint32_t), st>>>(sc.mean, sc.scale, sc.quat, sc.density,
                                                                       int32_t(n), hdr, L.leaf, L.n_leaves, sc.kappa,
                                                                       k0, v0);
    } else {
        uint32_t *hist = reinterpret_cast<uint32_t *>(base + L.hist);
        uint32_t *totals = reinterpret_cast<uint32_t *>(base + L.totals);
        Bounds *part = reinterpret_cast<Bounds *>(base + L.part);
        const int nb = L.n_sort_blocks;
        const int n_part = int(blocks_for(n, 256) < unsigned(kBoundsBlocks) ? blocks_for(n, 256) : kBoundsBlocks);
        k_bounds<<<n_part, 256, 0, st>>>(sc.mean, sc.scale, sc.quat, sc.density, n, part);
        k_codes<<<nb, 256, 0, st>>>(sc.mean, sc.scale, sc.quat, sc.density, n, part, n_part, hdr, L.leaf, L.n_leaves,
                                    sc.kappa, k0, v0, hist);
        uint32_t *kin = k0, *vin = v0, *kout = k1, *vout = v1;
        for (int pass = 0; pass < 4; ++pass) {
            const int shift = 8 * pass;
            if (pass > 0) k_sort_hist<<<nb, 256, 0, st>>>(kin, n, shift, hist);
            k_sort_rows<<<256, 256, 0, st>>>(hist, nb, totals);
            k_sort_scatter<<<nb, 256, 0, st>>>(kin, vin, kout, vout, n, shift, hist, totals);
            uint32_t *tk = kin, *tv = vin;
            kin = kout;
            vin = vout;
            kout = tk;
            vout = tv;
        }
        // four passes: the sorted keys and order are back in keys0 / vals0
    }
    enqueue_structure(sc, L, false, st);
    return hipGetLastError();
}

}  // namespace gr
