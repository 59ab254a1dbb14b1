// Tree construction on the device: bounds, Morton keys, stable LSD radix sort,
// gather into Morton order, level-synchronous octree build and cell geometry.
// Sec. 3.2 of the paper (Morton ordering of 3 x 21 coordinate bits in a 64-bit
// key; at most 21 levels).
#include "ctx.h"

#include <algorithm>
#include <cstring>

namespace vfmm {

static constexpr int TPB = 256;
// work-groups of the first bounds pass (each reduces a strided share of the particles)
static constexpr int BOUNDS_MAX_PARTS = 1024;
// up to this many particles one work-group of 1,024 threads does both passes
static constexpr int64_t BOUNDS_ONE_GROUP = 8192;

// ---------------------------------------------------------------------------
// Exclusive scan of int32 (in-place allowed).  2048 items per block, block
// totals scanned recursively.
// ---------------------------------------------------------------------------
static constexpr int SCAN_ITEMS = 8;
static constexpr int SCAN_TILE = TPB * SCAN_ITEMS;

__global__ __launch_bounds__(TPB) void k_scan_tile(const int *in, int *out, int64_t n, int *block_sums) {
    __shared__ int wsum[TPB / 64];
    const int tid = threadIdx.x;
    const int64_t base = (int64_t)blockIdx.x * SCAN_TILE + (int64_t)tid * SCAN_ITEMS;
    int v[SCAN_ITEMS];
    int run = 0;
#pragma unroll
    for (int i = 0; i < SCAN_ITEMS; ++i) {
        const int64_t k = base + i;
        v[i] = k < n ? in[k] : 0;
        run += v[i];
    }
    // wave inclusive scan of thread totals
    const int lane = tid & 63, w = tid >> 6;
    int incl = run;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
        const int t = __shfl_up(incl, o, 64);
        if (lane >= o) incl += t;
    }
    if (lane == 63) wsum[w] = incl;
    __syncthreads();
    int woff = 0;
    for (int i = 0; i < w; ++i) woff += wsum[i];
    int ex = woff + incl - run;
#pragma unroll
    for (int i = 0; i < SCAN_ITEMS; ++i) {
        const int64_t k = base + i;
        if (k < n) out[k] = ex;
        ex += v[i];
    }
    if (tid == TPB - 1 && block_sums) block_sums[blockIdx.x] = woff + incl;
}

__global__ __launch_bounds__(TPB) void k_scan_add(int *out, int64_t n, const int *offs) {
    const int64_t base = (int64_t)blockIdx.x * SCAN_TILE;
    const int add = offs[blockIdx.x];
    for (int i = threadIdx.x; i < SCAN_TILE; i += TPB) {
        const int64_t k = base + i;
        if (k < n) out[k] += add;
    }
}

// Up to SCAN_FEW_TILES tiles: reduce-then-scan in two launches, each tile's
// offset summed by its own work-group from the totals of the tiles before it.
static constexpr int SCAN_FEW_TILES = 1024;

__global__ __launch_bounds__(TPB) void k_scan_tile_sums(const int *in, int64_t n, int *block_sums) {
    __shared__ int wsum[TPB / 64];
    const int64_t base = (int64_t)blockIdx.x * SCAN_TILE + (int64_t)threadIdx.x * SCAN_ITEMS;
    int run = 0;
#pragma unroll
    for (int i = 0; i < SCAN_ITEMS; ++i) run += base + i < n ? in[base + i] : 0;
    for (int o = 32; o > 0; o >>= 1) run += __shfl_xor(run, o, 64);
    if ((threadIdx.x & 63) == 0) wsum[threadIdx.x >> 6] = run;
    __syncthreads();
    if (threadIdx.x == 0) {
        int t = 0;
        for (int w = 0; w < TPB / 64; ++w) t += wsum[w];
        block_sums[blockIdx.x] = t;
    }
}

__global__ __launch_bounds__(TPB) void k_scan_tile_offset(const int *in, int *out, int64_t n, const int *block_sums) {
    __shared__ int wsum[TPB / 64];
    __shared__ int boff;
    const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
    // offset of this tile: the totals of the tiles before it (at most SCAN_FEW_TILES - 1)
    int o = 0;
    for (int i = tid; i < (int)blockIdx.x; i += TPB) o += block_sums[i];
    for (int d = 32; d > 0; d >>= 1) o += __shfl_xor(o, d, 64);
    if (lane == 0) wsum[w] = o;
    __syncthreads();
    if (tid == 0) {
        int t = 0;
        for (int i = 0; i < TPB / 64; ++i) t += wsum[i];
        boff = t;
    }
    __syncthreads();  // wsum is reused below
    const int64_t base = (int64_t)blockIdx.x * SCAN_TILE + (int64_t)tid * SCAN_ITEMS;
    int v[SCAN_ITEMS];
    int run = 0;
#pragma unroll
    for (int i = 0; i < SCAN_ITEMS; ++i) {
        const int64_t k = base + i;
        v[i] = k < n ? in[k] : 0;
        run += v[i];
    }
    int incl = run;
#pragma unroll
    for (int d = 1; d < 64; d <<= 1) {
        const int t = __shfl_up(incl, d, 64);
        if (lane >= d) incl += t;
    }
    if (lane == 63) wsum[w] = incl;
    __syncthreads();
    int woff = boff;
    for (int i = 0; i < w; ++i) woff += wsum[i];
    int ex = woff + incl - run;
#pragma unroll
    for (int i = 0; i < SCAN_ITEMS; ++i) {
        const int64_t k = base + i;
        if (k < n) out[k] = ex;
        ex += v[i];
    }
}

static void scan_rec(hipStream_t s, const int *in, int *out, int64_t n, int *scratch) {
    if (n <= 0) return;
    const unsigned nb = cdiv(n, SCAN_TILE);
    if (nb == 1) {
        k_scan_tile<<<1, TPB, 0, s>>>(in, out, n, nullptr);
        VFMM_LAUNCH_CHECK();
        return;
    }
    if (nb <= (unsigned)SCAN_FEW_TILES) {  // in may alias out: the totals are taken before any write
        k_scan_tile_sums<<<nb, TPB, 0, s>>>(in, n, scratch);
        VFMM_LAUNCH_CHECK();
        k_scan_tile_offset<<<nb, TPB, 0, s>>>(in, out, n, scratch);
        VFMM_LAUNCH_CHECK();
        return;
    }
    int *sums = scratch;
    k_scan_tile<<<nb, TPB, 0, s>>>(in, out, n, sums);
    VFMM_LAUNCH_CHECK();
    scan_rec(s, sums, sums, nb, scratch + nb);
    k_scan_add<<<nb, TPB, 0, s>>>(out, n, sums);
    VFMM_LAUNCH_CHECK();
}

void scan_excl_i32(Ctx &c, const int *in, int *out, int64_t n) {
    size_t need = 0;
    for (int64_t m = cdiv(n, SCAN_TILE); m > 1; m = cdiv(m, SCAN_TILE)) need += m;
    c.scanC.ensure((need + 64) * sizeof(int));
    scan_rec(c.stream, in, out, n, c.scanC.as<int>());
}

struct IntPtrs {
    const int *p[4];
};

__global__ __launch_bounds__(64) void k_read_ints(IntPtrs src, int n, int *out) {
    const int i = threadIdx.x;
    if (i < n) out[i] = *src.p[i];
}

int *pinned_ints(Ctx &c) {
    if (!c.hpin) VFMM_HIP(hipHostMalloc((void **)&c.hpin, 64 * sizeof(int), hipHostMallocCoherent));
    return c.hpin;
}

void sync_ints(Ctx &c, int n, int *dst) {
    VFMM_HIP(hipStreamSynchronize(c.stream));
    for (int i = 0; i < n; ++i) dst[i] = c.hpin[i];
}

void read_ints(Ctx &c, std::initializer_list<const int *> src, int *dst) {
    if (src.size() == 0 || src.size() > 4) throw Error{VFMM_EINVAL, "read_ints: one to four values"};
    int *hp = pinned_ints(c);
    IntPtrs a{};
    int n = 0;
    for (const int *p : src) a.p[n++] = p;
    k_read_ints<<<1, 64, 0, c.stream>>>(a, n, hp);
    VFMM_LAUNCH_CHECK();
    sync_ints(c, n, dst);
}

// ---------------------------------------------------------------------------
// Bounds: min/max of positions, min/max core, float64 sums of alpha and of
// (x - ref) x alpha, non-finite and out-of-cube counts.  Deterministic two
// stage reduction.
// ---------------------------------------------------------------------------
struct BAcc {
    double lo[3], hi[3], smin, smax, sa[3], sxa[3], fp;
    int nf, out;
};

__device__ inline void bacc_init(BAcc &a) {
    for (int d = 0; d < 3; ++d) {
        a.lo[d] = 1e300; a.hi[d] = -1e300; a.sa[d] = 0; a.sxa[d] = 0;
    }
    a.smin = 1e300; a.smax = -1e300; a.fp = 0; a.nf = 0; a.out = 0;
}

__device__ inline void bacc_merge(BAcc &a, const BAcc &b) {
    for (int d = 0; d < 3; ++d) {
        a.lo[d] = fmin(a.lo[d], b.lo[d]); a.hi[d] = fmax(a.hi[d], b.hi[d]);
        a.sa[d] += b.sa[d]; a.sxa[d] += b.sxa[d];
    }
    a.smin = fmin(a.smin, b.smin); a.smax = fmax(a.smax, b.smax);
    a.fp += b.fp;
    a.nf += b.nf; a.out += b.out;
}

struct BoundsArgs {
    const float *x, *y, *z, *s, *ax, *ay, *az;
    int64_t n;
    int with_alpha, periodic;
    double ref[3];
    double plo[3], plen;
    int check_fp;  // evaluation: compare the fingerprint with fp_ref (the build's)
    double fp_ref;
};

// accumulates this thread's particles (i0, i0 + stride, ...)
__device__ inline void bacc_particles(const BoundsArgs &A, int64_t i0, int64_t stride, BAcc &a) {
    for (int64_t i = i0; i < A.n; i += stride) {
        const double p[3] = {A.x[i], A.y[i], A.z[i]};
        const double sg = A.s[i];
        bool fin = isfinite(p[0]) && isfinite(p[1]) && isfinite(p[2]) && isfinite(sg) && sg > 0.0;
        double al[3] = {0, 0, 0};
        if (A.with_alpha) {
            al[0] = A.ax[i]; al[1] = A.ay[i]; al[2] = A.az[i];
            fin = fin && isfinite(al[0]) && isfinite(al[1]) && isfinite(al[2]);
        }
        a.fp += (double)(1 + i % 61) * (p[0] + 3.0 * p[1] + 5.0 * p[2] + 7.0 * sg);
        if (!fin) { a.nf++; continue; }
        for (int d = 0; d < 3; ++d) { a.lo[d] = fmin(a.lo[d], p[d]); a.hi[d] = fmax(a.hi[d], p[d]); }
        a.smin = fmin(a.smin, sg); a.smax = fmax(a.smax, sg);
        if (A.periodic || A.plen > 0.0) {  // the periodic cell, or a caller-given root cube
            for (int d = 0; d < 3; ++d)
                if (!(p[d] >= A.plo[d] && p[d] < A.plo[d] + A.plen)) { a.out++; break; }
        }
        if (A.with_alpha) {
            const double r[3] = {p[0] - A.ref[0], p[1] - A.ref[1], p[2] - A.ref[2]};
            for (int d = 0; d < 3; ++d) a.sa[d] += al[d];
            a.sxa[0] += r[1] * al[2] - r[2] * al[1];
            a.sxa[1] += r[2] * al[0] - r[0] * al[2];
            a.sxa[2] += r[0] * al[1] - r[1] * al[0];
        }
    }
}

// merges the lanes' accumulators (a fixed tree over the lowest `lanes` lanes)
__device__ inline void bacc_wave(BAcc &a, int lanes) {
    for (int o = lanes / 2; o > 0; o >>= 1) {
        BAcc b;
        for (int d = 0; d < 3; ++d) {
            b.lo[d] = __shfl_xor(a.lo[d], o, 64); b.hi[d] = __shfl_xor(a.hi[d], o, 64);
            b.sa[d] = __shfl_xor(a.sa[d], o, 64); b.sxa[d] = __shfl_xor(a.sxa[d], o, 64);
        }
        b.smin = __shfl_xor(a.smin, o, 64); b.smax = __shfl_xor(a.smax, o, 64);
        b.fp = __shfl_xor(a.fp, o, 64);
        b.nf = __shfl_xor(a.nf, o, 64); b.out = __shfl_xor(a.out, o, 64);
        bacc_merge(a, b);
    }
}

// merges a work-group's accumulators into thread 0's; sh holds one per wave (a power of two)
__device__ inline void bacc_group(BAcc &a, BAcc *sh) {
    const int nw = blockDim.x / 64;
    bacc_wave(a, 64);
    if ((threadIdx.x & 63) == 0) sh[threadIdx.x >> 6] = a;
    __syncthreads();
    if (threadIdx.x < 64) {
        a = sh[threadIdx.x & (nw - 1)];
        bacc_wave(a, nw);
    }
}

// the result of a bounds pass; host (may be null) is pinned host memory
__device__ inline void bounds_result(const BAcc &a, int check_fp, double fp_ref, Bounds *res, Bounds *host) {
    Bounds b;
    for (int d = 0; d < 3; ++d) {
        b.lo[d] = a.lo[d]; b.hi[d] = a.hi[d];
        b.sum_a[d] = a.sa[d]; b.sum_xa[d] = a.sxa[d];
    }
    b.sig_min = a.smin; b.sig_max = a.smax;
    b.fp = a.fp;
    b.nonfinite = a.nf; b.outside = a.out;
    // the sums are deterministic: equal inputs give a bitwise equal fingerprint
    b.stale = (check_fp && !(a.fp == fp_ref)) ? 1 : 0;
    b.overfull = 0;
    *res = b;
    if (host) *host = b;
}

__global__ __launch_bounds__(TPB) void k_bounds_partial(BoundsArgs A, BAcc *part) {
    __shared__ BAcc sh[TPB / 64];
    BAcc a;
    bacc_init(a);
    bacc_particles(A, (int64_t)blockIdx.x * TPB + threadIdx.x, (int64_t)gridDim.x * TPB, a);
    bacc_group(a, sh);
    if (threadIdx.x == 0) part[blockIdx.x] = a;
}

__global__ __launch_bounds__(TPB) void k_bounds_final(const BAcc *part, int np, int check_fp, double fp_ref,
                                                      Bounds *res, Bounds *host) {
    __shared__ BAcc sh[TPB / 64];
    BAcc a;
    bacc_init(a);
    for (int i = threadIdx.x; i < np; i += TPB) bacc_merge(a, part[i]);
    bacc_group(a, sh);
    if (threadIdx.x == 0) bounds_result(a, check_fp, fp_ref, res, host);
}

// both stages in one work-group
__global__ __launch_bounds__(1024) void k_bounds_small(BoundsArgs A, int check_fp, double fp_ref, Bounds *res,
                                                       Bounds *host) {
    __shared__ BAcc sh[1024 / 64];
    BAcc a;
    bacc_init(a);
    bacc_particles(A, threadIdx.x, 1024, a);
    bacc_group(a, sh);
    if (threadIdx.x == 0) bounds_result(a, check_fp, fp_ref, res, host);
}

size_t bounds_scratch_bytes() { return sizeof(BAcc) * BOUNDS_MAX_PARTS; }

void launch_bounds(const Ctx &c, hipStream_t s, int64_t n, const float *x, const float *y, const float *z,
                   const float *sigma, const float *ax, const float *ay, const float *az, bool with_alpha,
                   bool check_fp, double fp_ref, void *part, Bounds *res, Bounds *host) {
    BoundsArgs A{};
    A.x = x; A.y = y; A.z = z; A.s = sigma; A.ax = ax; A.ay = ay; A.az = az;
    A.n = n;
    A.with_alpha = with_alpha ? 1 : 0;
    A.periodic = c.prm.periodic;
    for (int d = 0; d < 3; ++d) {
        A.plo[d] = c.prm.box_lo[d];
        A.ref[d] = c.prm.periodic ? c.prm.box_lo[d] + 0.5 * c.prm.box_len : 0.0;
    }
    A.plen = c.prm.box_len;
    if (n <= BOUNDS_ONE_GROUP) {
        k_bounds_small<<<1, 1024, 0, s>>>(A, check_fp ? 1 : 0, fp_ref, res, host);
        VFMM_LAUNCH_CHECK();
        return;
    }
    const int nb = (int)std::min<int64_t>(BOUNDS_MAX_PARTS, std::max<int64_t>(1, cdiv(n, TPB)));
    k_bounds_partial<<<nb, TPB, 0, s>>>(A, (BAcc *)part);
    VFMM_LAUNCH_CHECK();
    k_bounds_final<<<1, TPB, 0, s>>>((const BAcc *)part, nb, check_fp ? 1 : 0, fp_ref, res, host);
    VFMM_LAUNCH_CHECK();
}

void compute_bounds(Ctx &c, int64_t n, const float *x, const float *y, const float *z, const float *sigma,
                    const float *ax, const float *ay, const float *az, bool with_alpha, bool to_host) {
    c.bpart.ensure(bounds_scratch_bytes());
    c.bres.ensure(sizeof(Bounds));
    // an evaluation checks its positions and cores against those of the build
    launch_bounds(c, c.stream, n, x, y, z, sigma, ax, ay, az, with_alpha, with_alpha, c.build_fp, c.bpart.ptr,
                  c.bres.as<Bounds>(), to_host ? reinterpret_cast<Bounds *>(pinned_ints(c)) : nullptr);
}

void sync_bounds(Ctx &c, Bounds *dst) {
    VFMM_HIP(hipStreamSynchronize(c.stream));
    std::memcpy(dst, c.hpin, sizeof(Bounds));
}

// ---------------------------------------------------------------------------
// Morton keys: 21 bits per axis, bit 3b+2 = x bit b, 3b+1 = y bit b, 3b = z bit b.
// ---------------------------------------------------------------------------
__device__ inline uint64_t spread3(uint32_t v) {
    uint64_t x = v & 0x1fffffu;
    x = (x | (x << 32)) & 0x1f00000000ffffull;
    x = (x | (x << 16)) & 0x1f0000ff0000ffull;
    x = (x | (x << 8)) & 0x100f00f00f00f00full;
    x = (x | (x << 4)) & 0x10c30c30c30c30c3ull;
    x = (x | (x << 2)) & 0x1249249249249249ull;
    return x;
}

// Batched problems: the problem id occupies the bits above 3*KL (KL key
// levels per axis), so each problem's particles stay contiguous after the
// sort and every problem gets its own root cube.
__global__ __launch_bounds__(TPB) void k_morton(const float *x, const float *y, const float *z, int64_t n,
                                                const RootBox *boxes, const int *pid, int KL, uint64_t *keys,
                                                uint32_t *vals) {
    const int64_t i = (int64_t)blockIdx.x * TPB + threadIdx.x;
    if (i >= n) return;
    const int b = pid ? pid[i] : 0;
    const RootBox box = boxes[b];
    const float cells = (float)(1u << KL);
    const float sc = cells / box.len;
    const float p[3] = {x[i], y[i], z[i]};
    uint32_t q[3];
    for (int d = 0; d < 3; ++d) {
        float t = floorf((p[d] - box.lo[d]) * sc);
        t = fminf(fmaxf(t, 0.0f), cells - 1.0f);
        q[d] = (uint32_t)t;
    }
    keys[i] = ((uint64_t)b << (3 * KL)) | (spread3(q[0]) << 2) | (spread3(q[1]) << 1) | spread3(q[2]);
    vals[i] = (uint32_t)i;
}

// problem id of every particle and per-problem bounding cubes
__global__ __launch_bounds__(TPB) void k_problem_ids(const int64_t *off, int *pid) {
    const int b = blockIdx.x;
    for (int64_t i = off[b] + threadIdx.x; i < off[b + 1]; i += TPB) pid[i] = b;
}

// a work-group of 16 waves per problem, four loads of each coordinate in flight
// (64 problems of 15,500 particles: 72 us with four waves and one load, now 9)
__global__ __launch_bounds__(1024) void k_problem_boxes(const int64_t *off, const float *x, const float *y,
                                                        const float *z, RootBox *boxes) {
    __shared__ float lo[3][16], hi[3][16];
    const int b = blockIdx.x;
    const int64_t i1 = off[b + 1];
    float l[3] = {3.4e38f, 3.4e38f, 3.4e38f}, h[3] = {-3.4e38f, -3.4e38f, -3.4e38f};
    for (int64_t i = off[b] + threadIdx.x; i < i1; i += 4 * 1024) {
        float p[4][3];
#pragma unroll
        for (int u = 0; u < 4; ++u) {  // past the end: the thread's first particle again
            const int64_t k = i + 1024 * u < i1 ? i + 1024 * u : i;
            p[u][0] = x[k];
            p[u][1] = y[k];
            p[u][2] = z[k];
        }
#pragma unroll
        for (int u = 0; u < 4; ++u)
            for (int d = 0; d < 3; ++d) { l[d] = fminf(l[d], p[u][d]); h[d] = fmaxf(h[d], p[u][d]); }
    }
    auto wave_bounds = [&](int lanes) {
        for (int o = lanes / 2; o > 0; o >>= 1)
            for (int d = 0; d < 3; ++d) {
                l[d] = fminf(l[d], __shfl_xor(l[d], o, 64));
                h[d] = fmaxf(h[d], __shfl_xor(h[d], o, 64));
            }
    };
    wave_bounds(64);
    if ((threadIdx.x & 63) == 0)
        for (int d = 0; d < 3; ++d) { lo[d][threadIdx.x >> 6] = l[d]; hi[d][threadIdx.x >> 6] = h[d]; }
    __syncthreads();
    if (threadIdx.x < 64) {
        for (int d = 0; d < 3; ++d) { l[d] = lo[d][threadIdx.x & 15]; h[d] = hi[d][threadIdx.x & 15]; }
        wave_bounds(16);
    }
    if (threadIdx.x == 0) {
        float len = 0.f, c[3];
        for (int d = 0; d < 3; ++d) {
            len = fmaxf(len, h[d] - l[d]);
            c[d] = 0.5f * (l[d] + h[d]);
        }
        len = len * (1.0f + 1e-5f) + 1e-6f * fmaxf(fabsf(c[0]), fmaxf(fabsf(c[1]), fabsf(c[2]))) + 1e-30f;
        RootBox r;
        for (int d = 0; d < 3; ++d) r.lo[d] = c[d] - 0.5f * len;
        r.len = len;
        boxes[b] = r;
    }
}

// ---------------------------------------------------------------------------
// Stable LSD radix sort of (uint64 key, uint32 value), 8-bit digits.
// A wave takes consecutive items, 64 at a time, and ranks equal digits with
// ballots over the digit's bits after a running count per digit of its own, so
// equal digits keep their input order (stable, deterministic) and the waves meet
// only once per pass, to add up their counts.
// ---------------------------------------------------------------------------
// orders a wave's own LDS accesses (no other wave touches the counts meanwhile)
__device__ __forceinline__ void wave_fence() {
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
}

// off[r] = items of this wave before item r (of this lane) with the same digit;
// cnt[256]: the wave's counts per digit
template <int ITEMS>
__device__ __forceinline__ void rank_digits(const uint64_t *key, const bool *valid, int shift, int *cnt, int *off) {
    const int lane = threadIdx.x & 63;
    for (int j = lane; j < 256; j += 64) cnt[j] = 0;
    wave_fence();
    const uint64_t lt = (lane == 0) ? 0ull : ((~0ull) >> (64 - lane));
#pragma unroll
    for (int r = 0; r < ITEMS; ++r) {
        const int d = (int)((key[r] >> shift) & 255);
        uint64_t m = __ballot(valid[r]);
#pragma unroll
        for (int b = 0; b < 8; ++b) {
            const uint64_t mb = __ballot((d >> b) & 1);
            m &= ((d >> b) & 1) ? mb : ~mb;
        }
        const int rank = __popcll(m & lt), prev = cnt[d];
        wave_fence();
        if (valid[r] && rank == 0) cnt[d] = prev + __popcll(m);
        wave_fence();
        off[r] = prev + rank;
    }
}

// exclusive sum of v over the 256 threads t = 0 .. 255 (four whole waves; every
// thread of the work-group calls it); sh: int[4]
__device__ __forceinline__ int scan_256(int v, int t, int *sh) {
    int incl = v;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
        const int u = __shfl_up(incl, o, 64);
        if ((t & 63) >= o) incl += u;
    }
    if (t < 256 && (t & 63) == 63) sh[t >> 6] = incl;
    __syncthreads();
    int base = 0;
    if (t < 256)
        for (int w = 0; w < (t >> 6); ++w) base += sh[w];
    return base + incl - v;
}

// Up to RS_GROUP items: all passes in one work-group, the items in registers and
// exchanged through LDS.  A pass over several work-groups is a histogram, a scan
// and a scatter, 3 launches of 2 to 11 us each for 3,000 items; here it is about 3 us.
static constexpr int RS_GROUP = 8192;

template <int ITEMS>
__global__ __launch_bounds__(1024) void k_rs_group(uint64_t *key, uint32_t *val, int n, int passes) {
    __shared__ uint64_t buf[1024 * ITEMS];
    __shared__ int cnt[16][256];
    __shared__ int sh[4];
    const int t = threadIdx.x, lane = t & 63, w = t >> 6;
    const int i0 = w * 64 * ITEMS + lane;
    uint64_t k[ITEMS];
    uint32_t v[ITEMS];
    int off[ITEMS];
    bool valid[ITEMS];
#pragma unroll
    for (int r = 0; r < ITEMS; ++r) {  // padded with the largest key: stays behind the items
        const int i = i0 + 64 * r;
        valid[r] = true;
        k[r] = i < n ? key[i] : ~0ull;
        v[r] = i < n ? val[i] : 0u;
    }
    for (int p = 0; p < passes; ++p) {
        const int shift = 8 * p;
        rank_digits<ITEMS>(k, valid, shift, cnt[w], off);
        __syncthreads();
        int c[16], tot = 0;
        if (t < 256) {
#pragma unroll
            for (int j = 0; j < 16; ++j) c[j] = cnt[j][t];
#pragma unroll
            for (int j = 0; j < 16; ++j) tot += c[j];
        }
        int base = scan_256(tot, t, sh);
        if (t < 256) {
#pragma unroll
            for (int j = 0; j < 16; ++j) {
                cnt[j][t] = base;
                base += c[j];
            }
        }
        __syncthreads();
#pragma unroll
        for (int r = 0; r < ITEMS; ++r) {
            off[r] += cnt[w][(int)((k[r] >> shift) & 255)];
            buf[off[r]] = k[r];
        }
        __syncthreads();
#pragma unroll
        for (int r = 0; r < ITEMS; ++r) k[r] = buf[i0 + 64 * r];
        __syncthreads();
        uint32_t *vb = reinterpret_cast<uint32_t *>(buf);
#pragma unroll
        for (int r = 0; r < ITEMS; ++r) vb[off[r]] = v[r];
        __syncthreads();
#pragma unroll
        for (int r = 0; r < ITEMS; ++r) v[r] = vb[i0 + 64 * r];
        __syncthreads();
    }
#pragma unroll
    for (int r = 0; r < ITEMS; ++r) {
        const int i = i0 + 64 * r;
        if (i < n) {
            key[i] = k[r];
            val[i] = v[r];
        }
    }
}

// Larger sorts: tiles of 256 * ITEMS items.  Up to RS_ROWS tiles the scatter sums
// the histograms (one row of 256 per tile) itself; more are scanned digit by digit
// in launches between the two (SCANNED).  The tile's items are put in order in LDS
// first, so that a digit's run leaves in consecutive addresses.
static constexpr int RS_ROWS = 64;

template <bool SCANNED>
__global__ __launch_bounds__(TPB) void k_rs_hist(const uint64_t *keys, int64_t n, int shift, int items, int *hist) {
    __shared__ int h[256];
    h[threadIdx.x] = 0;
    __syncthreads();
    const int64_t base = (int64_t)blockIdx.x * items * TPB;
    for (int i = 0; i < items; ++i) {
        const int64_t k = base + (int64_t)i * TPB + threadIdx.x;
        if (k < n) atomicAdd(&h[(keys[k] >> shift) & 255], 1);
    }
    __syncthreads();
    hist[SCANNED ? (size_t)threadIdx.x * gridDim.x + blockIdx.x : (size_t)blockIdx.x * 256 + threadIdx.x] =
        h[threadIdx.x];
}

template <int ITEMS, bool SCANNED>
__global__ __launch_bounds__(TPB) void k_rs_scatter(const uint64_t *kin, const uint32_t *vin, uint64_t *kout,
                                                    uint32_t *vout, int64_t n, int shift, const int *offs) {
    __shared__ uint64_t lk[TPB * ITEMS];
    __shared__ uint32_t lv[TPB * ITEMS];
    __shared__ int cnt[TPB / 64][256];
    __shared__ int dst[256];
    __shared__ int sh[2][4];
    const int t = threadIdx.x, lane = t & 63, w = t >> 6;
    const int64_t base = (int64_t)blockIdx.x * (TPB * ITEMS);
    uint64_t k[ITEMS];
    uint32_t v[ITEMS];
    int off[ITEMS];
    bool valid[ITEMS];
#pragma unroll
    for (int r = 0; r < ITEMS; ++r) {
        const int64_t i = base + w * 64 * ITEMS + 64 * r + lane;
        valid[r] = i < n;
        k[r] = valid[r] ? kin[i] : 0ull;
        v[r] = valid[r] ? vin[i] : 0u;
    }
    int gbase;  // output position of the tile's first item of digit t
    if (SCANNED) {
        gbase = offs[(size_t)t * gridDim.x + blockIdx.x];
    } else {
        int before = 0, total = 0;
        for (int b0 = 0; b0 < (int)gridDim.x; b0 += 16) {
            int h[16];
#pragma unroll
            for (int j = 0; j < 16; ++j) h[j] = b0 + j < (int)gridDim.x ? offs[(b0 + j) * 256 + t] : 0;
#pragma unroll
            for (int j = 0; j < 16; ++j) {
                total += h[j];
                before += b0 + j < (int)blockIdx.x ? h[j] : 0;
            }
        }
        gbase = scan_256(total, t, sh[0]) + before;
    }
    rank_digits<ITEMS>(k, valid, shift, cnt[w], off);
    __syncthreads();
    int c[TPB / 64], tot = 0;
#pragma unroll
    for (int j = 0; j < TPB / 64; ++j) {
        c[j] = cnt[j][t];
        tot += c[j];
    }
    int lbase = scan_256(tot, t, sh[1]);
    dst[t] = gbase - lbase;
#pragma unroll
    for (int j = 0; j < TPB / 64; ++j) {
        cnt[j][t] = lbase;
        lbase += c[j];
    }
    __syncthreads();
#pragma unroll
    for (int r = 0; r < ITEMS; ++r) {
        if (!valid[r]) continue;
        const int o = off[r] + cnt[w][(int)((k[r] >> shift) & 255)];
        lk[o] = k[r];
        lv[o] = v[r];
    }
    __syncthreads();
    const int m = (int)min((int64_t)(TPB * ITEMS), n - base);
#pragma unroll
    for (int r = 0; r < ITEMS; ++r) {
        const int i = r * TPB + t;
        if (i >= m) continue;
        const uint64_t key = lk[i];
        const int o = dst[(int)((key >> shift) & 255)] + i;
        kout[o] = key;
        vout[o] = lv[i];
    }
}

template <int ITEMS, bool SCANNED>
static void rs_pass(Ctx &c, const DevBuf &kA, const DevBuf &vA, const DevBuf &kB, const DevBuf &vB, int64_t n,
                    int shift) {
    const int nblk = (int)cdiv(n, TPB * ITEMS);
    int *hist = c.hist.as<int>();
    k_rs_hist<SCANNED><<<nblk, TPB, 0, c.stream>>>(kA.as<uint64_t>(), n, shift, ITEMS, hist);
    VFMM_LAUNCH_CHECK();
    if (SCANNED) scan_excl_i32(c, hist, hist, 256LL * nblk);
    k_rs_scatter<ITEMS, SCANNED><<<nblk, TPB, 0, c.stream>>>(kA.as<uint64_t>(), vA.as<uint32_t>(), kB.as<uint64_t>(),
                                                             vB.as<uint32_t>(), n, shift, hist);
    VFMM_LAUNCH_CHECK();
}

// Sorts keyA/valA (n items, significant bits [0, nbits)); result ends in keyA/valA.
static void radix_sort(Ctx &c, DevBuf &kA, DevBuf &vA, DevBuf &kB, DevBuf &vB, int64_t n, int nbits) {
    if (n <= 1) return;
    const int passes = (nbits + 7) / 8;
    if (n <= RS_GROUP) {
        uint64_t *k = kA.as<uint64_t>();
        uint32_t *v = vA.as<uint32_t>();
        if (n <= 1024)
            k_rs_group<1><<<1, 1024, 0, c.stream>>>(k, v, (int)n, passes);
        else if (n <= 4096)
            k_rs_group<4><<<1, 1024, 0, c.stream>>>(k, v, (int)n, passes);
        else
            k_rs_group<8><<<1, 1024, 0, c.stream>>>(k, v, (int)n, passes);
        VFMM_LAUNCH_CHECK();
        return;
    }
    kB.ensure(sizeof(uint64_t) * n);
    vB.ensure(sizeof(uint32_t) * n);
    c.hist.ensure(sizeof(int) * 256 * (size_t)std::max<int64_t>(RS_ROWS, cdiv(n, 16 * TPB)));
    for (int p = 0; p < passes; ++p) {
        if (n <= RS_ROWS * 4 * TPB)
            rs_pass<4, false>(c, kA, vA, kB, vB, n, 8 * p);
        else if (n <= RS_ROWS * 8 * TPB)
            rs_pass<8, false>(c, kA, vA, kB, vB, n, 8 * p);
        else if (n <= RS_ROWS * 16 * TPB)
            rs_pass<16, false>(c, kA, vA, kB, vB, n, 8 * p);
        else
            rs_pass<16, true>(c, kA, vA, kB, vB, n, 8 * p);
        std::swap(kA, kB);
        std::swap(vA, vB);
    }
}

void sort_pairs_u64(Ctx &c, DevBuf &kA, DevBuf &vA, DevBuf &kB, DevBuf &vB, int64_t n, int nbits) {
    radix_sort(c, kA, vA, kB, vB, n, nbits);
}

// ---------------------------------------------------------------------------
// Gather into Morton order.
// ---------------------------------------------------------------------------
__global__ __launch_bounds__(TPB) void k_gather_pos(const uint32_t *perm, int64_t n, const float *x, const float *y,
                                                    const float *z, const float *s, float4 *rec, int *perm_out) {
    const int64_t i = (int64_t)blockIdx.x * TPB + threadIdx.x;
    if (i >= n) return;
    const uint32_t j = perm[i];
    rec[2 * i] = make_float4(x[j], y[j], z[j], s[j]);
    perm_out[i] = (int)j;
}

__global__ __launch_bounds__(TPB) void k_gather_alpha(const int *perm, int64_t n, const float *ax, const float *ay,
                                                      const float *az, float4 *rec) {
    const int64_t i = (int64_t)blockIdx.x * TPB + threadIdx.x;
    if (i >= n) return;
    const int j = perm[i];
    const float k = 0.0795774715459476679f;  // 1/(4 pi): the Green's function factor of G
    rec[2 * i + 1] = make_float4(ax[j] * k, ay[j] * k, az[j] * k, 0.0f);
}

void gather_strengths(Ctx &c, const float *ax, const float *ay, const float *az, const float *) {
    if (c.n == 0) return;
    k_gather_alpha<<<cdiv(c.n, TPB), TPB, 0, c.stream>>>(c.perm.as<int>(), c.n, ax, ay, az, c.rec.as<float4>());
    VFMM_LAUNCH_CHECK();
}

// float64 records for the float64 form: positions from the sorted float32
// records (exact), c^2 and c^3 with c = 1/(sqrt 2 sigma) of each core, strengths
// from the caller's arrays scaled in float64
__global__ __launch_bounds__(TPB) void k_gather_rec64(const int *perm, int64_t n, const float *ax, const float *ay,
                                                      const float *az, const float4 *rec, double4 *rec64) {
    const int64_t i = (int64_t)blockIdx.x * TPB + threadIdx.x;
    if (i >= n) return;
    const int j = perm[i];
    const double k = 0.079577471545947667884;  // 1/(4 pi)
    const float4 p = rec[2 * i];
    const double c = 0.70710678118654752440 / (double)p.w;  // 1/(sqrt 2 sigma)
    rec64[2 * i] = make_double4(p.x, p.y, p.z, c * c);
    rec64[2 * i + 1] = make_double4((double)ax[j] * k, (double)ay[j] * k, (double)az[j] * k, c * c * c);
}

void gather_records64(Ctx &c, const float *ax, const float *ay, const float *az) {
    if (c.n == 0) return;
    c.rec64.ensure(sizeof(double4) * 2 * (size_t)c.n);
    k_gather_rec64<<<cdiv(c.n, TPB), TPB, 0, c.stream>>>(c.perm.as<int>(), c.n, ax, ay, az, c.rec.as<float4>(),
                                                         c.rec64.as<double4>());
    VFMM_LAUNCH_CHECK();
}

// ---------------------------------------------------------------------------
// Separate target points: within every leaf the sources (caller index below
// n_src) are moved in front of the targets (a stable partition of the leaf's
// range, which leaves every cell's range unchanged), and each leaf records
// its number of sources, so that the near field never reads a target as a
// source.  One thread per leaf writes the new order of its range.
// ---------------------------------------------------------------------------
__global__ __launch_bounds__(TPB) void k_leaf_partition(int nl, const int *leaves, const int *start, const int *count,
                                                        const int *perm, int64_t n_src, uint32_t *order,
                                                        int *nsrc) {
    const int l = blockIdx.x * TPB + threadIdx.x;
    if (l >= nl) return;
    const int cell = leaves[l];
    const int s0 = start[cell], cnt = count[cell];
    int w = s0;
    for (int i = s0; i < s0 + cnt; ++i)
        if (perm[i] < n_src) order[w++] = (uint32_t)i;
    nsrc[cell] = w - s0;
    for (int i = s0; i < s0 + cnt; ++i)
        if (perm[i] >= n_src) order[w++] = (uint32_t)i;
}

__global__ __launch_bounds__(TPB) void k_apply_order(int64_t n, const uint32_t *order, const int *perm_in,
                                                     const float4 *rec_in, const uint64_t *key_in, int *perm_out,
                                                     float4 *pos_out, uint64_t *key_out) {
    const int64_t i = (int64_t)blockIdx.x * TPB + threadIdx.x;
    if (i >= n) return;
    const uint32_t j = order[i];
    perm_out[i] = perm_in[j];
    pos_out[i] = rec_in[2 * (size_t)j];
    key_out[i] = key_in[j];
}

void partition_sources(Ctx &c, int64_t n_src) {
    hipStream_t s = c.stream;
    const int64_t n = c.n;
    c.c_nsrc.ensure(sizeof(int) * (size_t)c.ncells);
    VFMM_HIP(hipMemsetAsync(c.c_nsrc.ptr, 0, sizeof(int) * (size_t)c.ncells, s));
    c.valB.ensure(sizeof(uint32_t) * n);
    c.keyB.ensure(sizeof(uint64_t) * n);
    c.part.ensure(sizeof(int) * n + 16 + sizeof(float4) * n);
    uint32_t *order = c.valB.as<uint32_t>();
    k_leaf_partition<<<cdiv(c.nleaves, TPB), TPB, 0, s>>>(c.nleaves, c.leaves.as<int>(), c.c_start.as<int>(),
                                                           c.c_count.as<int>(), c.perm.as<int>(), n_src, order,
                                                           c.c_nsrc.as<int>());
    VFMM_LAUNCH_CHECK();
    // gather into scratch, then copy back (perm, position records, keys)
    int *perm2 = c.part.as<int>();
    float4 *rec2 = reinterpret_cast<float4 *>(c.part.as<char>() + ((sizeof(int) * n + 15) / 16) * 16);
    k_apply_order<<<cdiv(n, TPB), TPB, 0, s>>>(n, order, c.perm.as<int>(), c.rec.as<float4>(), c.keyA.as<uint64_t>(),
                                                perm2, rec2, c.keyB.as<uint64_t>());
    VFMM_LAUNCH_CHECK();
    VFMM_HIP(hipMemcpyAsync(c.perm.ptr, perm2, sizeof(int) * n, hipMemcpyDeviceToDevice, s));
    VFMM_HIP(hipMemcpy2DAsync(c.rec.ptr, 2 * sizeof(float4), rec2, sizeof(float4), sizeof(float4), n,
                              hipMemcpyDeviceToDevice, s));
    VFMM_HIP(hipMemcpyAsync(c.keyA.ptr, c.keyB.ptr, sizeof(uint64_t) * n, hipMemcpyDeviceToDevice, s));
}

// ---------------------------------------------------------------------------
// Octree, level by level.  A cell at level l holds a contiguous range of the
// sorted keys sharing their top 3l bits; it is split while it holds more than
// ncrit particles and l < 21.  Children of a cell are contiguous.
// ---------------------------------------------------------------------------
__device__ inline int octant_at(uint64_t key, int lchild, int KL) { return (int)((key >> (3 * (KL - lchild))) & 7); }

// Eight lanes per cell, one per octant o: the end of octant o's run in the
// cell's key range (the first index whose octant is > o) by a binary search;
// the octants are non-decreasing along the range, so the cell's children are
// the non-empty runs, in octant order.  The lanes of a cell are consecutive
// lanes of one wave.
__device__ inline int octant_end(const uint64_t *keys, int s, int end, int o, int lchild, int KL) {
    int a = s, b = end;
    while (a < b) {
        const int mid = (a + b) >> 1;
        if (octant_at(keys[mid], lchild, KL) <= o) a = mid + 1; else b = mid;
    }
    return a;
}

__global__ __launch_bounds__(TPB) void k_count_children(int c0, int c1, int lvl, int ncrit, int KL, const int *start,
                                                        const int *count, const uint64_t *keys, int *nchild,
                                                        Bounds *res) {
    const int g = blockIdx.x * TPB + threadIdx.x;
    const int cell = c0 + g / 8, o = g % 8;
    const bool valid = cell < c1;
    const int s = valid ? start[cell] : 0, cnt = valid ? count[cell] : 0;
    // keys resolve no finer than level KL: such a leaf keeps all its particles
    // (coincident or nearly coincident ones), which the near field handles
    if (valid && o == 0 && cnt > ncrit && lvl >= KL) atomicAdd(&res->overfull, 1);
    const bool split = valid && cnt > ncrit && lvl < KL;
    const int e = split ? octant_end(keys, s, s + cnt, o, lvl + 1, KL) : s;
    const int prev = __shfl_up(e, 1, 8);
    const bool nonempty = split && e > (o == 0 ? s : prev);
    const unsigned long long bal = __ballot(nonempty);
    const int sh = (threadIdx.x & 63) & ~7;
    if (valid && o == 0) nchild[cell - c0] = __popcll((bal >> sh) & 0xffull);
}

__global__ __launch_bounds__(TPB) void k_make_children(int c0, int c1, int lvl, int cnext, int KL, const int *start,
                                                       const int *count, const uint64_t *keys, const int *choff,
                                                       const int *nchild_l, int *c_start, int *c_count,
                                                       int *c_parent, int *c_child, int *c_nchild, int *c_level) {
    const int g = blockIdx.x * TPB + threadIdx.x;
    const int cell = c0 + g / 8, o = g % 8;
    const bool valid = cell < c1;
    const int nc = valid ? nchild_l[cell - c0] : 0;
    const int s = valid ? start[cell] : 0, end = valid ? s + count[cell] : 0;
    const int e = nc > 0 ? octant_end(keys, s, end, o, lvl + 1, KL) : s;
    const int prev = __shfl_up(e, 1, 8);
    const int lo = o == 0 ? s : prev;
    const bool nonempty = nc > 0 && e > lo;
    const unsigned long long bal = __ballot(nonempty);
    const int sh = (threadIdx.x & 63) & ~7;
    const int first = valid ? cnext + choff[cell - c0] : 0;
    if (valid && o == 0) {
        c_nchild[cell] = nc;
        c_child[cell] = nc == 0 ? -1 : first;
    }
    if (nonempty) {
        const int ch = first + __popcll((bal >> sh) & ((1ull << o) - 1));  // non-empty octants before o
        c_start[ch] = lo;
        c_count[ch] = e - lo;
        c_parent[ch] = cell;
        c_level[ch] = lvl + 1;
    }
}

// The top levels in one work-group, while a level has at most TREE_GROUP cells:
// per level one launch instead of a count, a scan, a wait for the total and a
// write (25 us), and for a small tree the leaf list too (3,000 particles: 16
// launches and 4 waits, 110 us, become one launch and one wait).  Each of the
// 1,024 threads takes an octant of a cell, 128 cells at a time; a child's place is
// the number of non-empty octants before it.
static constexpr int TREE_GROUP = 512;

struct TreeGroupArgs {
    const uint64_t *keys;
    const int64_t *off;  // batched problems: first particle of each (else null)
    int nroot, n, ncrit, KL;
    int cap;  // cells that the arrays hold
    int *start, *count, *parent, *child, *nchild, *level, *leaves;
    Bounds *res;
    // pinned: [0] whether the tree is complete, [1] level offsets, [2] leaves,
    // [3] leaves over ncrit, [4 ...] the offsets
    int *host;
};

__global__ __launch_bounds__(1024) void k_tree_group(TreeGroupArgs T) {
    __shared__ int wsum[16];
    __shared__ int sh_over;
    const int t = threadIdx.x, lane = t & 63, w = t >> 6, o = t & 7;
    for (int b = t; b < T.nroot; b += 1024) {
        T.start[b] = T.off ? (int)T.off[b] : 0;
        T.count[b] = T.off ? (int)(T.off[b + 1] - T.off[b]) : T.n;
        T.parent[b] = -1;
        T.level[b] = 0;
    }
    if (t == 0) {
        sh_over = 0;
        T.host[4] = 0;
        T.host[5] = T.nroot;
    }
    __syncthreads();
    // this wave's sum of the lower waves' counts, and the total
    auto add_up = [&](int mine, int &pre) {
        if (lane == 0) wsum[w] = mine;
        __syncthreads();
        int tot = 0;
        pre = 0;
#pragma unroll
        for (int j = 0; j < 16; ++j) {
            const int v = wsum[j];
            pre += j < w ? v : 0;
            tot += v;
        }
        __syncthreads();
        return tot;
    };
    int c0 = 0, c1 = T.nroot, lvl = 0, done = 0, over = 0;
    while (c1 - c0 <= TREE_GROUP) {
        int next = c1, level_over = 0;
        bool fits = true;
        for (int base = c0; base < c1; base += 128) {
            const int cell = base + t / 8;
            const bool valid = cell < c1;
            const int s = valid ? T.start[cell] : 0, cnt = valid ? T.count[cell] : 0;
            const bool big = valid && cnt > T.ncrit, split = big && lvl < T.KL;
            // keys resolve no finer than level KL: such a leaf keeps all its particles
            if (big && !split && o == 0) ++level_over;
            const int e = split ? octant_end(T.keys, s, s + cnt, o, lvl + 1, T.KL) : s;
            const int prev = __shfl_up(e, 1, 8);
            const int lo = o == 0 ? s : prev;
            const bool nonempty = split && e > lo;
            const unsigned long long bal = __ballot(nonempty);
            int pre;
            const int tot = add_up(__popcll(bal), pre);
            if (next + tot > T.cap) {  // the caller grows the arrays and repeats the level
                fits = false;
                break;
            }
            const int sh = lane & ~7;
            const int first = next + pre + __popcll(bal & ((1ull << sh) - 1));
            const unsigned mine = (unsigned)(bal >> sh) & 0xffu;
            if (valid && o == 0) {
                T.nchild[cell] = __popc(mine);
                T.child[cell] = mine == 0 ? -1 : first;
            }
            if (nonempty) {
                const int ch = first + __popc(mine & ((1u << o) - 1));
                T.start[ch] = lo;
                T.count[ch] = e - lo;
                T.parent[ch] = cell;
                T.level[ch] = lvl + 1;
            }
            next += tot;
        }
        if (!fits) break;
        over += level_over;
        __syncthreads();  // the children are read by other threads
        if (next == c1) {
            done = 1;
            break;
        }
        c0 = c1;
        c1 = next;
        ++lvl;
        if (t == 0) T.host[5 + lvl] = next;
    }
    if (over) atomicAdd(&sh_over, over);
    int leaves = 0;
    if (done)
        for (int base = 0; base < c1; base += 1024) {
            const int cell = base + t;
            const bool leaf = cell < c1 && T.nchild[cell] == 0;
            const unsigned long long bal = __ballot(leaf);
            int pre;
            const int tot = add_up(__popcll(bal), pre);
            if (leaf) T.leaves[leaves + pre + __popcll(bal & ((1ull << lane) - 1))] = cell;
            leaves += tot;
        }
    __syncthreads();
    if (t == 0) {
        T.res->overfull = sh_over;
        T.host[0] = done;
        T.host[1] = lvl + 2;
        T.host[2] = leaves;
        T.host[3] = sh_over;
    }
}

// Centres from the key prefix of the first particle; leaves get their tight
// radius (max distance of a particle from the cube centre) and bounding box.
// Sixteen lanes per cell: one thread per leaf reads its records one after
// another, 32 bytes apart (140 us for 64 rings of 1,000 particles each with 64
// per leaf, 24 us for 3,000 particles; now 12 and 5).
static constexpr int GEO_LANES = 16;

__global__ __launch_bounds__(TPB) void k_leaf_geometry(int ncell, const RootBox *boxes, int KL, const int *start,
                                                       const int *count,
                                                       const int *level, const int *nchild, const uint64_t *keys,
                                                       const float4 *rec, float4 *geo, double4 *geo64, float *rad,
                                                       float4 *blo, float4 *bhi) {
    const int cell = blockIdx.x * (TPB / GEO_LANES) + threadIdx.x / GEO_LANES, sub = threadIdx.x % GEO_LANES;
    if (cell >= ncell) return;
    const int lvl = level[cell];
    const int s = start[cell];
    const uint64_t key = keys[s];
    const RootBox box = boxes[(int)(key >> (3 * KL))];
    // cell integer coordinates at this level
    uint32_t q[3] = {0, 0, 0};
    for (int b = 0; b < lvl; ++b) {
        const int o = octant_at(key, b + 1, KL);
        q[0] = (q[0] << 1) | ((o >> 2) & 1);
        q[1] = (q[1] << 1) | ((o >> 1) & 1);
        q[2] = (q[2] << 1) | (o & 1);
    }
    const double size = (double)box.len / (double)(1u << lvl);
    const double c[3] = {box.lo[0] + (q[0] + 0.5) * size, box.lo[1] + (q[1] + 0.5) * size,
                         box.lo[2] + (q[2] + 0.5) * size};
    const float4 g = make_float4((float)c[0], (float)c[1], (float)c[2], (float)size);
    if (sub == 0) {
        geo[cell] = g;
        // the acceptance test knows the float32 centres: where they are off by more than 1/256
        // of the cell (cells of about 128 float32 steps), expansions are about them too
        const double near = size / 256.0;
        geo64[cell] = make_double4(fabs(g.x - c[0]) <= near ? c[0] : g.x, fabs(g.y - c[1]) <= near ? c[1] : g.y,
                                   fabs(g.z - c[2]) <= near ? c[2] : g.z, size);
    }
    if (nchild[cell] != 0) return;
    float r2 = 0.f;
    float4 lo = make_float4(3.4e38f, 3.4e38f, 3.4e38f, 0.f), hi = make_float4(-3.4e38f, -3.4e38f, -3.4e38f, 0.f);
    const int end = s + count[cell];
    for (int i = s + sub; i < end; i += GEO_LANES) {
        const float4 p = rec[2 * (size_t)i];
        const float dx = p.x - g.x, dy = p.y - g.y, dz = p.z - g.z;
        r2 = fmaxf(r2, dx * dx + dy * dy + dz * dz);
        lo.x = fminf(lo.x, p.x); lo.y = fminf(lo.y, p.y); lo.z = fminf(lo.z, p.z);
        hi.x = fmaxf(hi.x, p.x); hi.y = fmaxf(hi.y, p.y); hi.z = fmaxf(hi.z, p.z);
        hi.w = fmaxf(hi.w, p.w);  // the cell's largest core
    }
#pragma unroll
    for (int o = GEO_LANES / 2; o > 0; o >>= 1) {
        r2 = fmaxf(r2, __shfl_xor(r2, o, GEO_LANES));
        lo.x = fminf(lo.x, __shfl_xor(lo.x, o, GEO_LANES));
        lo.y = fminf(lo.y, __shfl_xor(lo.y, o, GEO_LANES));
        lo.z = fminf(lo.z, __shfl_xor(lo.z, o, GEO_LANES));
        hi.x = fmaxf(hi.x, __shfl_xor(hi.x, o, GEO_LANES));
        hi.y = fmaxf(hi.y, __shfl_xor(hi.y, o, GEO_LANES));
        hi.z = fmaxf(hi.z, __shfl_xor(hi.z, o, GEO_LANES));
        hi.w = fmaxf(hi.w, __shfl_xor(hi.w, o, GEO_LANES));
    }
    if (sub != 0) return;
    // round the radius up by a few ulps so float rounding never makes it short
    rad[cell] = sqrtf(r2) * (1.0f + 4.0e-7f);
    blo[cell] = lo;
    bhi[cell] = hi;
}

// Internal cells, one level at a time bottom-up: radius bounded by the
// children's spheres, bounding box the union of the children's boxes, largest
// core (the box's fourth component) the largest of the children's.
__device__ inline void internal_geometry(int cell, const int *child, const int *nchild, const float4 *geo, float *rad,
                                         float4 *blo, float4 *bhi) {
    const int nc = nchild[cell];
    if (nc == 0) return;
    const float4 g = geo[cell];
    float r = 0.f;
    float4 lo = make_float4(3.4e38f, 3.4e38f, 3.4e38f, 0.f), hi = make_float4(-3.4e38f, -3.4e38f, -3.4e38f, 0.f);
    const int f = child[cell];
    for (int k = 0; k < nc; ++k) {
        const float4 cg = geo[f + k];
        const float dx = cg.x - g.x, dy = cg.y - g.y, dz = cg.z - g.z;
        r = fmaxf(r, sqrtf(dx * dx + dy * dy + dz * dz) + rad[f + k]);
        const float4 cl = blo[f + k], chh = bhi[f + k];
        lo.x = fminf(lo.x, cl.x); lo.y = fminf(lo.y, cl.y); lo.z = fminf(lo.z, cl.z);
        hi.x = fmaxf(hi.x, chh.x); hi.y = fmaxf(hi.y, chh.y); hi.z = fmaxf(hi.z, chh.z);
        hi.w = fmaxf(hi.w, chh.w);
    }
    rad[cell] = r * (1.0f + 4.0e-7f);
    blo[cell] = lo;
    bhi[cell] = hi;
}

__global__ __launch_bounds__(TPB) void k_internal_geometry(int c0, int c1, const int *child, const int *nchild,
                                                           const float4 *geo, float *rad, float4 *blo, float4 *bhi) {
    const int cell = c0 + blockIdx.x * TPB + threadIdx.x;
    if (cell < c1) internal_geometry(cell, child, nchild, geo, rad, blo, bhi);
}

// all levels of a tree of at most TREE_GEO_GROUP cells in one work-group
static constexpr int TREE_GEO_GROUP = 2048;

struct LevelOffsets {
    int v[26];
};

__global__ __launch_bounds__(1024) void k_internal_geometry_group(LevelOffsets L, int depth, const int *child,
                                                                  const int *nchild, const float4 *geo, float *rad,
                                                                  float4 *blo, float4 *bhi) {
    for (int l = depth - 1; l >= 0; --l) {
        for (int cell = L.v[l] + threadIdx.x; cell < L.v[l + 1]; cell += 1024)
            internal_geometry(cell, child, nchild, geo, rad, blo, bhi);
        __syncthreads();
    }
}

__global__ __launch_bounds__(TPB) void k_leaf_flags(int ncell, const int *nchild, int *flag) {
    const int cell = blockIdx.x * TPB + threadIdx.x;
    if (cell < ncell) flag[cell] = nchild[cell] == 0 ? 1 : 0;
}

__global__ __launch_bounds__(TPB) void k_leaf_compact(int ncell, const int *nchild, const int *pos, int *leaves) {
    const int cell = blockIdx.x * TPB + threadIdx.x;
    if (cell < ncell && nchild[cell] == 0) leaves[pos[cell]] = cell;
}

__global__ __launch_bounds__(TPB) void k_roots(int nprob, const int64_t *off, int n, int *start, int *count,
                                               int *parent, int *level) {
    const int b = blockIdx.x * TPB + threadIdx.x;
    if (b >= nprob) return;
    start[b] = off ? (int)off[b] : 0;
    count[b] = off ? (int)(off[b + 1] - off[b]) : n;
    parent[b] = -1;
    level[b] = 0;
}

// grow a cell array keeping its first `used` elements
static void grow_keep(Ctx &c, DevBuf &b, size_t bytes, size_t used) {
    if (bytes <= b.cap) return;
    DevBuf nb;
    nb.ensure(bytes * 2);
    if (used) VFMM_HIP(hipMemcpyAsync(nb.ptr, b.ptr, used, hipMemcpyDeviceToDevice, c.stream));
    VFMM_HIP(hipStreamSynchronize(c.stream));
    b.release();
    b = nb;
}

void build_tree(Ctx &c, int64_t n, const float *x, const float *y, const float *z, const float *sigma) {
    hipStream_t s = c.stream;
    // ---- Morton keys and sort ----
    c.keyA.ensure(sizeof(uint64_t) * n);
    c.valA.ensure(sizeof(uint32_t) * n);
    const int nprob = c.nprob;
    int pbits = 0;
    while ((1 << pbits) < nprob) ++pbits;
    c.key_levels = nprob > 1 ? (63 - pbits) / 3 : 21;
    const int KL = c.key_levels;
    c.pbox.ensure(sizeof(RootBox) * (size_t)nprob);
    int *pid = nullptr;
    if (nprob > 1) {
        c.pid.ensure(sizeof(int) * n);
        pid = c.pid.as<int>();
        k_problem_ids<<<nprob, TPB, 0, s>>>(c.poff.as<int64_t>(), pid);
        VFMM_LAUNCH_CHECK();
        k_problem_boxes<<<nprob, 1024, 0, s>>>(c.poff.as<int64_t>(), x, y, z, c.pbox.as<RootBox>());
        VFMM_LAUNCH_CHECK();
    } else {
        VFMM_HIP(hipMemcpyAsync(c.pbox.ptr, &c.box, sizeof(RootBox), hipMemcpyHostToDevice, s));
    }
    k_morton<<<cdiv(n, TPB), TPB, 0, s>>>(x, y, z, n, c.pbox.as<RootBox>(), pid, KL, c.keyA.as<uint64_t>(),
                                           c.valA.as<uint32_t>());
    VFMM_LAUNCH_CHECK();
    radix_sort(c, c.keyA, c.valA, c.keyB, c.valB, n, 3 * KL + pbits);
    c.rec.ensure(sizeof(float4) * 2 * n);
    c.perm.ensure(sizeof(int) * n);
    k_gather_pos<<<cdiv(n, TPB), TPB, 0, s>>>(c.valA.as<uint32_t>(), n, x, y, z, sigma, c.rec.as<float4>(),
                                               c.perm.as<int>());
    VFMM_LAUNCH_CHECK();
    c.record(2 * PH_BOUNDS_SORT + 1);
    c.record(2 * PH_TREE);

    // ---- levels ----
    size_t cap = (size_t)std::max<int64_t>(64, 2 * n / std::max(1, c.prm.ncrit) + 64 + 2 * (int64_t)nprob);
    DevBuf *arrs[] = {&c.c_start, &c.c_count, &c.c_parent, &c.c_child, &c.c_nchild, &c.c_level};
    for (DevBuf *b : arrs) b->ensure(sizeof(int) * cap);
    cap = std::min(c.c_start.cap, std::min(c.c_count.cap, c.c_parent.cap)) / sizeof(int);
    for (DevBuf *b : arrs) cap = std::min(cap, b->cap / sizeof(int));
    c.lvl_off.assign(1, 0);
    c.lvl_off.push_back(nprob);
    int lvl = 0;
    const uint64_t *keys = c.keyA.as<uint64_t>();
    const int64_t *poff = nprob > 1 ? c.poff.as<int64_t>() : nullptr;
    bool done = false;
    if (nprob <= TREE_GROUP) {
        TreeGroupArgs T{};
        T.keys = keys;
        T.off = poff;
        T.nroot = nprob;
        T.n = (int)n;
        T.ncrit = c.prm.ncrit;
        T.KL = KL;
        T.cap = (int)std::min<size_t>(cap, INT32_MAX);
        T.start = c.c_start.as<int>();
        T.count = c.c_count.as<int>();
        T.parent = c.c_parent.as<int>();
        T.child = c.c_child.as<int>();
        T.nchild = c.c_nchild.as<int>();
        T.level = c.c_level.as<int>();
        c.leaves.ensure(sizeof(int) * cap);
        T.leaves = c.leaves.as<int>();
        T.res = c.bres.as<Bounds>();
        T.host = pinned_ints(c);
        k_tree_group<<<1, 1024, 0, s>>>(T);
        VFMM_LAUNCH_CHECK();
        int h[32];
        sync_ints(c, 32, h);
        done = h[0] != 0;
        c.lvl_off.assign(h + 4, h + 4 + h[1]);
        lvl = h[1] - 2;
        if (done) {
            c.nleaves = h[2];
            c.overfull_leaves = h[3];
        }
    } else {
        k_roots<<<cdiv(nprob, TPB), TPB, 0, s>>>(nprob, poff, (int)n, c.c_start.as<int>(), c.c_count.as<int>(),
                                                  c.c_parent.as<int>(), c.c_level.as<int>());
        VFMM_LAUNCH_CHECK();
    }
    int h_tot[2];
    while (!done) {
        const int c0 = c.lvl_off[lvl], c1 = c.lvl_off[lvl + 1];
        const int nl = c1 - c0;
        c.c_tmp.ensure(sizeof(int) * (2 * (size_t)nl + 2));
        int *nch = c.c_tmp.as<int>();
        int *off = nch + nl + 1;
        k_count_children<<<cdiv(8 * (int64_t)nl, TPB), TPB, 0, s>>>(c0, c1, lvl, c.prm.ncrit, KL, c.c_start.as<int>(),
                                                        c.c_count.as<int>(), keys, nch, c.bres.as<Bounds>());
        VFMM_LAUNCH_CHECK();
        scan_excl_i32(c, nch, off, nl);
        read_ints(c, {off + nl - 1, nch + nl - 1}, h_tot);
        const int total = h_tot[0] + h_tot[1];
        if ((size_t)(c1 + total) > cap) {
            const size_t ncap = (size_t)(c1 + total) * 2;
            for (DevBuf *b : arrs) grow_keep(c, *b, sizeof(int) * ncap, sizeof(int) * (size_t)c1);
            cap = ncap;
        }
        k_make_children<<<cdiv(8 * (int64_t)nl, TPB), TPB, 0, s>>>(c0, c1, lvl, c1, KL, c.c_start.as<int>(), c.c_count.as<int>(),
                                                       keys, off, nch, c.c_start.as<int>(), c.c_count.as<int>(),
                                                       c.c_parent.as<int>(), c.c_child.as<int>(),
                                                       c.c_nchild.as<int>(), c.c_level.as<int>());
        VFMM_LAUNCH_CHECK();
        if (total == 0) break;
        c.lvl_off.push_back(c1 + total);
        ++lvl;
    }
    c.depth = lvl;
    c.ncells = c.lvl_off.back();
    const int nc = c.ncells;

    // ---- geometry ----
    c.c_geo.ensure(sizeof(float4) * nc);
    c.c_rad.ensure(sizeof(float) * nc);
    c.c_lo.ensure(sizeof(float4) * nc);
    c.c_hi.ensure(sizeof(float4) * nc);
    c.c_geo64.ensure(sizeof(double4) * nc);
    k_leaf_geometry<<<cdiv(nc * (int64_t)GEO_LANES, TPB), TPB, 0, s>>>(nc, c.pbox.as<RootBox>(), KL, c.c_start.as<int>(), c.c_count.as<int>(),
                                                   c.c_level.as<int>(), c.c_nchild.as<int>(), keys,
                                                   c.rec.as<float4>(), c.c_geo.as<float4>(),
                                                   c.c_geo64.as<double4>(), c.c_rad.as<float>(),
                                                   c.c_lo.as<float4>(), c.c_hi.as<float4>());
    VFMM_LAUNCH_CHECK();
    if (nc <= TREE_GEO_GROUP) {
        LevelOffsets L{};
        std::copy(c.lvl_off.begin(), c.lvl_off.end(), L.v);
        k_internal_geometry_group<<<1, 1024, 0, s>>>(L, c.depth, c.c_child.as<int>(), c.c_nchild.as<int>(),
                                                     c.c_geo.as<float4>(), c.c_rad.as<float>(), c.c_lo.as<float4>(),
                                                     c.c_hi.as<float4>());
        VFMM_LAUNCH_CHECK();
    }
    for (int l = nc <= TREE_GEO_GROUP ? -1 : c.depth - 1; l >= 0; --l) {
        const int c0 = c.lvl_off[l], c1 = c.lvl_off[l + 1];
        k_internal_geometry<<<cdiv(c1 - c0, TPB), TPB, 0, s>>>(c0, c1, c.c_child.as<int>(), c.c_nchild.as<int>(),
                                                                c.c_geo.as<float4>(), c.c_rad.as<float>(),
                                                                c.c_lo.as<float4>(), c.c_hi.as<float4>());
        VFMM_LAUNCH_CHECK();
    }
    // ---- leaf list ----
    if (done) {
        c.record(2 * PH_TREE + 1);
        return;
    }
    c.c_tmp.ensure(sizeof(int) * (2 * (size_t)nc + 2));
    int *flag = c.c_tmp.as<int>();
    int *pos = flag + nc + 1;
    k_leaf_flags<<<cdiv(nc, TPB), TPB, 0, s>>>(nc, c.c_nchild.as<int>(), flag);
    VFMM_LAUNCH_CHECK();
    scan_excl_i32(c, flag, pos, nc);
    int h3[3];
    read_ints(c, {pos + nc - 1, flag + nc - 1, &c.bres.as<Bounds>()->overfull}, h3);
    h_tot[0] = h3[0];
    h_tot[1] = h3[1];
    const int h_ovf = h3[2];
    c.nleaves = h_tot[0] + h_tot[1];
    c.overfull_leaves = h_ovf;
    c.leaves.ensure(sizeof(int) * (size_t)c.nleaves);
    k_leaf_compact<<<cdiv(nc, TPB), TPB, 0, s>>>(nc, c.c_nchild.as<int>(), pos, c.leaves.as<int>());
    VFMM_LAUNCH_CHECK();
    c.record(2 * PH_TREE + 1);
}

}  // namespace vfmm
