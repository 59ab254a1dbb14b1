// Shell-binned kinetic-energy spectrum E(k) of a velocity field sampled on a
// uniform n^3 lattice (Sec. 4.3: the spectrum of the velocity induced on a
// lattice of points that are not the particles).
//
// u_hat(kappa) = (1/n^3) sum_t u(x_t) exp(-2 pi i kappa.t / n) for the integer
// wavevectors kappa of the lattice (centred, |kappa_d| <= n/2), and
//     E(k) = 1/2 sum over kappa with round(|kappa|) = k of |u_hat(kappa)|^2,
// k = 0 .. round(sqrt(3) n / 2); wavenumbers are in units of 2 pi / L, and
// sum_k E(k) = 1/2 mean |u|^2.
//
// The transform is three passes of FFTs along the lattice axes in float64, so
// the spectrum carries float64 rounding only.  Two symmetries of real fields
// halve it: u and v travel as one complex field u + i v, whose |.|^2 summed over
// a shell (closed under kappa -> -kappa) is that of u plus that of v; and lines
// of w are transformed two at a time, of whose spectra only kz = 0 .. n/2 is
// kept (the others count twice).  A work-group takes SP_T neighbouring lines
// (whole 128-byte rows of the strided axes) through LDS: decimation in
// frequency, two stages per pass over LDS, twiddles from one table per
// work-group, output left in bit-reversed order, which only the wavevectors of
// the binning see.  The last pass bins |.|^2 as it goes instead of writing the
// field back: per-work-group partial bins (LDS atomics, whose order varies in
// the last bits of float64) added in a fixed order.
// Bound by memory: at 128^3 25 MB of float32 in, 50 MB of float64 written and
// read twice (three complex fields, each of four passes over 100 MB, and a
// sincospi per butterfly before: 650 us; now 82 us of kernels, 97 us a call).
#include <cstring>

#include "ctx.h"

namespace vfmm {

static constexpr int SP_TPB = 256;
static constexpr int SP_PARTS = 1024;  // work-groups of the last pass (bins are kept over its tiles)

// lines per tile: eight rows of 16 bytes fill a 128-byte segment; at n >= 512 four, so that several work-groups share
// a CU's 160 KB of LDS (44 KB each at 512; at 1,024 one, of up to 88 KB)
__host__ __device__ constexpr int sp_t(int n) { return n >= 512 ? 4 : 8; }

struct SpArgs {
    int n, logn;
    int T, TP;         // lines per tile, LDS row stride (elements)
    const float *ux, *uy, *uz;
    double2 *A;        // u + i v: [n][n][n]
    double2 *B;        // w: [n][n][n/2 + 1]
};

__device__ inline int sp_rev(int v, int logn) { return (int)(__brev((unsigned)v) >> (32 - logn)); }

// tw[k] = exp(-2 pi i k / n), k < n / 2
__device__ inline void sp_twiddles(double2 *tw, int n) {
    for (int k = threadIdx.x; k < n / 2; k += SP_TPB) {
        double sn, cs;
        sincospi(-2.0 * (double)k / (double)n, &sn, &cs);
        tw[k] = make_double2(cs, sn);
    }
}

__device__ inline double2 sp_add(double2 a, double2 b) { return make_double2(a.x + b.x, a.y + b.y); }
__device__ inline double2 sp_sub_mul(double2 a, double2 b, double2 w) {  // (a - b) w
    const double x = a.x - b.x, y = a.y - b.y;
    return make_double2(x * w.x - y * w.y, x * w.y + y * w.x);
}

// In-place forward transforms of the T lines of a tile, x[idx * TP + t], natural
// order in, bit-reversed order out.  Begins and ends with the tile complete.
__device__ inline void sp_fft(double2 *x, const double2 *tw, int n, int logn, int T, int TP) {
    int h = n >> 1;  // half length of the stage
    if (logn & 1) {  // an odd stage first
        for (int i = threadIdx.x; i < h * T; i += SP_TPB) {
            const int t = i % T, pos = i / T;
            double2 *p = x + pos * TP + t, *q = p + h * TP;
            const double2 a = *p, b = *q;
            *p = sp_add(a, b);
            *q = sp_sub_mul(a, b, tw[pos]);
        }
        __syncthreads();
        h >>= 1;
    }
    for (; h >= 2; h >>= 2) {  // two stages, of half lengths h and h / 2
        const int g = h >> 1, step = (n >> 1) / h;
        for (int i = threadIdx.x; i < (n >> 2) * T; i += SP_TPB) {
            const int t = i % T, b = i / T;
            const int pos = b & (g - 1), grp = b / g;
            double2 *p = x + (grp * 2 * h + pos) * TP + t;
            const double2 x0 = p[0], x1 = p[g * TP], x2 = p[h * TP], x3 = p[(h + g) * TP];
            const double2 w = tw[pos * step], w2 = tw[2 * pos * step];
            const double2 wq = make_double2(w.y, -w.x);  // w of pos + g: times -i
            const double2 y0 = sp_add(x0, x2), y2 = sp_sub_mul(x0, x2, w);
            const double2 y1 = sp_add(x1, x3), y3 = sp_sub_mul(x1, x3, wq);
            p[0] = sp_add(y0, y1);
            p[g * TP] = sp_sub_mul(y0, y1, w2);
            p[h * TP] = sp_add(y2, y3);
            p[(h + g) * TP] = sp_sub_mul(y2, y3, w2);
        }
        __syncthreads();
    }
}

// First pass, along k: the first n^2 / T work-groups transform lines of u + i v,
// the others pairs of lines of w, of which the two half spectra are written in
// natural order.
__global__ __launch_bounds__(SP_TPB) void k_sp_lines(SpArgs S) {
    extern __shared__ double2 smem[];
    const int n = S.n, T = S.T, TP = S.TP;
    double2 *tw = smem, *x = smem + n / 2;
    const int nl = n * n, ntA = (nl + T - 1) / T;
    const bool isB = (int)blockIdx.x >= ntA;
    const int l0 = (isB ? (int)blockIdx.x - ntA : (int)blockIdx.x) * T;  // first line, or pair of lines
    const int lines = min(T, (isB ? nl / 2 : nl) - l0);
    sp_twiddles(tw, n);
    for (int i = threadIdx.x; i < T * n; i += SP_TPB) {
        const int t = i / n, k = i % n;
        double2 v = make_double2(0.0, 0.0);
        if (t < lines) {
            const int64_t at = (int64_t)(l0 + t) * (isB ? 2 * n : n) + k;
            v = isB ? make_double2((double)S.uz[at], (double)S.uz[at + n])
                    : make_double2((double)S.ux[at], (double)S.uy[at]);
        }
        x[k * TP + t] = v;
    }
    __syncthreads();
    sp_fft(x, tw, n, S.logn, T, TP);
    if (!isB) {
        for (int i = threadIdx.x; i < lines * n; i += SP_TPB) {
            const int t = i / n, k = i % n;
            S.A[(int64_t)(l0 + t) * n + k] = x[k * TP + t];
        }
    } else {
        const int nh = n / 2 + 1;
        for (int i = threadIdx.x; i < lines * nh; i += SP_TPB) {
            const int t = i / nh, k = i % nh;
            const double2 a = x[sp_rev(k, S.logn) * TP + t], b = x[sp_rev((n - k) & (n - 1), S.logn) * TP + t];
            const int64_t at = (int64_t)(l0 + t) * 2 * nh + k;
            S.B[at] = make_double2(0.5 * (a.x + b.x), 0.5 * (a.y - b.y));       // (Z + conj Z') / 2
            S.B[at + nh] = make_double2(0.5 * (a.y + b.y), 0.5 * (b.x - a.x));  // (Z - conj Z') / 2i
        }
    }
}

// A tile of T neighbouring columns of field A or B: tile number -> field, row
// width, fixed index, first column, columns
struct SpTile {
    double2 *f;
    int R, fix, c0, cols;
    bool isB;
};

__device__ inline SpTile sp_tile(const SpArgs &S, int tile) {
    const int n = S.n, nh = n / 2 + 1;
    const int pa = (n + S.T - 1) / S.T, pb = (nh + S.T - 1) / S.T;
    SpTile q;
    q.isB = tile >= n * pa;
    if (q.isB) tile -= n * pa;
    const int per = q.isB ? pb : pa;
    q.f = q.isB ? S.B : S.A;
    q.R = q.isB ? nh : n;
    q.fix = tile / per;
    q.c0 = (tile % per) * S.T;
    q.cols = min(S.T, q.R - q.c0);
    return q;
}

// loads (or stores) the lines p[idx * stride + column] of a tile
__device__ inline void sp_load(double2 *x, const double2 *p, int64_t stride, int n, int cols, int T, int TP) {
    for (int i = threadIdx.x; i < n * T; i += SP_TPB) {
        const int t = i % T, idx = i / T;
        x[idx * TP + t] = t < cols ? p[idx * stride + t] : make_double2(0.0, 0.0);
    }
    __syncthreads();
}

// Second pass, along j, in place: one tile per work-group (fixed i).
__global__ __launch_bounds__(SP_TPB) void k_sp_cols(SpArgs S) {
    extern __shared__ double2 smem[];
    const int n = S.n;
    double2 *tw = smem, *x = smem + n / 2;
    const SpTile q = sp_tile(S, blockIdx.x);
    double2 *p = q.f + (int64_t)q.fix * n * q.R + q.c0;
    sp_twiddles(tw, n);
    sp_load(x, p, q.R, n, q.cols, S.T, S.TP);
    sp_fft(x, tw, n, S.logn, S.T, S.TP);
    for (int i = threadIdx.x; i < n * S.T; i += SP_TPB) {
        const int t = i % S.T, idx = i / S.T;
        if (t < q.cols) p[(int64_t)idx * q.R + t] = x[idx * S.TP + t];
    }
}

// Third pass, along i (fixed j), binned: part[g * nbins + shell].
__global__ __launch_bounds__(SP_TPB) void k_sp_bins(SpArgs S, int tiles, int nbins, double *part) {
    extern __shared__ double2 smem[];
    const int n = S.n, logn = S.logn, T = S.T, TP = S.TP;
    double2 *tw = smem, *x = smem + n / 2;
    double *bins = reinterpret_cast<double *>(x + (size_t)n * TP);
    sp_twiddles(tw, n);
    for (int k = threadIdx.x; k < nbins; k += SP_TPB) bins[k] = 0.0;
    auto mag = [&](int k) { return k <= n / 2 ? k : n - k; };  // |wavenumber| of an index
    for (int tile = blockIdx.x; tile < tiles; tile += gridDim.x) {
        const SpTile q = sp_tile(S, tile);
        sp_load(x, q.f + (int64_t)q.fix * q.R + q.c0, (int64_t)n * q.R, n, q.cols, T, TP);
        sp_fft(x, tw, n, logn, T, TP);
        const int ky = mag(sp_rev(q.fix, logn));
        for (int i = threadIdx.x; i < n * T; i += SP_TPB) {
            const int t = i % T, idx = i / T;
            if (t >= q.cols) continue;
            const int kx = mag(sp_rev(idx, logn));
            const int kz = q.isB ? q.c0 + t : mag(sp_rev(q.c0 + t, logn));
            const double2 v = x[idx * TP + t];
            const double e = (v.x * v.x + v.y * v.y) * (q.isB && kz > 0 && kz < n / 2 ? 2.0 : 1.0);
            // |kappa|^2 < 2^24 is exact in float32, and no square root of an integer lies close
            // enough to a half-integer for float32 rounding to move it across
            const int sh = (int)rintf(sqrtf((float)(kx * kx + ky * ky + kz * kz)));
            atomicAdd(&bins[sh], e);
        }
        __syncthreads();  // the tile and the bins are complete
    }
    for (int k = threadIdx.x; k < nbins; k += SP_TPB) part[(int64_t)blockIdx.x * nbins + k] = bins[k];
}

// one work-group per shell: the partial bins in a fixed order, straight to pinned host memory
__global__ __launch_bounds__(SP_TPB) void k_sp_sum(const double *part, int nparts, int nbins, double scale, double *E) {
    __shared__ double sh[SP_TPB / 64];
    const int k = blockIdx.x;
    double s = 0.0;
    for (int g = threadIdx.x; g < nparts; g += SP_TPB) s += part[(int64_t)g * nbins + k];
    for (int o = 32; o > 0; o >>= 1) s += __shfl_xor(s, o, 64);
    if ((threadIdx.x & 63) == 0) sh[threadIdx.x >> 6] = s;
    __syncthreads();
    if (threadIdx.x == 0) {
        for (int w = 1; w < SP_TPB / 64; ++w) s += sh[w];
        E[k] = s * scale;
    }
}

// shells 0 .. round(sqrt(3) n / 2): the lattice corner |kappa| = sqrt(3) n / 2 rounds up
int spectrum_bins(int n) { return (int)std::lrint(std::sqrt(3.0) * n / 2.0) + 1; }

template <class K>
static void allow_lds(K kernel, size_t lds) {
    if (lds > 64 * 1024)
        VFMM_HIP(hipFuncSetAttribute((const void *)kernel, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds));
}

void energy_spectrum_run(Ctx &c, int n, const float *ux, const float *uy, const float *uz, double *E_host) {
    int logn = 0;
    while ((1 << logn) < n) ++logn;
    if (n < 2 || n > 1024 || (1 << logn) != n)
        throw Error{VFMM_EINVAL, "vfmm_energy_spectrum: n must be a power of two in [2, 1024]"};
    const int64_t N = (int64_t)n * n * n;
    const int nh = n / 2 + 1, nbins = spectrum_bins(n);
    hipStream_t s = c.stream;
    if (!c.hspec) VFMM_HIP(hipHostMalloc((void **)&c.hspec, sizeof(double) * spectrum_bins(1024), hipHostMallocCoherent));
    SpArgs S{};
    S.n = n;
    S.logn = logn;
    S.T = sp_t(n);
    S.ux = ux;
    S.uy = uy;
    S.uz = uz;
    const size_t nA = (size_t)N, nB = (size_t)n * n * nh;
    c.spec.ensure(sizeof(double2) * (nA + nB) + sizeof(double) * (size_t)SP_PARTS * nbins);
    S.A = c.spec.as<double2>();
    S.B = S.A + nA;
    double *part = reinterpret_cast<double *>(S.B + nB);
    // the first pass reads and writes along the LDS columns: an odd row stride spreads the banks
    S.TP = S.T + 1;
    const size_t tw = sizeof(double2) * (n / 2);
    const size_t lds1 = tw + sizeof(double2) * (size_t)n * S.TP;
    allow_lds(k_sp_lines, lds1);
    k_sp_lines<<<cdiv(n * n, S.T) + cdiv(n * n / 2, S.T), SP_TPB, lds1, s>>>(S);
    VFMM_LAUNCH_CHECK();
    S.TP = S.T;
    const int tiles = n * (int)(cdiv(n, S.T) + cdiv(nh, S.T));
    const size_t lds2 = tw + sizeof(double2) * (size_t)n * S.TP;
    allow_lds(k_sp_cols, lds2);
    k_sp_cols<<<tiles, SP_TPB, lds2, s>>>(S);
    VFMM_LAUNCH_CHECK();
    const size_t lds3 = lds2 + sizeof(double) * nbins;
    const int groups = std::min(tiles, SP_PARTS);
    allow_lds(k_sp_bins, lds3);
    k_sp_bins<<<groups, SP_TPB, lds3, s>>>(S, tiles, nbins, part);
    VFMM_LAUNCH_CHECK();
    const double inv = 1.0 / (double)N;
    k_sp_sum<<<nbins, SP_TPB, 0, s>>>(part, groups, nbins, 0.5 * inv * inv, c.hspec);
    VFMM_LAUNCH_CHECK();
    VFMM_HIP(hipStreamSynchronize(s));
    std::memcpy(E_host, c.hspec, sizeof(double) * nbins);
}

}  // namespace vfmm
