// Far field: P2M, M2M, M2L, L2L, L2P and the periodic lattice term (Sec. 3.1,
// Sec. 3.5, Sec. 3.6) for the three Laplace potentials
//   psi_m(x) = sum_j alpha_j,m / (4 pi |x - x_j|),   m = x, y, z,
// from which u = curl psi and du_l/dx_k = eps_{l n m} d_k d_n psi_m.
//
// Expansions are normalised by the cell size s (Sec. 4.2: normalised
// coefficients keep float32 in range): a cell with centre c stores
//   Mt_n^m = sum_j q_j conj(R_n^m((x_j - c)/s)),        psi = (1/s) sum Mt I_n^m((x-c)/s)
//   Lt_n^m with psi(x) = (1/s) sum Lt_n^m R_n^m((x - c)/s)
// and sums run from the highest degree to the lowest (Sec. 4.2).  Centres are in
// float64 whatever the expansions' type: the translations by operator take the
// difference of two centres as whole quarter cells, which rounded centres are not.
#include "ctx.h"

namespace vfmm {

static constexpr int TPB = 256;

template <class V2>
__device__ inline V2 cmul(V2 a, V2 b) { return V2{a.x * b.x - a.y * b.y, a.x * b.y + a.y * b.x}; }
template <class V2>
__device__ inline V2 cconj(V2 a) { return V2{a.x, -a.y}; }

__device__ inline float fmar(float a, float b, float c) { return fmaf(a, b, c); }
__device__ inline double fmar(double a, double b, double c) { return fma(a, b, c); }

// rt^e for a ratio of cell sizes (a power of two) and an integer e >= 0
__device__ inline float powr(float rt, int e) { return __builtin_amdgcn_exp2f((float)e * __log2f(rt)); }
__device__ inline double powr(double rt, int e) { return exp2((double)e * log2(rt)); }

// c_n^m for any sign of m from the m >= 0 storage: c_n^{-m} = (-1)^m conj(c_n^m).
template <class V2>
__device__ inline V2 getc(const V2 *a, int n, int m) {
    if (m >= 0) return a[CIDX(n, m)];
    const V2 v = a[CIDX(n, -m)];
    return (m & 1) ? V2{-v.x, v.y} : V2{v.x, -v.y};
}

__device__ inline void decode_nm(int t, int &n, int &m) {
    n = (int)((sqrtf(8.0f * t + 1.0f) - 1.0f) * 0.5f);
    while ((n + 1) * (n + 2) / 2 <= t) ++n;
    while (n * (n + 1) / 2 > t) --n;
    m = t - n * (n + 1) / 2;
}

// ---------------------------------------------------------------------------
// P2M: one wave per leaf, particles staged CH at a time.
// ---------------------------------------------------------------------------
template <int P, class R>
__global__ __launch_bounds__(64) void k_p2m(const int *leaves, const int *start, const int *count, const int *nsrc,
                                            const double4 *geo, const typename VT<R>::V4 *rec,
                                            typename VT<R>::V2 *Mexp) {
    using V2 = typename VT<R>::V2;
    using V4 = typename VT<R>::V4;
    constexpr int NCP = NC(P);
    // particles staged per pass: 32 (17 KB of LDS in float32) lets nine
    // one-wave work-groups share a CU; 64 (34 KB) allowed four and was slower
    constexpr int CH = 32;
    __shared__ V2 Rs[CH][NCP];
    __shared__ V4 al[CH];
    const int lane = threadIdx.x;
    const int cell = leaves[blockIdx.x];
    const auto g = geo[cell];
    const R inv = R(1) / R(g.w);
    const int s0 = start[cell], cnt = nsrc ? nsrc[cell] : count[cell];  // target points carry no strength
    constexpr int NT = (NCP + 63) / 64;
    V2 acc[NT][3];
#pragma unroll
    for (int t = 0; t < NT; ++t)
        for (int c = 0; c < 3; ++c) acc[t][c] = V2{R(0), R(0)};
    for (int b = 0; b < cnt; b += CH) {
        if (lane < CH) {
            const int j = s0 + b + lane;
            if (b + lane < cnt) {
                const V4 p = rec[2 * j];
                V2 Rl[NCP];
                regular_harmonics<P, R, V2>(R(p.x - g.x) * inv, R(p.y - g.y) * inv, R(p.z - g.z) * inv, Rl);
#pragma unroll
                for (int t = 0; t < NCP; ++t) Rs[lane][t] = Rl[t];
                al[lane] = rec[2 * j + 1];
            } else {
                al[lane] = V4{R(0), R(0), R(0), R(0)};
#pragma unroll
                for (int t = 0; t < NCP; ++t) Rs[lane][t] = V2{R(0), R(0)};
            }
        }
        __syncthreads();
        const int jmax = min(CH, cnt - b);
#pragma unroll
        for (int t = 0; t < NT; ++t) {
            const int coef = lane + 64 * t;
            if (coef < NCP) {
                for (int jj = 0; jj < jmax; ++jj) {
                    const V2 r = Rs[jj][coef];
                    const V4 a = al[jj];
                    acc[t][0].x += a.x * r.x; acc[t][0].y -= a.x * r.y;
                    acc[t][1].x += a.y * r.x; acc[t][1].y -= a.y * r.y;
                    acc[t][2].x += a.z * r.x; acc[t][2].y -= a.z * r.y;
                }
            }
        }
        __syncthreads();
    }
#pragma unroll
    for (int t = 0; t < NT; ++t) {
        const int coef = lane + 64 * t;
        if (coef < NCP)
            for (int c = 0; c < 3; ++c) Mexp[((size_t)cell * 3 + c) * NCP + coef] = acc[t][c];
    }
}

// ---------------------------------------------------------------------------
// M2M: one work-group per parent cell of one level, one thread per (child,
// coefficient n >= m >= 0 of the parent) for the three potentials.
//   Mt_n^m(P) = sum_children sum_{k,l} conj(R_k^l(d)) (s_c/s_P)^{n-k} Mt_{n-k}^{m-l}(c),
//   d = (c - P)/s_P.
// The children are staged in LDS as full-order tables (m from -n to n, negative
// orders expanded once) with the size ratio folded into the child's
// coefficients, so the inner loop is a plain complex multiply-add; the children
// of a coefficient are neighbouring lanes, summed by shuffles.  The first wave
// or two take the harmonics, a lane per child and order, the others stage.
// S is the storage type of the expansions, R the arithmetic type (the mixed
// precision form keeps float storage and accumulates in double).
// Bound by latency at the coarse levels and by LDS reads at the fine ones (32
// bytes for the three potentials' terms).  One child after another with a thread
// per potential: 33 us a level of 1 to 8 cells at p = 8 and 0.33 ms for the five
// levels of 80^3 particles at p = 10; now 8 us and 0.21 ms.
// ---------------------------------------------------------------------------
template <int P, class R = float>
struct XferCfg {
    static constexpr int NCP = NC(P);
    static constexpr int W = 2 * P + 1;                       // full-order row width
    static constexpr int ROWS = (P + 1) * W;
    static constexpr int CH = sizeof(R) == 8 ? 4 : 8;         // children staged at once by M2M
    static constexpr int M2M_HARM = ((CH * (P + 1) + 63) / 64) * 64;  // threads that take the harmonics
    static constexpr int L2L_HARM = ((8 * (P + 1) + 63) / 64) * 64;
    static constexpr int M2M_THREADS = ((CH * NCP + 63) / 64) * 64 + 64;
    static constexpr int L2L_THREADS = ((8 * NCP + 63) / 64) * 64 + 64;
};

// The orders +-m of R(d) (common.h regular_harmonics, one order's recursion) into
// the full-order table T; CONJ: its conjugate
template <int P, class R, bool CONJ, class V2>
__device__ inline void harmonics_order(R x, R y, R z, int m, V2 *T) {
    constexpr int W = 2 * P + 1;
    const R r2 = x * x + y * y + z * z;
    R cr = R(1), ci = R(0);  // R_m^m
    for (int k = 1; k <= m; ++k) {
        const R f = R(-1) / R(2 * k);
        const R nr = f * (x * cr - y * ci);
        const R ni = f * (x * ci + y * cr);
        cr = nr;
        ci = ni;
    }
    auto put = [&](int n, R vr, R vi) {
        const R v = CONJ ? -vi : vi;
        T[n * W + P + m] = V2{vr, v};
        if (m > 0) T[n * W + P - m] = (m & 1) ? V2{-vr, v} : V2{vr, -v};
    };
    put(m, cr, ci);
    R pr = R(0), pi = R(0);  // R_{n-2}^m
    for (int n = m + 1; n <= P; ++n) {
        const R inv = R(1) / R(n * n - m * m);
        const R a = R(2 * n - 1) * z;
        // R_{m+1}^m = z R_m^m
        const R vr = n == m + 1 ? z * cr : (a * cr - r2 * pr) * inv;
        const R vi = n == m + 1 ? z * ci : (a * ci - r2 * pi) * inv;
        put(n, vr, vi);
        pr = cr;
        pi = ci;
        cr = vr;
        ci = vi;
    }
}

template <int P, class R, class S>
__global__ __launch_bounds__((XferCfg<P, R>::M2M_THREADS)) void k_m2m(int c0, int c1, const int *child,
                                                                     const int *nchild, const double4 *geo,
                                                                     typename VT<S>::V2 *Mexp) {
    using V2 = typename VT<R>::V2;
    using C = XferCfg<P, R>;
    constexpr int NCP = C::NCP, W = C::W, CH = C::CH;
    __shared__ V2 Mf[CH][3][C::ROWS];   // child multipole, scaled by (s_c/s_P)^n, full orders
    __shared__ V2 Rf[CH][C::ROWS];      // conj R_k^l(d), full orders
    const int cell = c0 + blockIdx.x;
    if (cell >= c1) return;
    const int nc = nchild[cell];
    if (nc == 0) return;
    const int f = child[cell];
    const auto gp = geo[cell];
    const int tid = threadIdx.x;
    const R inv = R(1) / R(gp.w);
    const int ch = tid % CH, q = tid / CH;  // the high coefficients, whose sums are longest, share waves
    const bool active = q < NCP;
    int n = 0, m = 0;
    decode_nm(active ? q : 0, n, m);
    V2 acc[3];
#pragma unroll
    for (int c = 0; c < 3; ++c) acc[c] = V2{R(0), R(0)};
    for (int k0 = 0; k0 < nc; k0 += CH) {
        const int nk = min(CH, nc - k0);
        if (k0 > 0) __syncthreads();
        if (tid < C::M2M_HARM) {
            const int k = tid % CH;
            if (k < nk && tid / CH <= P) {
                const auto gc = geo[f + k0 + k];
                harmonics_order<P, R, true>(R(gc.x - gp.x) * inv, R(gc.y - gp.y) * inv, R(gc.z - gp.z) * inv,
                                            tid / CH, Rf[k]);
            }
        } else {
            for (int i = tid - C::M2M_HARM; i < nk * 3 * NCP; i += C::M2M_THREADS - C::M2M_HARM) {
                const int k = i / (3 * NCP), cc = i / NCP % 3;
                int a, b;
                decode_nm(i % NCP, a, b);
                const auto v = Mexp[(size_t)(f + k0) * 3 * NCP + i];
                const R sc = powr(R(geo[f + k0 + k].w) * inv, a);
                const R vr = sc * R(v.x), vi = sc * R(v.y);
                Mf[k][cc][a * W + P + b] = V2{vr, vi};
                if (b > 0) Mf[k][cc][a * W + P - b] = (b & 1) ? V2{-vr, vi} : V2{vr, -vi};
            }
        }
        __syncthreads();
        if (active && ch < nk) {
            // sum from high source degree n - kk to low: kk from 0 up
            for (int kk = 0; kk <= n; ++kk) {
                const int nm = n - kk;
                const int lo = max(-kk, m - nm), hi = min(kk, m + nm);
                const V2 *r = &Rf[ch][kk * W + P], *v = &Mf[ch][0][nm * W + P + m];
                for (int l = lo; l <= hi; ++l) {
                    const V2 h = r[l];
#pragma unroll
                    for (int c = 0; c < 3; ++c) {
                        const V2 w = v[c * C::ROWS - l];
                        acc[c].x = fmar(h.x, w.x, fmar(-h.y, w.y, acc[c].x));
                        acc[c].y = fmar(h.x, w.y, fmar(h.y, w.x, acc[c].y));
                    }
                }
            }
        }
    }
#pragma unroll
    for (int c = 0; c < 3; ++c)
#pragma unroll
        for (int o = CH / 2; o > 0; o >>= 1) {
            acc[c].x += __shfl_xor(acc[c].x, o, CH);
            acc[c].y += __shfl_xor(acc[c].y, o, CH);
        }
    if (active && ch < 3) {
        const V2 v = ch == 0 ? acc[0] : ch == 1 ? acc[1] : acc[2];
        auto &dst = Mexp[((size_t)cell * 3 + ch) * NCP + q];
        dst.x = (S)v.x;
        dst.y = (S)v.y;
    }
}

// ---------------------------------------------------------------------------
// M2L, one translation at a time (Sec. 3.6): short lists, rare operators, trees
// whose translations do not group, and the float64 form at p = 12.
//   Lt_k^l(A) = (-1)^{k+l} lambda^{-(k+1)} sum_{n,m} Mt_n^m(B) I_{n+k}^{m-l}((c_A - c_B)/s_B),
//   lambda = s_B/s_A.
// With I^{-mu} = (-1)^mu conj(I^mu), Mt^{-m} = (-1)^m conj(Mt^m), z1 = I_{n+k}^{m-l},
// z2 = (-1)^l I_{n+k}^{m+l}, the terms of +-m are
//   Re: Mr (z1r + z2r) - Mi (z1i + z2i),   Im: Mr (z1i - z2i) + Mi (z1r - z2r).
// Target lists are cut into parts (m2l_pair_plan), a work-group each, whose
// partial sums k_m2l_add adds to the local expansions in list order: with a
// work-group per target the 64 targets of a 3,000-particle tree ran on 64 CUs,
// its longest list of 43 sources in one serial loop (235 -> 18 us).  A
// work-group stages SB sources at a time in LDS (the harmonics |M| <= N <= 2P of
// each, a column of one order per thread, and the multipoles), and a subgroup
// of LP threads takes each source.  A thread holds one order l and KB
// consecutive degrees k of the output, real and imaginary, for the three
// potentials; with KB > 1 it walks n downwards at fixed m, so that each harmonic
// that it reads serves KB degrees (n + k = N), and so does each multipole.  In float64 the
// kernel is bound by LDS reads, so KB = 3 (64^3, 1.43 million translations: 7.5
// ms; KB = 2 8.6, KB = 1 16.8, a thread per real output row 16.2 ms); in float32
// the walk's registers outweigh them, so KB = 1 with n outermost (70,516
// translations at p = 8: 0.18 ms; KB = 2 0.30, KB = 3 0.33 ms, a thread per real
// output row 0.44 ms).
// ---------------------------------------------------------------------------
__host__ __device__ constexpr int m2l_kb(bool dbl) { return dbl ? 3 : 1; }
__host__ __device__ constexpr int m2l_lanes(int P, bool dbl) {  // threads per source
    int n = 0;
    for (int l = 0; l <= P; ++l) n += (P + m2l_kb(dbl) - l) / m2l_kb(dbl);
    return n;
}
__host__ __device__ constexpr int m2l_sources(int P, bool dbl) {  // sources staged at once
    const int s = (dbl ? 192 : 320) / m2l_lanes(P, dbl);
    return s < 8 ? s : 8;
}

template <int P, class R = float>
struct M2LCfg {
    static constexpr int NCP = NC(P);
    static constexpr int KB = m2l_kb(sizeof(R) == 8);
    static constexpr int LP = m2l_lanes(P, sizeof(R) == 8);
    static constexpr int SB = m2l_sources(P, sizeof(R) == 8);
    static constexpr int THREADS = ((SB * LP + 63) / 64) * 64;
    static constexpr int Q = 2 * P;
    // I_N^M at PAD + N (N + 1) + M; a thread's lowest degrees may lie below l, whose
    // (unused) sums read up to two elements in front
    static constexpr int PAD = 2;
    static constexpr int ISZ = PAD + (Q + 1) * (Q + 1);
    using V2 = typename VT<R>::V2;
    static constexpr size_t LDS = sizeof(V2) * SB * (ISZ + 3 * NCP) + sizeof(R) * SB;
};

template <int P, class R>
__global__ __launch_bounds__((M2LCfg<P, R>::THREADS)) void k_m2l(const int4 *parts, const int2 *src,
                                                               const double4 *geo,
                                                               const typename VT<R>::V2 *__restrict__ Mexp,
                                                               typename VT<R>::V2 *__restrict__ partial, int B,
                                                               float len) {
    using C = M2LCfg<P, R>;
    using V2 = typename VT<R>::V2;
    constexpr int KB = C::KB, NCP = C::NCP;
    extern __shared__ double2 smem[];
    V2 *Is = reinterpret_cast<V2 *>(smem);   // [SB][ISZ]
    V2 *Ms = Is + C::SB * C::ISZ;            // [SB][3][NCP]
    R *lam = reinterpret_cast<R *>(Ms + C::SB * 3 * NCP);
    const int4 part = parts[blockIdx.x];  // (target, first entry, end entry)
    const int tgt = part.x;
    if (tgt < 0) return;
    const int o0 = part.y, o1 = part.z;
    const int tid = threadIdx.x;
    const auto ga = geo[tgt];
    const int sub = tid / C::LP;
    int j = tid % C::LP, l = 0;
    for (int cnt = (P + KB) / KB; j >= cnt; cnt = (P - l + KB) / KB) {
        j -= cnt;
        ++l;
    }
    const int kt = P - KB * j;  // this thread's degrees: kt, kt - 1, .. (those >= l)
    const R sg = (l & 1) ? R(-1) : R(1);
    R re[KB][3], im[KB][3];
#pragma unroll
    for (int q = 0; q < KB; ++q)
#pragma unroll
        for (int c = 0; c < 3; ++c) re[q][c] = im[q][c] = R(0);
    const int W = 2 * B + 1;
    for (int e0 = o0; e0 < o1; e0 += C::SB) {
        const int nb = min(C::SB, o1 - e0);
        __syncthreads();
        // ---- stage nb sources ----
        for (int i = tid; i < nb * (C::Q + 1); i += C::THREADS) {
            const int s = i / (C::Q + 1), M = i % (C::Q + 1);
            const int2 ent = src[e0 + s];
            const auto gb = geo[ent.x];
            const double L = len;
            const R inv = R(1) / R(gb.w);
            const R dx = R(ga.x - gb.x - (ent.y % W - B) * L) * inv;
            const R dy = R(ga.y - gb.y - ((ent.y / W) % W - B) * L) * inv;
            const R dz = R(ga.z - gb.z - (ent.y / (W * W) - B) * L) * inv;
            const R r2 = dx * dx + dy * dy + dz * dz;
            const R ir2 = R(1) / r2;
            // I_M^M by the diagonal recurrence, then upward in N
            R cr = rsqr(r2), ci = R(0);
            for (int mm = 1; mm <= M; ++mm) {
                const R f = -(R)(2 * mm - 1) * ir2;
                const R nr = f * (dx * cr - dy * ci);
                const R ni = f * (dx * ci + dy * cr);
                cr = nr;
                ci = ni;
            }
            V2 *I = Is + s * C::ISZ + C::PAD;
            auto put = [&](int N, R vr, R vi) {
                I[N * (N + 1) + M] = V2{vr, vi};
                if (M > 0) I[N * (N + 1) - M] = (M & 1) ? V2{-vr, vi} : V2{vr, -vi};  // (-1)^M conj
            };
            put(M, cr, ci);
            R pr = cr, pi = ci;
            R qr = R(0), qi = R(0);
            if (M + 1 <= C::Q) {
                const R a0 = (R)(2 * M + 1) * dz * ir2;
                qr = a0 * cr;
                qi = a0 * ci;
                put(M + 1, qr, qi);
            }
            for (int N = M + 2; N <= C::Q; ++N) {
                const R a = (R)(2 * N - 1) * dz;
                const R b = (R)((N - 1) * (N - 1) - M * M);
                const R vr = (a * qr - b * pr) * ir2;
                const R vi = (a * qi - b * pi) * ir2;
                put(N, vr, vi);
                pr = qr; pi = qi; qr = vr; qi = vi;
            }
            if (M == 0) lam[s] = R(ga.w) / R(gb.w);  // 1/lambda
        }
        for (int i = tid; i < nb * 3 * NCP; i += C::THREADS) {
            const int s = i / (3 * NCP), q = i % (3 * NCP);
            Ms[i] = Mexp[(size_t)src[e0 + s].x * 3 * NCP + q];
        }
        __syncthreads();
        if (sub >= nb) continue;
        const V2 *I = Is + sub * C::ISZ + C::PAD, *Mt = Ms + sub * 3 * NCP;
        R ar[KB][3], ai[KB][3];
#pragma unroll
        for (int q = 0; q < KB; ++q)
#pragma unroll
            for (int c = 0; c < 3; ++c) ar[q][c] = ai[q][c] = R(0);
        if constexpr (KB == 1) {
#pragma unroll
            for (int n = P; n >= 0; --n) {
                const V2 *row = I + (n + kt) * (n + kt + 1);
                {
                    const V2 z = row[-l];
#pragma unroll
                    for (int c = 0; c < 3; ++c) {
                        const R w = Mt[c * NCP + CIDX(n, 0)].x;
                        ar[0][c] = fmar(w, z.x, ar[0][c]);
                        ai[0][c] = fmar(w, z.y, ai[0][c]);
                    }
                }
#pragma unroll
                for (int m = 1; m <= n; ++m) {
                    const V2 z1 = row[m - l], z2 = row[m + l];
                    const R ur = fmar(sg, z2.x, z1.x), ui = fmar(sg, z2.y, z1.y);
                    const R vr = fmar(-sg, z2.x, z1.x), vi = fmar(-sg, z2.y, z1.y);
#pragma unroll
                    for (int c = 0; c < 3; ++c) {
                        const V2 w = Mt[c * NCP + CIDX(n, m)];
                        ar[0][c] = fmar(w.x, ur, fmar(-w.y, ui, ar[0][c]));
                        ai[0][c] = fmar(w.x, vi, fmar(w.y, vr, ai[0][c]));
                    }
                }
            }
        } else {
#pragma unroll
            for (int m = 0; m <= P; ++m) {
                // z1 + z2 and z1 - z2 of the KB degrees N = n + kt - q
                V2 u[KB], v[KB];
                auto get = [&](int N, V2 &a, V2 &b) {
                    const V2 *row = I + N * (N + 1) + m;
                    const V2 z1 = row[-l];
                    if (m == 0) {  // one term, not two
                        a = z1;
                        b = z1;
                    } else {
                        const V2 z2 = row[l];
                        a = V2{fmar(sg, z2.x, z1.x), fmar(sg, z2.y, z1.y)};
                        b = V2{fmar(-sg, z2.x, z1.x), fmar(-sg, z2.y, z1.y)};
                    }
                };
#pragma unroll
                for (int q = 0; q < KB - 1; ++q) get(P + kt - q, u[q], v[q]);
#pragma unroll
                for (int n = P; n >= m; --n) {
                    get(n + kt - (KB - 1), u[KB - 1], v[KB - 1]);
#pragma unroll
                    for (int c = 0; c < 3; ++c) {
                        const V2 w = Mt[c * NCP + CIDX(n, m)];
#pragma unroll
                        for (int q = 0; q < KB; ++q) {
                            if (m == 0) {
                                ar[q][c] = fmar(w.x, u[q].x, ar[q][c]);
                                ai[q][c] = fmar(w.x, u[q].y, ai[q][c]);
                            } else {
                                ar[q][c] = fmar(w.x, u[q].x, fmar(-w.y, u[q].y, ar[q][c]));
                                ai[q][c] = fmar(w.x, v[q].y, fmar(w.y, v[q].x, ai[q][c]));
                            }
                        }
                    }
#pragma unroll
                    for (int q = 0; q < KB - 1; ++q) {
                        u[q] = u[q + 1];
                        v[q] = v[q + 1];
                    }
                }
            }
        }
#pragma unroll
        for (int q = 0; q < KB; ++q) {
            const R sc = powr(lam[sub], kt - q + 1);
#pragma unroll
            for (int c = 0; c < 3; ++c) {
                re[q][c] = fmar(sc, ar[q][c], re[q][c]);
                im[q][c] = fmar(sc, ai[q][c], im[q][c]);
            }
        }
    }
    // the subgroups' sums, added in order
    __syncthreads();
    static_assert(3 * NCP <= C::ISZ, "the sums fit the harmonics' space");
    if (sub < C::SB)
#pragma unroll
        for (int q = 0; q < KB; ++q)
            if (kt - q >= l)
#pragma unroll
                for (int c = 0; c < 3; ++c) Is[(sub * 3 + c) * NCP + CIDX(kt - q, l)] = V2{re[q][c], im[q][c]};
    __syncthreads();
    for (int i = tid; i < 3 * NCP; i += C::THREADS) {
        V2 w = Is[i];
        for (int t = 1; t < C::SB; ++t) {
            const V2 x = Is[t * 3 * NCP + i];
            w.x += x.x;
            w.y += x.y;
        }
        int kk, ll;
        decode_nm(i % NCP, kk, ll);
        const R f = ((kk + ll) & 1) ? R(-1) : R(1);
        partial[(size_t)blockIdx.x * 3 * NCP + i] = V2{f * w.x, ll == 0 ? R(0) : f * w.y};
    }
}

// slot of part p of target t's list; distinct for all parts of all targets
__device__ inline int m2l_slot(const int *off, int t, int part) { return off[t] / part + t; }

// (target, first entry, end entry, 0) of every part; the other slots hold target -1
__global__ __launch_bounds__(TPB) void k_m2l_parts(int ncells, const int *off, int part, int4 *parts) {
    const int t = blockIdx.x * (TPB / 64) + (threadIdx.x >> 6), lane = threadIdx.x & 63;
    if (t >= ncells) return;
    const int o0 = off[t], o1 = off[t + 1], s0 = m2l_slot(off, t, part);
    const int s1 = t + 1 < ncells ? m2l_slot(off, t + 1, part) : o1 / part + ncells;
    for (int s = s0 + lane; s < s1; s += 64) {
        const int e = o0 + (s - s0) * part;
        parts[s] = e < o1 ? make_int4(t, e, min(e + part, o1), 0) : make_int4(-1, 0, 0, 0);
    }
}

// Lt(t) += its parts' sums, in list order
template <class V2>
__global__ __launch_bounds__(TPB) void k_m2l_add(const int *off, int part, int nc3, const V2 *__restrict__ partial,
                                                 V2 *__restrict__ Lexp) {
    const int t = blockIdx.x;
    const int np = (off[t + 1] - off[t] + part - 1) / part;
    if (np == 0) return;
    const V2 *p = partial + (size_t)m2l_slot(off, t, part) * nc3;
    for (int i = threadIdx.x; i < nc3; i += TPB) {
        V2 v = Lexp[(size_t)t * nc3 + i];
        for (int q = 0; q < np; ++q) {
            const V2 w = p[(size_t)q * nc3 + i];
            v.x += w.x;
            v.y += w.y;
        }
        Lexp[(size_t)t * nc3 + i] = v;
    }
}

// Parts of the target lists for the translations one at a time: the sources of
// one pass where the whole list would otherwise leave CUs idle, else four
// passes, growing with the list so that the partial sums stay within the size
// of the expansions.
void m2l_pair_plan(Ctx &c, const int *off, int64_t n) {
    if (n == 0) return;
    const int sb = m2l_sources(c.prm.p, c.prm.precision == VFMM_PRECISION_FP64);
    c.m2l_part = n < 65536 ? sb : (int)std::max<int64_t>(4 * sb, n / 65536 / sb * sb);
    c.m2l_nparts = (int)(n / c.m2l_part) + c.ncells;
    const size_t vs = c.prm.precision == VFMM_PRECISION_FP64 ? sizeof(double2) : sizeof(float2);
    c.m2l_parts.ensure(sizeof(int4) * (size_t)c.m2l_nparts);
    c.m2l_partial.ensure(vs * 3 * NC(c.prm.p) * (size_t)c.m2l_nparts);
    k_m2l_parts<<<cdiv(c.ncells, TPB / 64), TPB, 0, c.stream>>>(c.ncells, off, c.m2l_part, c.m2l_parts.as<int4>());
    VFMM_LAUNCH_CHECK();
}

// ---------------------------------------------------------------------------
// L2L: one work-group per parent cell of one level, one thread per (child,
// coefficient k >= l >= 0) for the three potentials (storage S, arithmetic R as in
// M2M); the parent's expansion, staged once, and each child's R(d) as full-order
// tables.
//   Lt_k^l(c) = (s_c/s_P)^{k+1} sum_{n >= k, m} Lt_n^m(P) R_{n-k}^{m-l}(d),  d = (c - P)/s_P.
// A work-group per child with a thread per potential: 0.27 ms for the five levels
// of 80^3 particles at p = 10; now 0.12.
// ---------------------------------------------------------------------------
template <int P, class R, class S>
__global__ __launch_bounds__((XferCfg<P, R>::L2L_THREADS)) void k_l2l(int c0, int c1, const int *child,
                                                                     const int *nchild, const double4 *geo,
                                                                     typename VT<S>::V2 *Lexp) {
    using V2 = typename VT<R>::V2;
    using C = XferCfg<P, R>;
    constexpr int NCP = C::NCP, W = C::W;
    __shared__ V2 Lf[3][C::ROWS];
    __shared__ V2 Rf[8][C::ROWS];
    const int cell = c0 + blockIdx.x;
    if (cell >= c1) return;
    const int nc = nchild[cell];
    if (nc == 0) return;
    const int f = child[cell];
    const auto gp = geo[cell];
    const int tid = threadIdx.x;
    const R inv = R(1) / R(gp.w);
    if (tid < C::L2L_HARM) {
        const int j = tid % 8;
        if (j < nc && tid / 8 <= P) {
            const auto gc = geo[f + j];
            harmonics_order<P, R, false>(R(gc.x - gp.x) * inv, R(gc.y - gp.y) * inv, R(gc.z - gp.z) * inv, tid / 8,
                                         Rf[j]);
        }
    } else {
        for (int i = tid - C::L2L_HARM; i < 3 * NCP; i += C::L2L_THREADS - C::L2L_HARM) {
            const int cc = i / NCP;
            int a, b;
            decode_nm(i % NCP, a, b);
            const auto v = Lexp[(size_t)cell * 3 * NCP + i];
            const R vr = R(v.x), vi = R(v.y);
            Lf[cc][a * W + P + b] = V2{vr, vi};
            if (b > 0) Lf[cc][a * W + P - b] = (b & 1) ? V2{-vr, vi} : V2{vr, -vi};
        }
    }
    __syncthreads();
    const int ch = tid % 8, q = tid / 8;
    if (q >= NCP || ch >= nc) return;
    int k, l;
    decode_nm(q, k, l);
    V2 acc[3];
#pragma unroll
    for (int c = 0; c < 3; ++c) acc[c] = V2{R(0), R(0)};
    for (int n = P; n >= k; --n) {
        const int dn = n - k;
        const int lo = max(-n, l - dn), hi = min(n, l + dn);
        const V2 *L = &Lf[0][n * W + P], *r = &Rf[ch][dn * W + P - l];
        for (int m = lo; m <= hi; ++m) {
            const V2 h = r[m];
#pragma unroll
            for (int c = 0; c < 3; ++c) {
                const V2 w = L[c * C::ROWS + m];
                acc[c].x = fmar(w.x, h.x, fmar(-w.y, h.y, acc[c].x));
                acc[c].y = fmar(w.x, h.y, fmar(w.y, h.x, acc[c].y));
            }
        }
    }
    const R sc = powr(R(geo[f + ch].w) * inv, k + 1);
#pragma unroll
    for (int c = 0; c < 3; ++c) {
        auto &dst = Lexp[((size_t)(f + ch) * 3 + c) * NCP + q];
        dst.x = (S)((R)dst.x + sc * acc[c].x);
        dst.y = (S)((R)dst.y + sc * acc[c].y);
    }
}

// ---------------------------------------------------------------------------
// L2P: one wave per leaf, one lane per target.  With psi = (1/s) sum Lt R(r/s)
// and the ladder identities of the scaled harmonics
//   d_z R_n^m = R_{n-1}^m,  (d_x + i d_y) R_n^m = R_{n-1}^{m+1},  (d_x - i d_y) R_n^m = -R_{n-1}^{m-1},
// the first and second derivatives of each potential are sums of Lt_n^m
// against R_{n-1} and R_{n-2}.
// ---------------------------------------------------------------------------
template <int P, class R>
__global__ __launch_bounds__(64) void k_l2p(const int *leaves, const int *start, const int *count,
                                            const double4 *geo, const typename VT<R>::V4 *rec,
                                            const typename VT<R>::V2 *Lexp,
                                            int64_t n_all, R *far_u, R *far_da, int scheme) {
    using V2 = typename VT<R>::V2;
    using V4 = typename VT<R>::V4;
    constexpr int NCP = NC(P);
    constexpr int NR = NC(P - 1);
    __shared__ V2 Ls[3][NCP];
    const int cell = leaves[blockIdx.x];
    const int lane = threadIdx.x;
    for (int i = lane; i < 3 * NCP; i += 64) Ls[i / NCP][i % NCP] = Lexp[(size_t)cell * 3 * NCP + i];
    __syncthreads();
    const auto g = geo[cell];
    const R inv = R(1) / R(g.w);
    const int s0 = start[cell], cnt = count[cell];
    for (int b = 0; b < cnt; b += 64) {
        if (b + lane >= cnt) continue;
        const int j = s0 + b + lane;
        const V4 p = rec[2 * j];
        V2 Rl[NR];
        regular_harmonics<P - 1, R, V2>(R(p.x - g.x) * inv, R(p.y - g.y) * inv, R(p.z - g.z) * inv, Rl);
        R G[3][3], H[3][3][3];
        for (int c = 0; c < 3; ++c) {
            R pz = R(0), pzz = R(0);
            V2 pp = V2{R(0), R(0)}, pzp = V2{R(0), R(0)}, ppp = V2{R(0), R(0)};
#pragma unroll
            for (int n = P; n >= 1; --n) {
#pragma unroll
                for (int m = -n; m <= n; ++m) {
                    const V2 L = getc(Ls[c], n, m);
                    if (m >= -(n - 1) && m <= n - 1) pz += cmul(L, getc(Rl, n - 1, m)).x;
                    if (m + 1 >= -(n - 1) && m + 1 <= n - 1) {
                        const V2 v = cmul(L, getc(Rl, n - 1, m + 1));
                        pp.x += v.x; pp.y += v.y;
                    }
                    if (n >= 2) {
                        if (m >= -(n - 2) && m <= n - 2) pzz += cmul(L, getc(Rl, n - 2, m)).x;
                        if (m + 1 >= -(n - 2) && m + 1 <= n - 2) {
                            const V2 v = cmul(L, getc(Rl, n - 2, m + 1));
                            pzp.x += v.x; pzp.y += v.y;
                        }
                        if (m + 2 >= -(n - 2) && m + 2 <= n - 2) {
                            const V2 v = cmul(L, getc(Rl, n - 2, m + 2));
                            ppp.x += v.x; ppp.y += v.y;
                        }
                    }
                }
            }
            const R i2 = inv * inv, i3 = i2 * inv;
            G[c][0] = pp.x * i2;
            G[c][1] = pp.y * i2;
            G[c][2] = pz * i2;
            const R hzz = pzz * i3;
            const R hxx = R(0.5) * (ppp.x * i3 - hzz);
            const R hyy = R(0.5) * (-ppp.x * i3 - hzz);
            const R hxy = R(0.5) * ppp.y * i3;
            const R hxz = pzp.x * i3, hyz = pzp.y * i3;
            H[c][0][0] = hxx; H[c][0][1] = hxy; H[c][0][2] = hxz;
            H[c][1][0] = hxy; H[c][1][1] = hyy; H[c][1][2] = hyz;
            H[c][2][0] = hxz; H[c][2][1] = hyz; H[c][2][2] = hzz;
        }
        // u_l = eps_{l k c} d_k psi_c ; J_kl = eps_{l n c} d_k d_n psi_c
        const R u0 = G[2][1] - G[1][2], u1 = G[0][2] - G[2][0], u2 = G[1][0] - G[0][1];
        R J[3][3];
        for (int kk = 0; kk < 3; ++kk) {
            J[kk][0] = H[2][kk][1] - H[1][kk][2];
            J[kk][1] = H[0][kk][2] - H[2][kk][0];
            J[kk][2] = H[1][kk][0] - H[0][kk][1];
        }
        const V4 at = rec[2 * j + 1];
        const R fp = R(12.566370614359172);  // alpha_i = 4 pi * stored (alpha/4pi)
        const R a[3] = {at.x * fp, at.y * fp, at.z * fp};
        R d[3];
        if (scheme == VFMM_SCHEME_TRANSPOSE) {
            for (int kk = 0; kk < 3; ++kk) d[kk] = J[kk][0] * a[0] + J[kk][1] * a[1] + J[kk][2] * a[2];
        } else {
            for (int ll = 0; ll < 3; ++ll) d[ll] = a[0] * J[0][ll] + a[1] * J[1][ll] + a[2] * J[2][ll];
        }
        far_u[j] = u0;
        far_u[n_all + j] = u1;
        far_u[2 * n_all + j] = u2;
        far_da[j] = d[0];
        far_da[n_all + j] = d[1];
        far_da[2 * n_all + j] = d[2];
    }
}

// ---------------------------------------------------------------------------
// Periodic lattice: Lt_root += T Mt_root with the precomputed real operator T
// acting on (Re, Im) of the root coefficients, for each potential.  The
// operator and the arithmetic are in R; the expansions are stored in S.
// ---------------------------------------------------------------------------
template <int P, class R, class S>
__global__ __launch_bounds__(256) void k_lattice(const R *op, const typename VT<S>::V2 *Mexp,
                                                 typename VT<S>::V2 *Lexp) {
    constexpr int NCP = NC(P);
    constexpr int D = 2 * NCP;
    __shared__ R v[3][D];
    for (int i = threadIdx.x; i < 3 * D; i += 256) {
        const int c = i / D, r = i % D;
        const auto mm = Mexp[(size_t)c * NCP + r / 2];
        v[c][r] = (r & 1) ? R(mm.y) : R(mm.x);
    }
    __syncthreads();
    for (int i = threadIdx.x; i < 3 * D; i += 256) {
        const int c = i / D, r = i % D;
        R acc = R(0);
        for (int q = D - 1; q >= 0; --q) acc = fmar(op[(size_t)r * D + q], v[c][q], acc);
        S *dst = reinterpret_cast<S *>(&Lexp[(size_t)c * NCP + r / 2]) + (r & 1);
        *dst = (S)((R)*dst + acc);
    }
}

// zero nw 32-bit words (any count; whole float4 stores except for the tail)
__global__ __launch_bounds__(256) void k_zero(float *p, int64_t nw) {
    const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
    const int64_t w = 4 * i;
    if (w + 4 <= nw) {
        reinterpret_cast<float4 *>(p)[i] = make_float4(0.f, 0.f, 0.f, 0.f);
    } else {
        for (int64_t q = w; q < nw; ++q) p[q] = 0.f;
    }
}

template <int P>
static void far_prealloc_p(Ctx &c) {
    constexpr int NCP = NC(P);
    const size_t rs = c.prm.precision == VFMM_PRECISION_FP64 ? sizeof(double) : sizeof(float);
    const size_t bytes = 2 * rs * (size_t)c.ncells * 3 * NCP;
    c.Mexp.ensure(bytes);
    c.Lexp.ensure(bytes);
    c.far_u.ensure(rs * 3 * (size_t)c.n);
    c.far_da.ensure(rs * 3 * (size_t)c.n);
    c.near.ensure(rs * 6 * (size_t)std::max(c.n_partial, 1));  // the near-field parts
    if (c.prm.precision == VFMM_PRECISION_FP64) c.rec64.ensure(sizeof(double4) * 2 * (size_t)c.n);
    else {
        c.recp.ensure(sizeof(float4) * (c.var_sigma ? 4 : 3) * (size_t)c.n);
    }
}

void far_prealloc(Ctx &c) {
    switch (c.prm.p) {
        case 4: far_prealloc_p<4>(c); break;
        case 6: far_prealloc_p<6>(c); break;
        case 8: far_prealloc_p<8>(c); break;
        case 10: far_prealloc_p<10>(c); break;
        case 12: far_prealloc_p<12>(c); break;
        default: throw Error{VFMM_EINVAL, "unsupported expansion degree p"};
    }
}

// ---------------------------------------------------------------------------
// S: storage and arithmetic type of the expansions, P2M, M2L and L2P;
// RA: arithmetic type of M2M, L2L and the lattice operator.
//   plain float32 <float, float>, mixed <float, double>, float64 <double, double>.
// ---------------------------------------------------------------------------
template <int P, class S, class RA>
static void far_field_t(Ctx &c) {
    using V2 = typename VT<S>::V2;
    using V4 = typename VT<S>::V4;
    hipStream_t s = c.stream;
    constexpr int NCP = NC(P);
    const size_t bytes = sizeof(V2) * (size_t)c.ncells * 3 * NCP;
    c.Mexp.ensure(bytes);
    c.Lexp.ensure(bytes);
    c.far_u.ensure(sizeof(S) * 3 * (size_t)c.n);
    c.far_da.ensure(sizeof(S) * 3 * (size_t)c.n);
    const V4 *rec = (sizeof(S) == 8) ? reinterpret_cast<const V4 *>(c.rec64.ptr) : reinterpret_cast<const V4 *>(c.rec.ptr);
    const double4 *geo = c.c_geo64.as<double4>();
    c.record(2 * PH_P2M_M2M);
    // a fill kernel rather than a memset, so that the evaluation can be captured in a graph
    k_zero<<<cdiv(cdiv(bytes, 16), 256), 256, 0, s>>>(c.Lexp.as<float>(), (int64_t)(bytes / 4));
    VFMM_LAUNCH_CHECK();
    const int *nsrc = eval_sources(c);
    k_p2m<P, S><<<c.nleaves, 64, 0, s>>>(c.leaves.as<int>(), c.c_start.as<int>(), c.c_count.as<int>(), nsrc,
                                         geo, rec, c.Mexp.as<V2>());
    VFMM_LAUNCH_CHECK();
    for (int l = c.depth - 1; l >= 0; --l) {
        const int c0 = c.lvl_off[l], c1 = c.lvl_off[l + 1];
        k_m2m<P, RA, S><<<c1 - c0, XferCfg<P, RA>::M2M_THREADS, 0, s>>>(c0, c1, c.c_child.as<int>(), c.c_nchild.as<int>(),
                                                geo, c.Mexp.as<V2>());
        VFMM_LAUNCH_CHECK();
    }
    c.record(2 * PH_P2M_M2M + 1);
    c.record(2 * PH_LATTICE);
    if (c.prm.periodic && c.prm.images >= 3) {
        k_lattice<P, RA, S><<<1, 256, 0, s>>>(c.lat_op.as<RA>(), c.Mexp.as<V2>(), c.Lexp.as<V2>());
        VFMM_LAUNCH_CHECK();
    }
    c.record(2 * PH_LATTICE + 1);
    c.record(2 * PH_M2L);
    const bool batched = c.n_m2l > 0 && c.m2lb_ok;
    if (batched) m2lb_run(c);
    if (batched ? c.mb_keyed && c.mb_nrest > 0 : c.n_m2l > 0) {  // all translations, or those the plan left out
        const int2 *src = batched ? c.mb_rsrc.as<int2>() : c.m2l_src.as<int2>();
        const int *off = batched ? c.mb_roff.as<int>() : c.m2l_off.as<int>();
        using MC = M2LCfg<P, S>;
        const unsigned bit = 1u << (P / 2 + (sizeof(S) == 8 ? 8 : 0));
        if (MC::LDS > 64 * 1024 && !(c.m2l_lds_set & bit)) {  // once per context (a context lives on one device)
            VFMM_HIP(hipFuncSetAttribute((const void *)k_m2l<P, S>, hipFuncAttributeMaxDynamicSharedMemorySize,
                                         (int)MC::LDS));
            c.m2l_lds_set |= bit;
        }
        k_m2l<P, S><<<c.m2l_nparts, MC::THREADS, MC::LDS, s>>>(c.m2l_parts.as<int4>(), src,
                                                                   geo, c.Mexp.as<V2>(),
                                                                   c.m2l_partial.as<V2>(), c.img_B,
                                                                   c.prm.periodic ? (float)c.prm.box_len : 0.f);
        VFMM_LAUNCH_CHECK();
        k_m2l_add<V2><<<c.ncells, TPB, 0, s>>>(off, c.m2l_part, 3 * NCP, c.m2l_partial.as<V2>(),
                                               c.Lexp.as<V2>());
        VFMM_LAUNCH_CHECK();
    }
    c.record(2 * PH_M2L + 1);
    c.record(2 * PH_L2L_L2P);
    for (int l = 0; l < c.depth; ++l) {  // from the cells of level l to their children
        const int c0 = c.lvl_off[l], c1 = c.lvl_off[l + 1];
        k_l2l<P, RA, S><<<c1 - c0, XferCfg<P, RA>::L2L_THREADS, 0, s>>>(c0, c1, c.c_child.as<int>(),
                                                                        c.c_nchild.as<int>(), geo,
                                                                        c.Lexp.as<V2>());
        VFMM_LAUNCH_CHECK();
    }
    k_l2p<P, S><<<c.nleaves, 64, 0, s>>>(c.leaves.as<int>(), c.c_start.as<int>(), c.c_count.as<int>(),
                                          geo, rec, c.Lexp.as<V2>(), c.n, c.far_u.as<S>(),
                                          c.far_da.as<S>(), c.prm.scheme);
    VFMM_LAUNCH_CHECK();
    c.record(2 * PH_L2L_L2P + 1);
}

template <int P>
static void far_field_p(Ctx &c) {
    switch (c.prm.precision) {
        case VFMM_PRECISION_FP64: far_field_t<P, double, double>(c); break;
        case VFMM_PRECISION_MIXED: far_field_t<P, float, double>(c); break;
        default: far_field_t<P, float, float>(c); break;
    }
}

void far_field(Ctx &c) {
    switch (c.prm.p) {
        case 4: far_field_p<4>(c); break;
        case 6: far_field_p<6>(c); break;
        case 8: far_field_p<8>(c); break;
        case 10: far_field_p<10>(c); break;
        case 12: far_field_p<12>(c); break;
        default: throw Error{VFMM_EINVAL, "unsupported expansion degree p"};
    }
}

}  // namespace vfmm
