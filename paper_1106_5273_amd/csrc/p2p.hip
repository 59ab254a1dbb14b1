// Near field P2P (Sec. 3.1, Sec. 3.6) of the regularised Biot-Savart law and
// the stretching term, Eqs. (1)-(3).  The P2P kernel writes its results in
// sorted order, one buffer per part of the lists (below), and a finalize
// kernel adds the parts and the far field and scatters to the caller's order.
//
// Work item: one wave64 per part (a piece of about equal work) of the P2P list of a block of
// <= 64 targets of a leaf (one target per lane).  Source particles are the
// same for every lane at a given step, so their records are read with scalar
// loads and enter the vector ALU as scalar operands: no LDS staging and no
// cross-lane traffic in the pair loop.  Per-target sums are accumulated per
// source leaf and then added to the running total (blocked summation, with an
// optional compensated add).
//
// Scaled, leaf-local coordinates.  With c = 1/(sqrt 2 sigma) and
// lambda = log2 e, lengths are multiplied by kappa = c sqrt(lambda), so that
// e^{-x} = 2^{-r'^2} for x = (rho/(sqrt 2 sigma))^2 and the Gaussian needs no
// argument scaling.  Each particle's record holds its offset from the centre
// of its own leaf, delta' = kappa (x - c_leaf), and each list entry holds the
// offset between the two leaves, D' = kappa (c_t - c_s - image shift), so
// that r' = (delta'_i + D') - delta'_j = y_i - delta'_j is formed from small
// numbers.  Strengths are stored as ah = kappa^3 alpha/(4 pi), together with
// bh = ah x delta'.
//
// Per pair, with E = 2^{-r2'}, rho' = |r'| and a = (2/sqrt pi)/sqrt(lambda):
//   G3 = 1 - a E (rho' + (1/rho') pe(1/rho'))      = P(3/2, x)
//   G5 = G3 - a E b rho'^3,  b = 2/(3 lambda)       = P(5/2, x)
//   Fh = G3 / rho'^3,  Hh = G5 / rho'^5 = (Fh - a b E) / rho'^2
// where pe is the erfcx fit rescaled to 1/rho' and P(a, x) is the regularised
// lower incomplete gamma function (P(3/2, x) is the cutoff g of Eq. (2)).
// Then, in physical units, q alpha_j x r = Fh (ah_j x r') / kappa and
// (q'/rho)(alpha_i . (alpha_j x r)) r = -3 Hh (alpha_i . (ah_j x r')) r', and
//   transpose reading of Eq. (3):
//     Ah += Fh ah_j,  Bh += Fh bh_j,  T += Hh d r',
//     d = alpha_i . (ah_j x r') = ah_j . (y_i x alpha_i) - alpha_i . bh_j,
//     and per source leaf  U += Ah x y_i - Bh  (= sum Fh ah_j x r');
//   classical reading: U += Fh (ah_j x r'), Ah += Fh ah_j,
//     T += Hh (alpha_i . r') (ah_j x r');
//   u_i = U / kappa,  dalpha_i = alpha_i x Ah - 3 T  (or Ah x alpha_i - 3 T).
// Three forms of the cutoff, chosen per source leaf from the leaf boxes:
//   full : some pair may have s < 1: Kummer series for s < 1, the erfcx form else;
//   mid  : every pair has s >= 1: the erfcx form, no branch;
//   sing : the float32 cutoff is 1 for every pair (s >= 5.1): G3 = G5 = 1/a.
// Per-particle cores use unscaled offsets and evaluate the cutoff at
// kappa_j r with each source's kappa_j (see pair()); a list entry's source
// count covers only the sources of a leaf whose target points were moved
// behind them.
#include <type_traits>

#include "ctx.h"
#include "cutoff_fits.h"

namespace vfmm {

// The launch constant that depends on the core: the strengths are
// kappa^3 alpha/(4 pi) and the velocity sum is scaled back by 1/kappa.
struct P2PConst {
    float inv_kappa; // u = U / kappa
};

// Constants of the scaled cutoff (in the scaled units every one is
// independent of sigma; the normalisation a of the cutoff is in them),
// evaluated at compile time (lam = log2 e, a = (2/sqrt pi) sqrt(ln 2)), so
// that the pair loop takes them as instruction literals (v_fmaak_f32 and the
// like) instead of reading them from registers: a constant in a vector
// register can share a register bank with another operand of the same
// instruction, which halves that instruction's issue rate.
//   a, ab      : a and a b, b = 2/(3 lam)
//   K3         : the series form's Fh at r = 0 (times E)
//   r2_small   : s < 1  <=>  r2' < r2_small
//   pe(i)      : erfcx fit in powers of 1/rho', times a
//   q(i)       : series, Hh = E sum q_k r2'^k,  Fh = E (K3 + r2' sum q_k r2'^k)
namespace cutoff_ce {
constexpr double sqrt_newton(double x) {
    double r = x > 1.0 ? x : 1.0;
    for (int i = 0; i < 200; ++i) r = 0.5 * (r + x / r);
    return r;
}
constexpr double LN2 = 0.693147180559945309417232121458;
constexpr double PI = 3.14159265358979323846264338328;
constexpr double LAM = 1.0 / LN2;
constexpr double SQRT_LAM = sqrt_newton(LAM);
constexpr double SQRT_PI = sqrt_newton(PI);
constexpr double lam_pow_half(int k) {  // lam^(k/2)
    double r = 1.0;
    for (int i = 0; i < k / 2; ++i) r *= LAM;
    return (k & 1) ? r * SQRT_LAM : r;
}
constexpr double A = 2.0 / SQRT_PI * sqrt_newton(LN2);
constexpr float a = (float)A;
constexpr float ab = (float)(A * 2.0 / (3.0 * LAM));
constexpr float K3 = (float)(4.0 / (3.0 * SQRT_PI) / lam_pow_half(3));
constexpr float r2_small = (float)((double)VFMM_CUTOFF_XSPLIT * LAM);
constexpr float pe(int i) { return (float)((double)VFMM_ERFCX_C[i] * lam_pow_half(i + 1)); }
constexpr float q(int i) { return (float)(8.0 / (15.0 * SQRT_PI) * (double)VFMM_M2_C[i] / lam_pow_half(5 + 2 * i)); }
}  // namespace cutoff_ce

// Beside the two stretching schemes: the velocity alone, for target points that
// are no particles (they have no strength to stretch): the pair then takes 21
// vector instructions and two transcendentals instead of 33 and two.  A leaf's
// particles and points are in separate blocks for it.  128^3 particles and as
// many points: near field 31.4 -> 28.8 ms, the evaluation 40.4 -> 37.9.
constexpr int VELOCITY_ONLY = 2;

struct P2PArgs {
    const float4 *__restrict__ rec;  // float4[3n] (uniform cores) or float4[4n] (per-particle cores) records
    const int4 *__restrict__ items;  // (target start, targets, first entry, entries) per wave
    const int *__restrict__ item_out; // tree mode: first partial result of every item
    const int4 *__restrict__ blocks;  // (target start, targets, first partial result, parts)
    const int4 *__restrict__ ent;
    const float4 *__restrict__ sh;   // per entry: (D', 0)
    int item0[5];  // items by kind: whole waves (k_p2p), lane groups (k_p2p_group), the same for the velocity alone
    int kind;      // the kind of this launch
    int velocity;  // target points get the velocity alone
    int nblocks;
    const float *__restrict__ far_u;
    const float *__restrict__ far_da;
    int64_t n;
    const int *__restrict__ perm;
    const Bounds *__restrict__ bounds;
    float inv3V;
    int surface;
    float *ux, *uy, *uz, *dax, *day, *daz;
    float *near;  // tree mode: u and dalpha of an item's targets go to near + 6 item_out, [6][targets]
                  // (the finalize kernel adds the parts of a block)
};

struct Acc9 {
    float u0, u1, u2, a0, a1, a2, t0, t1, t2;
};

// Target-side quantities for one list entry.
struct Tgt {
    float y0, y1, y2;     // y_i = delta'_i + D'
    float w0, w1, w2;     // y_i x alpha_i (transpose reading)
    float ai0, ai1, ai2;  // alpha_i
};

// On gfx950 a run of FP32 VALU operations that read a scalar register issues
// at half the rate of ones whose operands are all vector registers (measured:
// 38.7e12 against 66-74e12 lane operations/s), and so does one whose vector
// operands share a register bank.  The loop-invariant constants of the cutoff
// are instruction literals (cutoff_ce).  The source records stay scalar
// operands: copying them into vector registers every step costs more issue
// slots than it saves.

// VAR (per-source cores): records hold unscaled leaf-local offsets, the
// strengths ah = kappa_j^3 alpha/(4 pi) and kappa_j^2, 1/kappa_j of the source
// in their fourth components.  The cutoff factors are those of the scaled form
// at r' = kappa_j r, and F ah and H (ah . (r x alpha_i)) equal the unscaled
// sums once H carries one more kappa_j^2.
// One pair in three parts, so that a loop over several sources can issue the
// transcendental instructions of all of them back to back (see leaf_loop).
struct Geo {
    float dx, dy, dz;  // r' (scaled) or r (per-source cores)
    float r2;          // |r|^2 in the units of the offsets
    float r2s;         // rho'^2
    float rinv;        // 1 / rho'
    float E;           // 2^{-rho'^2} (not for the singular form)
};

template <bool VAR>
__device__ __forceinline__ void geo_offsets(const Tgt &t, float4 sp, Geo &g) {
    g.dx = t.y0 - sp.x;
    g.dy = t.y1 - sp.y;
    g.dz = t.y2 - sp.z;
    g.r2 = fmaf(g.dx, g.dx, fmaf(g.dy, g.dy, g.dz * g.dz));
    g.r2s = VAR ? g.r2 * sp.w : g.r2;  // rho'^2
}

template <int V, bool VAR>
__device__ __forceinline__ void geo_trans(float4 sa, Geo &g) {
    const float rinv0 = __builtin_amdgcn_rsqf(g.r2);
    g.rinv = VAR ? rinv0 * sa.w : rinv0;  // 1 / rho' (rho' = kappa_j rho)
    if (V != 2) g.E = __builtin_amdgcn_exp2f(-g.r2s);
}

template <int V, int SCHEME, bool VAR>
__device__ __forceinline__ void pair_rest(const P2PConst &k, const Tgt &t, const Geo &g, float4 sp, float4 sa,
                                          float4 sb, Acc9 &p) {
    const float dx = g.dx, dy = g.dy, dz = g.dz;
    const float rinv = g.rinv;
    const float rinv2 = rinv * rinv;
    float F, H;
    if (V == 2) {
        F = rinv2 * rinv;
        H = F * rinv2;
    } else {
        const float r2s = g.r2s;
        const float E = g.E;
        namespace ce = cutoff_ce;
        float pe = ce::pe(VFMM_ERFCX_DEG);
#pragma unroll
        for (int i = VFMM_ERFCX_DEG - 1; i >= 0; --i) pe = fmaf(pe, rinv, ce::pe(i));
        // G3 = 1 - a E (rho' + pe(1/rho')/rho') and G5 = G3 - a b E rho'^3, so that
        // F = G3 / rho'^3 = (1/rho' - E (a + rho'^-2 a pe)) / rho'^2 and
        // H = G5 / rho'^5 = (F - a b E) / rho'^2
        F = rinv2 * fmaf(-E, fmaf(rinv2, pe, ce::a), rinv);
        H = rinv2 * fmaf(-E, ce::ab, F);
        if (V == 0) {
            if (__any(r2s < ce::r2_small)) {
                float q2 = ce::q(VFMM_M2_DEG);
#pragma unroll
                for (int i = VFMM_M2_DEG - 1; i >= 0; --i) q2 = fmaf(q2, r2s, ce::q(i));
                const float Fs = E * fmaf(r2s, q2, ce::K3);  // 2^{-r2'} K3 1F1(1; 5/2; x)
                const float Hs = E * q2;                   // 2^{-r2'} K5 1F1(1; 7/2; x)
                const bool sm = r2s < ce::r2_small;
                F = sm ? Fs : F;
                H = sm ? Hs : H;
            }
        }
    }
    if (SCHEME == VELOCITY_ONLY) {
        p.u0 = fmaf(F, sb.x, p.u0);
        p.u1 = fmaf(F, sb.y, p.u1);
        p.u2 = fmaf(F, sb.z, p.u2);
        p.a0 = fmaf(F, sa.x, p.a0);
        p.a1 = fmaf(F, sa.y, p.a1);
        p.a2 = fmaf(F, sa.z, p.a2);
        return;
    }
    if (VAR) H *= sp.w;  // kappa_j^2
    if (SCHEME == VFMM_SCHEME_TRANSPOSE) {
        float d = fmaf(sa.x, t.w0, fmaf(sa.y, t.w1, sa.z * t.w2));
        d = fmaf(-t.ai0, sb.x, fmaf(-t.ai1, sb.y, fmaf(-t.ai2, sb.z, d)));
        p.u0 = fmaf(F, sb.x, p.u0);
        p.u1 = fmaf(F, sb.y, p.u1);
        p.u2 = fmaf(F, sb.z, p.u2);
        p.a0 = fmaf(F, sa.x, p.a0);
        p.a1 = fmaf(F, sa.y, p.a1);
        p.a2 = fmaf(F, sa.z, p.a2);
        const float hd = H * d;
        p.t0 = fmaf(hd, dx, p.t0);
        p.t1 = fmaf(hd, dy, p.t1);
        p.t2 = fmaf(hd, dz, p.t2);
    } else {
        const float c0 = sa.y * dz - sa.z * dy;
        const float c1 = sa.z * dx - sa.x * dz;
        const float c2 = sa.x * dy - sa.y * dx;
        p.u0 = fmaf(F, c0, p.u0);
        p.u1 = fmaf(F, c1, p.u1);
        p.u2 = fmaf(F, c2, p.u2);
        p.a0 = fmaf(F, sa.x, p.a0);
        p.a1 = fmaf(F, sa.y, p.a1);
        p.a2 = fmaf(F, sa.z, p.a2);
        const float d = fmaf(t.ai0, dx, fmaf(t.ai1, dy, t.ai2 * dz));
        const float hd = H * d;
        p.t0 = fmaf(hd, c0, p.t0);
        p.t1 = fmaf(hd, c1, p.t1);
        p.t2 = fmaf(hd, c2, p.t2);
    }
}

template <int V, int SCHEME, bool VAR>
__device__ __forceinline__ void pair(const P2PConst &k, const Tgt &t, float4 sp, float4 sa, float4 sb, Acc9 &p) {
    Geo g;
    geo_offsets<VAR>(t, sp, g);
    geo_trans<V, VAR>(sa, g);
    pair_rest<V, SCHEME, VAR>(k, t, g, sp, sa, sb, p);
}

// One group of U sources against the lane's target: the offsets of all U
// pairs, then their transcendental instructions back to back, then the rest.
// On gfx950 two waves issue their vector instructions together (about two
// clocks each) unless a scalar-register operand, a bank conflict or a nearby
// v_rsq/v_exp stops the pairing; a v_rsq/v_exp spread among the other
// instructions slows them more than the same instructions issued together.
// The scheduling barriers keep the compiler from spreading them again.
template <int V, int SCHEME, bool VAR, int U>
__device__ __forceinline__ void trip(const P2PConst &k, const Tgt &t, const float4 *sp, const float4 *sa,
                                     const float4 *sb, Acc9 &p) {
    Geo g[U];
#pragma unroll
    for (int u = 0; u < U; ++u) geo_offsets<VAR>(t, sp[u], g[u]);
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int u = 0; u < U; ++u) geo_trans<V, VAR>(sa[u], g[u]);
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int u = 0; u < U; ++u) pair_rest<V, SCHEME, VAR>(k, t, g[u], sp[u], sa[u], sb[u], p);
}

// All sources of one list entry, two per trip.  The scalar loads of the next
// trip's records are issued before the current trip is evaluated (the last
// full trip's records are loaded twice), so that their latency is covered by
// the trip's arithmetic instead of stalling the wave at the top of each trip.
// The sums are taken in source order whatever the grouping.
template <int V, int SCHEME, bool VAR>
__device__ __forceinline__ void leaf_loop(const P2PConst &k, const float4 *__restrict__ rec, int s0, int cnt,
                                          const Tgt &t, Acc9 &p) {
    constexpr int RS = VAR ? 4 : 3;  // float4 per record
    constexpr int U = 2;
    const float4 *src = rec + RS * (size_t)s0;
    int j = 0;
    if (cnt >= U) {
        const int jlast = cnt - U;
        float4 np[U], na[U], nb[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            np[u] = src[RS * u];
            na[u] = src[RS * u + 1];
            nb[u] = src[RS * u + 2];
        }
        for (; j + U <= cnt; j += U) {
            float4 sp[U], sa[U], sb[U];
#pragma unroll
            for (int u = 0; u < U; ++u) {
                sp[u] = np[u];
                sa[u] = na[u];
                sb[u] = nb[u];
            }
            const int jn = min(j + U, jlast);
#pragma unroll
            for (int u = 0; u < U; ++u) {
                np[u] = src[RS * (jn + u)];
                na[u] = src[RS * (jn + u) + 1];
                nb[u] = src[RS * (jn + u) + 2];
            }
            trip<V, SCHEME, VAR, U>(k, t, sp, sa, sb, p);
        }
    }
    if (j < cnt) pair<V, SCHEME, VAR>(k, t, src[RS * j], src[RS * j + 1], src[RS * j + 2], p);
}

__device__ __forceinline__ void kahan_add(float &s, float &c, float v) {
    const float y = v - c;
    const float t = s + y;
    c = (t - s) - y;
    s = t;
}

// Sums that are compensated within a wave are put together from several in float64.
template <bool KAHAN>
using Acc = std::conditional_t<KAHAN, double, float>;

template <bool KAHAN>
__device__ __forceinline__ Acc<KAHAN> kahan_value(float s, float c) {
    return KAHAN ? (Acc<KAHAN>)s - (Acc<KAHAN>)c : (Acc<KAHAN>)s;
}

// Target of a lane: its offset in its leaf and its strength.
template <bool VAR>
__device__ __forceinline__ float4 load_target(const P2PArgs &A, int i, Tgt &t) {
    float4 r0;
    if (VAR) {
        r0 = A.rec[4 * (size_t)i];
        const float4 r3 = A.rec[4 * (size_t)i + 3];
        t.ai0 = r3.x;
        t.ai1 = r3.y;
        t.ai2 = r3.z;
    } else {
        r0 = A.rec[3 * (size_t)i];
        t.ai0 = r0.w;
        t.ai1 = A.rec[3 * (size_t)i + 1].w;
        t.ai2 = A.rec[3 * (size_t)i + 2].w;
    }
    return r0;
}

template <int SCHEME>
__device__ __forceinline__ void set_offset(float4 r0, float4 D, Tgt &t) {
    t.y0 = r0.x + D.x;
    t.y1 = r0.y + D.y;
    t.y2 = r0.z + D.z;
    if (SCHEME == VFMM_SCHEME_TRANSPOSE) {
        t.w0 = t.y1 * t.ai2 - t.y2 * t.ai1;
        t.w1 = t.y2 * t.ai0 - t.y0 * t.ai2;
        t.w2 = t.y0 * t.ai1 - t.y1 * t.ai0;
    }
}

// adds one source leaf's sums to the running totals
template <int SCHEME, bool KAHAN>
__device__ __forceinline__ void add_leaf(const Tgt &t, const Acc9 &p, float *S, float *Cc) {
    float u0 = p.u0, u1 = p.u1, u2 = p.u2;
    if (SCHEME != VFMM_SCHEME_CLASSICAL) {  // Ah x y_i - Bh
        u0 = fmaf(p.a1, t.y2, fmaf(-p.a2, t.y1, -p.u0));
        u1 = fmaf(p.a2, t.y0, fmaf(-p.a0, t.y2, -p.u1));
        u2 = fmaf(p.a0, t.y1, fmaf(-p.a1, t.y0, -p.u2));
    }
    const float pv[9] = {u0, u1, u2, p.a0, p.a1, p.a2, p.t0, p.t1, p.t2};
    if (KAHAN) {
#pragma unroll
        for (int q = 0; q < 9; ++q) kahan_add(S[q], Cc[q], pv[q]);
    } else {
#pragma unroll
        for (int q = 0; q < 9; ++q) S[q] += pv[q];
    }
}

// u and dalpha of target i (number tl of its block of tc) from the sums S: a
// partial result when near is given, else (direct mode) the outputs
template <int SCHEME>
__device__ __forceinline__ void finish(const P2PConst &k, const P2PArgs &A, int i, int tl, int tc, const Tgt &t,
                                       const float *S, float *near) {
    if (SCHEME == VELOCITY_ONLY) {
        near[tl] = S[0] * k.inv_kappa;
        near[tc + tl] = S[1] * k.inv_kappa;
        near[2 * tc + tl] = S[2] * k.inv_kappa;
        return;
    }
    const float ai0 = t.ai0, ai1 = t.ai1, ai2 = t.ai2;
    // dalpha = alpha_i x A - 3 T (transpose) or A x alpha_i - 3 T (classical)
    float d0, d1, d2;
    if (SCHEME == VFMM_SCHEME_TRANSPOSE) {
        d0 = ai1 * S[5] - ai2 * S[4];
        d1 = ai2 * S[3] - ai0 * S[5];
        d2 = ai0 * S[4] - ai1 * S[3];
    } else {
        d0 = S[4] * ai2 - S[5] * ai1;
        d1 = S[5] * ai0 - S[3] * ai2;
        d2 = S[3] * ai1 - S[4] * ai0;
    }
    d0 = fmaf(-3.0f, S[6], d0);
    d1 = fmaf(-3.0f, S[7], d1);
    d2 = fmaf(-3.0f, S[8], d2);
    float u0 = S[0] * k.inv_kappa, u1 = S[1] * k.inv_kappa, u2 = S[2] * k.inv_kappa;
    if (near) {
        near[tl] = u0;
        near[tc + tl] = u1;
        near[2 * tc + tl] = u2;
        near[3 * tc + tl] = d0;
        near[4 * tc + tl] = d1;
        near[5 * tc + tl] = d2;
        return;
    }
    if (A.bounds->stale) u0 = u1 = u2 = d0 = d1 = d2 = __builtin_nanf("");  // positions differ from the build's
    A.ux[i] = u0;
    A.uy[i] = u1;
    A.uz[i] = u2;
    A.dax[i] = d0;
    A.day[i] = d1;
    A.daz[i] = d2;
}

// A block of more than 32 targets: a lane per target, sources as scalar operands.
template <int SCHEME, bool KAHAN, bool VAR>
__device__ __forceinline__ void p2p_block(const P2PConst &k, const P2PArgs &A, int t0, int tc, int l0, int lc,
                                          float *near) {
    const int lane = threadIdx.x & 63;
    const bool valid = lane < tc;
    const int i = t0 + (valid ? lane : 0);
    Tgt t;
    const float4 r0 = load_target<VAR>(A, i, t);
    float S[9] = {0, 0, 0, 0, 0, 0, 0, 0, 0};
    float Cc[9] = {0, 0, 0, 0, 0, 0, 0, 0, 0};
    for (int e = 0; e < lc; ++e) {
        const int4 en = A.ent[l0 + e];
        const int s0 = __builtin_amdgcn_readfirstlane(en.x);
        const int sc = __builtin_amdgcn_readfirstlane(en.y);
        const int var = __builtin_amdgcn_readfirstlane(en.w);
        set_offset<SCHEME>(r0, A.sh[l0 + e], t);
        Acc9 p = {0, 0, 0, 0, 0, 0, 0, 0, 0};
        if (var == 1)
            leaf_loop<1, SCHEME, VAR>(k, A.rec, s0, sc, t, p);
        else if (var == 0)
            leaf_loop<0, SCHEME, VAR>(k, A.rec, s0, sc, t, p);
        else
            leaf_loop<2, SCHEME, VAR>(k, A.rec, s0, sc, t, p);
        add_leaf<SCHEME, KAHAN>(t, p, S, Cc);
    }
    if (valid) finish<SCHEME>(k, A, i, lane, tc, t, S, near);
}

// A block of at most 32 targets.  With a lane per target most of the wave would
// idle, so ng = p2p_groups(tc) groups of tc lanes each hold every target and
// take every ng-th source.  Scalar loads cannot give the groups different
// sources, and vector loads of them pass the L1 separately for every lane, so
// the wave stages 64 sources at a time in LDS, one per lane, and the groups
// read them back as broadcasts.  The list is taken as one stream of sources,
// 64 entries at a time: a prefix sum of the entries' source counts tells each
// lane which source it stages (a binary search), so that the groups always
// have equal work whatever the leaves' sizes, and a lane moves its source into
// the target leaf's frame as it stages it (delta_j - D', and ah x of it), so
// that there is no work per entry left in the pair loop.  Lanes past the end of
// the stream stage the last source, which is of the same pass, without its
// strength: the pass's form of the cutoff is finite for its pairs, so it contributes
// exactly zero (a record at a place of its own could meet a target).
// Bound by VALU issue like the scalar form (70 of about 85 instructions per
// trip of two sources are pair arithmetic).  An 80^3 jittered lattice (15.6
// particles per leaf, 2.88e9 pairs): 7.1 ms with groups of 16 or 32 lanes that
// read every source from memory, 4.6 ms with groups that take whole entries
// from LDS, 2.7 ms so; per-particle cores at 50^3 (27 to 64 per leaf): 1.8,
// 1.6 and 1.2 ms.
struct GroupLds {
    float4 rec[3 * 64];  // staged records
    float4 hd[64];       // D' of an entry; its first source less the sources before it
    int incl[64];        // inclusive prefix sum of the source counts
    int form[64];        // cutoff form
};

template <int V, int SCHEME, bool VAR>
__device__ __forceinline__ void group_loop(const P2PConst &k, const float4 *stage, int ng, int trips, const Tgt &t,
                                           Acc9 &p) {
    for (int j = 0; j < trips; ++j) {
        float4 sp[2], sa[2], sb[2];
#pragma unroll
        for (int u = 0; u < 2; ++u) {
            sp[u] = stage[0];
            sa[u] = stage[1];
            sb[u] = stage[2];
            stage += 3 * ng;
        }
        trip<V, SCHEME, VAR, 2>(k, t, sp, sa, sb, p);
    }
}

template <int SCHEME, bool KAHAN, bool VAR>
__device__ __forceinline__ void p2p_group(const P2PConst &k, const P2PArgs &A, int t0, int tc, int l0, int lc,
                                          float *near, GroupLds &L) {
    constexpr int RS = VAR ? 4 : 3;
    const int lane = threadIdx.x & 63;
    const int ng = p2p_groups(tc);
    const int chunk = ((64 / ng) & ~1) * ng;  // sources per pass: an even number per group
    const int g0 = (int)(((float)lane + 0.5f) / (float)tc);
    const int grp = min(g0, ng - 1);          // lanes past the last group repeat its reads
    const int tl = lane - g0 * tc;
    const int i = t0 + tl;
    Tgt t;
    const float4 r0 = load_target<VAR>(A, i, t);
    set_offset<SCHEME>(r0, make_float4(0.f, 0.f, 0.f, 0.f), t);
    float S[9] = {0, 0, 0, 0, 0, 0, 0, 0, 0};
    float Cc[9] = {0, 0, 0, 0, 0, 0, 0, 0, 0};
    for (int b = 0; b < lc; b += 64) {
        const bool has = b + lane < lc;
        const int4 en = has ? A.ent[l0 + b + lane] : make_int4(0, 0, 0, 2);
        const float4 D = has ? A.sh[l0 + b + lane] : make_float4(0.f, 0.f, 0.f, 0.f);
        int x = en.y;  // inclusive prefix sum
#pragma unroll
        for (int o = 1; o < 64; o <<= 1) {
            const int y = __shfl_up(x, o, 64);
            if (lane >= o) x += y;
        }
        const int total = __builtin_amdgcn_readlane(x, 63);
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");  // LDS order within the wave
        L.hd[lane] = make_float4(D.x, D.y, D.z, __int_as_float(en.x - (x - en.y)));
        L.incl[lane] = x;
        L.form[lane] = en.w;
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        for (int f0 = 0; f0 < total; f0 += chunk) {
            const int f = f0 + lane;
            const bool ok = lane < chunk && f < total;
            const int ff = ok ? f : total - 1;
            int e = 0;  // the first entry whose inclusive sum exceeds ff
#pragma unroll
            for (int o = 32; o > 0; o >>= 1)
                if (L.incl[e + o - 1] <= ff) e += o;
            const float4 h = L.hd[e];
            const int form = ok ? L.form[e] : 2;
            const float4 *src = A.rec + RS * (size_t)(__float_as_int(h.w) + ff);
            float4 sp = src[0], sa = src[1], sb = src[2];
            // into the target leaf's frame
            sp.x -= h.x;
            sp.y -= h.y;
            sp.z -= h.z;
            sb.x = fmaf(sa.z, h.y, fmaf(-sa.y, h.z, sb.x));
            sb.y = fmaf(sa.x, h.z, fmaf(-sa.z, h.x, sb.y));
            sb.z = fmaf(sa.y, h.x, fmaf(-sa.x, h.y, sb.z));
            if (!ok) {  // the last source again without its strength: its form holds for it
                sa = make_float4(0.f, 0.f, 0.f, sa.w);
                sb = make_float4(0.f, 0.f, 0.f, sb.w);
            }
            // the form that every staged source allows
            const int any0 = __any(form == 0), any1 = __any(form == 1);
            const int own = __any(ok && h.x == 0.f && h.y == 0.f && h.z == 0.f);  // of the target leaf
            __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");  // the last pass has read its records
            L.rec[3 * lane] = sp;
            L.rec[3 * lane + 1] = sa;
            L.rec[3 * lane + 2] = sb;
            __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
            const int trips = (min(chunk, total - f0) + 2 * ng - 1) / (2 * ng);
            const float4 *stage = L.rec + 3 * grp;
            // A particle's own term is zero in u, but as the difference of two sums it cancels only
            // to their rounding, and with a small core it is many times a neighbour's: the passes of
            // the target leaf take it source by source, before anything is added to it (in the
            // classical reading u has no such difference, but compensated sums would lose theirs).
            if (own && (KAHAN || SCHEME != VFMM_SCHEME_CLASSICAL)) {
                for (int j = 0; j < 2 * trips; ++j, stage += 3 * ng) {
                    Acc9 p = {0, 0, 0, 0, 0, 0, 0, 0, 0};
                    pair<0, SCHEME, VAR>(k, t, stage[0], stage[1], stage[2], p);
                    add_leaf<SCHEME, KAHAN>(t, p, S, Cc);
                }
                continue;
            }
            Acc9 p = {0, 0, 0, 0, 0, 0, 0, 0, 0};
            if (any0)
                group_loop<0, SCHEME, VAR>(k, stage, ng, trips, t, p);
            else if (any1)
                group_loop<1, SCHEME, VAR>(k, stage, ng, trips, t, p);
            else
                group_loop<2, SCHEME, VAR>(k, stage, ng, trips, t, p);
            add_leaf<SCHEME, KAHAN>(t, p, S, Cc);
        }
    }
    // the groups' sums, added pairwise
#pragma unroll
    for (int q = 0; q < 9; ++q) {
        Acc<KAHAN> v = kahan_value<KAHAN>(S[q], Cc[q]);
        for (int w = 1; w < ng; w <<= 1) {
            const Acc<KAHAN> x = __shfl(v, (lane + w * tc) & 63, 64);
            if (g0 % (2 * w) == 0 && g0 + w < ng) v += x;
        }
        S[q] = (float)v;
    }
    if (lane < tc) finish<SCHEME>(k, A, i, tl, tc, t, S, near);
}

// One wave per item; neighbouring waves take the parts of one block (they share
// its target records and much of its source data in the caches).  The two kinds
// of blocks are two kernels: the group form needs 74 vector registers, which
// would cost the scalar form (51) two of its eight waves per SIMD.
__device__ __forceinline__ bool load_item(const P2PArgs &A, int item0, int item1, int &t0, int &tc, int &l0, int &lc,
                                          float *&near) {
    const int j = xcd_logical(blockIdx.x, gridDim.x) * 4 + (threadIdx.x >> 6);
    const int item = item0 + j;
    if (item >= item1) return false;
    const int4 it = A.items[item];
    t0 = __builtin_amdgcn_readfirstlane(it.x);
    tc = __builtin_amdgcn_readfirstlane(it.y);
    l0 = __builtin_amdgcn_readfirstlane(it.z);
    lc = __builtin_amdgcn_readfirstlane(it.w);
    near = A.near + 6 * (size_t)__builtin_amdgcn_readfirstlane(A.item_out[item]);
    return true;
}

template <int SCHEME, bool KAHAN, bool VAR>
__global__ __launch_bounds__(256) void k_p2p(P2PConst k, P2PArgs A) {
    int t0, tc, l0, lc;
    float *near;
    if (load_item(A, A.item0[A.kind], A.item0[A.kind + 1], t0, tc, l0, lc, near))
        p2p_block<SCHEME, KAHAN, VAR>(k, A, t0, tc, l0, lc, near);
}

template <int SCHEME, bool KAHAN, bool VAR>
__global__ __launch_bounds__(256) void k_p2p_group(P2PConst k, P2PArgs A) {
    __shared__ GroupLds lds[4];
    int t0, tc, l0, lc;
    float *near;
    if (load_item(A, A.item0[A.kind], A.item0[A.kind + 1], t0, tc, l0, lc, near))
        p2p_group<SCHEME, KAHAN, VAR>(k, A, t0, tc, l0, lc, near, lds[threadIdx.x >> 6]);
}

// Records of the float32 near field (sorted order), one wave per leaf.
// Uniform cores (kappa the scale of the shared core):
//   rec[3i] = (kappa (x_i - c_leaf), alpha_x), rec[3i+1] = (ah_i, alpha_y),
//   rec[3i+2] = (ah_i x delta'_i, alpha_z),   ah = kappa^3 alpha/(4 pi).
// Per-source cores (kappa_j of each particle's own core):
//   rec[4i] = (x_i - c_leaf, kappa_i^2), rec[4i+1] = (ah_i, 1/kappa_i),
//   rec[4i+2] = (ah_i x delta_i, kappa_i^3), rec[4i+3] = (alpha_i, 0),  ah = kappa_i^3 alpha/(4 pi).
// Computed in float64 and rounded once.
template <bool VAR>
__device__ __forceinline__ void put_record(float4 *__restrict__ out, int64_t i, double d0, double d1, double d2,
                                           double kap, double a0, double a1, double a2, float al0, float al1,
                                           float al2) {
    const double s3 = kap * kap * kap;  // a: alpha / (4 pi)
    const double h0 = s3 * a0, h1 = s3 * a1, h2 = s3 * a2;
    const double b0 = h1 * d2 - h2 * d1, b1 = h2 * d0 - h0 * d2, b2 = h0 * d1 - h1 * d0;
    if (VAR) {
        out[4 * i] = make_float4((float)d0, (float)d1, (float)d2, (float)(kap * kap));
        out[4 * i + 1] = make_float4((float)h0, (float)h1, (float)h2, (float)(1.0 / kap));
        out[4 * i + 2] = make_float4((float)b0, (float)b1, (float)b2, (float)s3);
        out[4 * i + 3] = make_float4(al0, al1, al2, 0.f);
    } else {
        out[3 * i] = make_float4((float)d0, (float)d1, (float)d2, al0);
        out[3 * i + 1] = make_float4((float)h0, (float)h1, (float)h2, al1);
        out[3 * i + 2] = make_float4((float)b0, (float)b1, (float)b2, al2);
    }
}

template <bool VAR>
__global__ __launch_bounds__(256) void k_p2p_records(const int *__restrict__ leaves, int nleaves,
                                                     const int *__restrict__ start, const int *__restrict__ count,
                                                     const float4 *__restrict__ geo, double kappa,
                                                     const float4 *__restrict__ rec_in, float4 *__restrict__ out) {
    const int w = blockIdx.x * 4 + (threadIdx.x >> 6);
    if (w >= nleaves) return;
    const int cell = leaves[w];
    const int64_t i0 = start[cell], i1 = i0 + count[cell];
    const float4 g = geo[cell];
    const double fp = 12.566370614359172954;  // 4 pi: rec_in holds alpha/(4 pi)
    for (int64_t i = i0 + (threadIdx.x & 63); i < i1; i += 64) {
        const float4 p = rec_in[2 * i], a = rec_in[2 * i + 1];
        // VAR: kappa argument = sqrt(log2 e)/sqrt(2), divided by each core
        const double kap = VAR ? kappa / (double)p.w : kappa;
        const double sc = VAR ? 1.0 : kappa;
        put_record<VAR>(out, i, sc * ((double)p.x - g.x), sc * ((double)p.y - g.y), sc * ((double)p.z - g.z), kap,
                        a.x, a.y, a.z, (float)(fp * a.x), (float)(fp * a.y), (float)(fp * a.z));
    }
}

// ---------------------------------------------------------------------------
// Float64 reference form: the same work items and lists, every quantity in
// double and the cutoff always in its full form:
//   F = P(3/2, x)/rho^3,  H = P(5/2, x)/rho^5,  x = c^2 rho^2,  c = 1/(sqrt 2 sigma_j)
// of the source's own core (c^2 and c^3 in the fourth components of its record).
// For x < 3 the power series of the lower incomplete gamma function,
//   P(a, x) = x^a e^{-x} sum_k x^k / Gamma(a + k + 1),
// divided by rho^{2a}, gives F and H without cancellation (finite at rho = 0);
// the sum for a = 5/2 is a fitted polynomial (relative error 5e-17 with its
// coefficients as doubles), the one for 3/2 follows from it.  For x >= 3, with
// u = x^{-1/2},
//   1 - P(3/2, x) = e^{-x} (u Pe(u) + (2/sqrt pi) / u),  Pe(1/s) = s erfcx(s),
// Pe fitted for 3 <= x <= 43 (it changes P by less than 2e-17), and
// P(5/2, x) = P(3/2, x) - (4/(3 sqrt pi)) x^{3/2} e^{-x}; beyond x = 43 both are 1
// to double precision.  Bound by float64 VALU issue (4 clocks an instruction):
// about 75 instructions per pair in place of the library's exp, erfc and sqrt
// and a series of up to 60 divisions (64^3 lattice, 2.47e9 pairs: 21.4 -> 7.3 ms).
// ---------------------------------------------------------------------------
struct P2P64Args {
    const double4 *__restrict__ rec;
    const int4 *__restrict__ items;
    const int *__restrict__ item_out;
    const int4 *__restrict__ blocks;  // (target start, targets, first partial result, parts)
    const int4 *__restrict__ ent;
    int nitems, nblocks;
    int n_long;  // > 0: the blocks of many parts are summed into their first
    int B;
    double len;
    double *near;  // partial results, [6][targets] per item
    const double *__restrict__ far_u;
    const double *__restrict__ far_da;
    int64_t n;
    const int *__restrict__ perm;
    const Bounds *__restrict__ bounds;
    double inv3V;
    int surface;
    float *ux, *uy, *uz, *dax, *day, *daz;
};

// a b + k with the constant k in scalar registers: left to itself the compiler
// keeps the polynomials' constants in vector registers (168 in all, three waves
// per SIMD) and copies each into the accumulator first (a v_mov_b64 per v_fmac_f64)
__device__ __forceinline__ double fma_const(double a, double b, double k) {
    double d;
    asm("v_fma_f64 %0, %1, %2, %3" : "=v"(d) : "v"(a), "v"(b), "s"(k));
    return d;
}

// e^{-x}, x >= 0: 2^n e^r with |r| <= ln 2 / 2 and e^r by its Taylor sum.  Zero
// from x = 745 on; larger x are cut off, as r would grow with their rounding.
__device__ __forceinline__ double exp_minus(double x) {
    x = fmin(x, 800.0);
    const double n = __builtin_rint(-1.4426950408889634 * x);
    double r = fma(n, -VFMM64_LN2_HI, -x);
    r = fma(n, -VFMM64_LN2_LO, r);
    double p = 1.0 / 6227020800.0;
    p = fma_const(p, r, 1.0 / 479001600.0);
    p = fma_const(p, r, 1.0 / 39916800.0);
    p = fma_const(p, r, 1.0 / 3628800.0);
    p = fma_const(p, r, 1.0 / 362880.0);
    p = fma_const(p, r, 1.0 / 40320.0);
    p = fma_const(p, r, 1.0 / 5040.0);
    p = fma_const(p, r, 1.0 / 720.0);
    p = fma_const(p, r, 1.0 / 120.0);
    p = fma_const(p, r, 1.0 / 24.0);
    p = fma_const(p, r, 1.0 / 6.0);
    p = fma_const(p, r, 0.5);
    p = fma_const(p, r, 1.0);
    p = fma_const(p, r, 1.0);
    return ldexp(p, (int)n);
}

// P(3/2, x)/x^{3/2} and P(5/2, x)/x^{5/2}
__device__ __forceinline__ void cutoff64(double x, double &F, double &H) {
    // x^{-1/2}: the hardware's estimate and one third-order step
    double u = __builtin_amdgcn_rsq(x);
    const double d = fma(-x * u, u, 1.0);
    u = fma(u * d, fma(d, 0.375, 0.5), u);
    const double u2 = u * u;
    F = u2 * u;
    H = F * u2;
    const bool near = x < VFMM64_XSPLIT;
    if (!__any(x < VFMM64_XMAX)) return;
    const double e = exp_minus(x);
    if (__any(!near)) {
        const double t = fma(u, VFMM64_PE_SCALE, VFMM64_PE_SHIFT);
        constexpr int DEG = sizeof(VFMM64_PE_C) / sizeof(double) - 1;
        double pe = VFMM64_PE_C[DEG];
#pragma unroll
        for (int k = DEG - 1; k >= 0; --k) pe = fma_const(pe, t, VFMM64_PE_C[k]);
        const double q = fma(u, pe, 1.1283791670955125739 * (x * u));  // (1 - P(3/2, x)) e^x
        F *= fma(-e, q, 1.0);
        H = u2 * fma(-0.75225277806367504925, e, F);  // 4 / (3 sqrt pi)
    }
    if (__any(near)) {
        constexpr int DEG = sizeof(VFMM64_M2_C) / sizeof(double) - 1;
        double s = VFMM64_M2_C[DEG];
#pragma unroll
        for (int k = DEG - 1; k >= 0; --k) s = fma_const(s, x, VFMM64_M2_C[k]);
        const double Fs = e * fma(x, s, 0.75225277806367504925);  // 1/Gamma(5/2)
        F = near ? Fs : F;
        H = near ? e * s : H;
    }
}

template <int SCHEME>
__device__ __forceinline__ void pair64(double xi, double yi, double zi, double ai0, double ai1, double ai2, double4 sp,
                                       double4 sa, bool ok, double *S) {
    const double dx = xi - sp.x, dy = yi - sp.y, dz = zi - sp.z;
    double F, H;
    cutoff64((dx * dx + dy * dy + dz * dz) * sp.w, F, H);
    F *= ok ? sa.w : 0.0;              // c^3
    H *= ok ? sa.w * sp.w : 0.0;       // c^5
    const double c0 = sa.y * dz - sa.z * dy;
    const double c1 = sa.z * dx - sa.x * dz;
    const double c2 = sa.x * dy - sa.y * dx;
    S[0] += F * c0;
    S[1] += F * c1;
    S[2] += F * c2;
    S[3] += F * sa.x;
    S[4] += F * sa.y;
    S[5] += F * sa.z;
    if (SCHEME == VFMM_SCHEME_TRANSPOSE) {
        const double hd = H * (ai0 * c0 + ai1 * c1 + ai2 * c2);
        S[6] += hd * dx;
        S[7] += hd * dy;
        S[8] += hd * dz;
    } else {
        const double hd = H * (ai0 * dx + ai1 * dy + ai2 * dz);
        S[6] += hd * c0;
        S[7] += hd * c1;
        S[8] += hd * c2;
    }
}

// One wave per item, as in the float32 form; the lane groups of a small block
// take every ng-th source of each entry.
template <int SCHEME>
__global__ __launch_bounds__(256) void k_p2p64(P2P64Args A) {
    const int item = xcd_logical(blockIdx.x, gridDim.x) * 4 + (threadIdx.x >> 6);
    if (item >= A.nitems) return;
    const int lane = threadIdx.x & 63;
    const int4 it = A.items[item];
    const int t0 = __builtin_amdgcn_readfirstlane(it.x), tc = __builtin_amdgcn_readfirstlane(it.y);
    const int l0 = __builtin_amdgcn_readfirstlane(it.z), lc = __builtin_amdgcn_readfirstlane(it.w);
    const int ng = p2p_groups(tc);
    const int g0 = ng > 1 ? (int)(((float)lane + 0.5f) / (float)tc) : 0;
    const int tl = lane - g0 * tc;
    const bool member = ng > 1 ? g0 < ng : lane < tc;  // lanes past the last group (or target) add nothing
    const int i = t0 + min(tl, tc - 1);
    const double4 xp = A.rec[2 * (size_t)i];
    const double4 xa = A.rec[2 * (size_t)i + 1];
    const double fp = 12.566370614359172954;  // 4 pi
    const double ai0 = xa.x * fp, ai1 = xa.y * fp, ai2 = xa.z * fp;
    double S[9] = {0, 0, 0, 0, 0, 0, 0, 0, 0};
    const int W = 2 * A.B + 1;
    for (int e = l0; e < l0 + lc; ++e) {
        const int4 en = A.ent[e];
        const int s0 = __builtin_amdgcn_readfirstlane(en.x), sc = __builtin_amdgcn_readfirstlane(en.y);
        const double xi = xp.x - (double)(en.z % W - A.B) * A.len;
        const double yi = xp.y - (double)((en.z / W) % W - A.B) * A.len;
        const double zi = xp.z - (double)(en.z / (W * W) - A.B) * A.len;
        if (ng == 1) {
            for (int j = s0; j < s0 + sc; ++j)
                pair64<SCHEME>(xi, yi, zi, ai0, ai1, ai2, A.rec[2 * (size_t)j], A.rec[2 * (size_t)j + 1], true, S);
        } else {
            for (int j0 = 0; j0 < sc; j0 += ng) {
                const bool ok = member && j0 + g0 < sc;
                const int j = s0 + (ok ? j0 + g0 : 0);
                pair64<SCHEME>(xi, yi, zi, ai0, ai1, ai2, A.rec[2 * (size_t)j], A.rec[2 * (size_t)j + 1], ok, S);
            }
        }
    }
    if (ng > 1) {
#pragma unroll
        for (int q = 0; q < 9; ++q) {
            double v = S[q];
            for (int g = 1; g < ng; ++g) v += __shfl(S[q], (lane + g * tc) & 63, 64);
            S[q] = v;
        }
    }
    if (lane >= tc) return;
    double d0, d1, d2;
    if (SCHEME == VFMM_SCHEME_TRANSPOSE) {
        d0 = ai1 * S[5] - ai2 * S[4];
        d1 = ai2 * S[3] - ai0 * S[5];
        d2 = ai0 * S[4] - ai1 * S[3];
    } else {
        d0 = S[4] * ai2 - S[5] * ai1;
        d1 = S[5] * ai0 - S[3] * ai2;
        d2 = S[3] * ai1 - S[4] * ai0;
    }
    double *near = A.near + 6 * (size_t)A.item_out[item];
    near[lane] = S[0];
    near[tc + lane] = S[1];
    near[2 * tc + lane] = S[2];
    near[3 * tc + lane] = d0 - 3.0 * S[6];
    near[4 * tc + lane] = d1 - 3.0 * S[7];
    near[5 * tc + lane] = d2 - 3.0 * S[8];
}

// Blocks of many parts: the parts of block pblong[blockIdx.x] are summed into the
// first, one result component (blockIdx.y) per work-group, by up to 64 groups of
// as many threads as the block has targets (parts g, g + groups, ...; then the
// groups in order; A: the sums' type).  A wave per block in k_finalize adds them one after another:
// with 1,600 parts for a lone particle beside a cluster that chain took 570 us of
// the 100,003-particle clustered evaluation, with the parts summed here 30.
template <class T, class A>
__global__ __launch_bounds__(1024) void k_sum_parts(const int4 *__restrict__ blocks, const int *__restrict__ pblong,
                                                    T *__restrict__ near) {
    __shared__ A red[1024];
    const int4 blk = blocks[pblong[blockIdx.x]];
    const int tc = blk.y, np = blk.w & PBLOCK_PARTS, t = threadIdx.x;
    const int G = min(64, 1024 / tc), g = t / tc, e = t - g * tc;
    T *q = near + 6 * (size_t)blk.z + (size_t)blockIdx.y * tc;
    const size_t stride = 6 * (size_t)tc;
    A v = 0;
    if (g < G)
        for (int p0 = g; p0 < np; p0 += 8 * G) {
            T w[8];
#pragma unroll
            for (int k = 0; k < 8; ++k) w[k] = p0 + k * G < np ? q[(size_t)(p0 + k * G) * stride + e] : T(0);
#pragma unroll
            for (int k = 0; k < 8; ++k) v += w[k];
        }
    red[t] = v;
    __syncthreads();
    if (t < tc) {
        for (int k = 1; k < G; ++k) v += red[k * tc + t];
        q[t] = (T)v;
    }
}

template <class T, class A>
static void sum_parts(Ctx &c) {
    if (c.n_long == 0) return;
    k_sum_parts<T, A>
        <<<dim3(c.n_long, 6), 1024, 0, c.stream>>>(c.pblocks.as<int4>(), c.pblong.as<int>(), c.near.as<T>());
    VFMM_LAUNCH_CHECK();
}

// the parts of a block in list order, the far field and the zero-mean term,
// rounded to float32 once
__global__ __launch_bounds__(256) void k_finalize64(P2P64Args A) {
    const int b = blockIdx.x * 4 + (threadIdx.x >> 6), lane = threadIdx.x & 63;
    if (b >= A.nblocks) return;
    const int4 blk = A.blocks[b];
    if (lane >= blk.y) return;
    const int64_t i = blk.x + lane;
    const double *q = A.near + 6 * (size_t)blk.z + lane;
    double v[6] = {0, 0, 0, 0, 0, 0};
    const int np = A.n_long > 0 ? parts_left(blk.w) : blk.w & PBLOCK_PARTS;
    for (int p = 0; p < np; ++p)
#pragma unroll
        for (int c = 0; c < 6; ++c) v[c] += q[(size_t)(6 * p + c) * blk.y];
    if (A.far_u)
        for (int c = 0; c < 3; ++c) {
            v[c] += A.far_u[c * A.n + i];
            v[3 + c] += A.far_da[c * A.n + i];
        }
    if (A.surface)
        for (int c = 0; c < 3; ++c) v[c] -= A.bounds->sum_xa[c] * A.inv3V;
    if (A.bounds->stale)  // positions differ from the build's
        for (int c = 0; c < 6; ++c) v[c] = __builtin_nan("");
    const int o = A.perm[i];
    A.ux[o] = (float)v[0];
    A.uy[o] = (float)v[1];
    A.uz[o] = (float)v[2];
    A.dax[o] = (float)v[3];
    A.day[o] = (float)v[4];
    A.daz[o] = (float)v[5];
}

static void launch_p2p64(Ctx &c, const P2P64Args &A) {
    c.record(2 * PH_P2P);
    if (A.nitems > 0) {
        const unsigned g = xcd_grid(cdiv(A.nitems, 4));
        if (c.prm.scheme == VFMM_SCHEME_TRANSPOSE)
            k_p2p64<VFMM_SCHEME_TRANSPOSE><<<g, 256, 0, c.stream>>>(A);
        else
            k_p2p64<VFMM_SCHEME_CLASSICAL><<<g, 256, 0, c.stream>>>(A);
        VFMM_LAUNCH_CHECK();
        if (A.n_long > 0) sum_parts<double, double>(c);
        k_finalize64<<<cdiv(A.nblocks, 4), 256, 0, c.stream>>>(A);
        VFMM_LAUNCH_CHECK();
    }
    c.record(2 * PH_P2P + 1);
}

// The launch constant of the scaled form (the cutoff's constants are cutoff_ce).
static P2PConst make_const(double sigma, bool var) {
    P2PConst k{};
    k.inv_kappa = var ? 1.0f : (float)(1.0 / p2p_kappa(sigma));
    return k;
}

// Scale of the records: kappa of the shared core, or the numerator of kappa_j.
static double record_kappa(bool var, float sigma_uniform) { return var ? p2p_kappa(1.0) : p2p_kappa(sigma_uniform); }

// The float32 near-field records of the tree's leaves, one wave per leaf.
static void p2p_records(Ctx &c) {
    if (c.n == 0) return;
    c.recp.ensure(sizeof(float4) * (c.var_sigma ? 4 : 3) * (size_t)c.n);
    const double kap = record_kappa(c.var_sigma, c.sigma_uniform);
    const unsigned grid = cdiv(c.nleaves, 4);
    if (c.var_sigma)
        k_p2p_records<true><<<grid, 256, 0, c.stream>>>(c.leaves.as<int>(), c.nleaves, c.c_start.as<int>(),
                                                        c.c_count.as<int>(), c.c_geo.as<float4>(), kap,
                                                        c.rec.as<float4>(), c.recp.as<float4>());
    else
        k_p2p_records<false><<<grid, 256, 0, c.stream>>>(c.leaves.as<int>(), c.nleaves, c.c_start.as<int>(),
                                                         c.c_count.as<int>(), c.c_geo.as<float4>(), kap,
                                                         c.rec.as<float4>(), c.recp.as<float4>());
    VFMM_LAUNCH_CHECK();
}

void p2p_prepare(Ctx &c) { p2p_records(c); }

// the items of kind (whole waves) and kind + 1 (lane groups)
template <int SCHEME, bool KAHAN>
static void launch_p2p(const P2PConst &k, P2PArgs A, int kind, bool var, hipStream_t s) {
    const int nw = A.item0[kind + 1] - A.item0[kind], ng = A.item0[kind + 2] - A.item0[kind + 1];
    if (nw > 0) {
        A.kind = kind;
        const unsigned g = xcd_grid(cdiv(nw, 4));
        if (var)
            k_p2p<SCHEME, KAHAN, true><<<g, 256, 0, s>>>(k, A);
        else
            k_p2p<SCHEME, KAHAN, false><<<g, 256, 0, s>>>(k, A);
        VFMM_LAUNCH_CHECK();
    }
    if (ng > 0) {
        A.kind = kind + 1;
        const unsigned g = xcd_grid(cdiv(ng, 4));
        if (var)
            k_p2p_group<SCHEME, KAHAN, true><<<g, 256, 0, s>>>(k, A);
        else
            k_p2p_group<SCHEME, KAHAN, false><<<g, 256, 0, s>>>(k, A);
        VFMM_LAUNCH_CHECK();
    }
}

template <bool KAHAN>
static void launch_kinds(int scheme, bool var, const P2PConst &k, const P2PArgs &A, hipStream_t s) {
    for (int kind = 0; kind < 4; kind += 2) {  // particles, then target points
        if (kind == 2 && A.velocity)
            launch_p2p<VELOCITY_ONLY, KAHAN>(k, A, kind, var, s);
        else if (scheme == VFMM_SCHEME_TRANSPOSE)
            launch_p2p<VFMM_SCHEME_TRANSPOSE, KAHAN>(k, A, kind, var, s);
        else
            launch_p2p<VFMM_SCHEME_CLASSICAL, KAHAN>(k, A, kind, var, s);
    }
}

// whether the per-target sums are compensated
static bool compensated(const vfmm_params &prm) { return prm.kahan != 0 || prm.precision == VFMM_PRECISION_MIXED; }

static void dispatch_p2p(const vfmm_params &prm, bool var, const P2PConst &k, const P2PArgs &A, hipStream_t s) {
    if (compensated(prm))
        launch_kinds<true>(prm.scheme, var, k, A, s);
    else
        launch_kinds<false>(prm.scheme, var, k, A, s);
}

static P2PArgs tree_args(Ctx &c) {
    P2PArgs A{};
    A.rec = c.recp.as<float4>();
    A.items = c.items.as<int4>();
    A.item_out = c.item_out.as<int>();
    A.blocks = c.pblocks.as<int4>();
    A.ent = c.p2p_ent.as<int4>();
    A.sh = c.p2p_sh.as<float4>();
    for (int k = 0; k < 5; ++k) A.item0[k] = c.item0[k];
    A.velocity = eval_sources(c) ? 1 : 0;
    A.nblocks = c.n_pblocks;
    A.n = c.n;
    A.perm = c.perm.as<int>();
    A.bounds = c.bres.as<Bounds>();
    A.surface = (c.prm.periodic && c.prm.zero_mean) ? 1 : 0;
    A.inv3V = c.prm.periodic ? (float)(1.0 / (3.0 * c.prm.box_len * c.prm.box_len * c.prm.box_len)) : 0.f;
    return A;
}

// Near field alone, on stream s, into c.near (the partial results of every
// work item); the far field runs before, after or beside it on the library
// stream and finalize_near_far adds a block's parts and the far field.  At
// 128^3 a block's list is eight parts: its 32,768 one-block waves would fill
// every SIMD exactly four times over, and the uneven end of the last round
// costs a few percent; a work-group's waves then also share one block, so fewer
// target neighbourhoods are in flight on each XCD and more source records hit in
// L2.
void p2p_near(Ctx &c, hipStream_t s) {
    const P2PConst k = make_const(c.sigma_uniform, c.var_sigma);
    c.near.ensure(sizeof(float) * 6 * (size_t)std::max(c.n_partial, 1));
    P2PArgs A = tree_args(c);
    A.near = c.near.as<float>();
    c.record(2 * PH_P2P, s);
    dispatch_p2p(c.prm, c.var_sigma, k, A, s);
    c.record(2 * PH_P2P + 1, s);
}

// out[perm[i]] = (sum of the near-field parts)[i] + far[i] (- the zero-mean
// surface term for u); one wave per block, a lane per target, parts added in
// list order with four parts' loads in flight.  R: the sums' type, double where the
// parts' own are compensated (an evaluation of 128^3 with four parts a block takes 15.3
// ms either way, the 100,003 clustered particles with up to 32 5.00 instead of 4.86)
template <class R>
__global__ __launch_bounds__(256) void k_finalize(P2PArgs A, const float *__restrict__ near) {
    const int b = blockIdx.x * 4 + (threadIdx.x >> 6), lane = threadIdx.x & 63;
    if (b >= A.nblocks) return;
    const int4 blk = A.blocks[b];
    if (lane >= blk.y) return;
    const int64_t i = blk.x + lane;
    const int64_t n = A.n;
    const int tc = blk.y, np = parts_left(blk.w);
    const float *q = near + 6 * (size_t)blk.z + lane;
    if (A.velocity && (blk.w & PBLOCK_VELOCITY)) {  // target points: no stretching was computed, none is read
        R v[3] = {A.far_u[i], A.far_u[n + i], A.far_u[2 * n + i]};
        for (int p = 0; p < np; ++p)
#pragma unroll
            for (int c = 0; c < 3; ++c) v[c] += q[(size_t)(6 * p + c) * tc];
        if (A.surface)
            for (int c = 0; c < 3; ++c) v[c] -= (float)(A.bounds->sum_xa[c]) * A.inv3V;
        if (A.bounds->stale) v[0] = v[1] = v[2] = __builtin_nanf("");
        const int o = A.perm[i];
        A.ux[o] = (float)v[0];
        A.uy[o] = (float)v[1];
        A.uz[o] = (float)v[2];
        return;
    }
    R v[6] = {0, 0, 0, 0, 0, 0};
    for (int p0 = 0; p0 < np; p0 += 4) {
        float w[4][6];
#pragma unroll
        for (int p = 0; p < 4; ++p)
#pragma unroll
            for (int c = 0; c < 6; ++c) w[p][c] = p0 + p < np ? q[(size_t)(6 * (p0 + p) + c) * tc] : 0.f;
#pragma unroll
        for (int p = 0; p < 4; ++p)
#pragma unroll
            for (int c = 0; c < 6; ++c) v[c] += w[p][c];
    }
    R u0 = v[0] + A.far_u[i], u1 = v[1] + A.far_u[n + i], u2 = v[2] + A.far_u[2 * n + i];
    R d0 = v[3] + A.far_da[i], d1 = v[4] + A.far_da[n + i], d2 = v[5] + A.far_da[2 * n + i];
    if (A.surface) {
        u0 -= (float)(A.bounds->sum_xa[0]) * A.inv3V;
        u1 -= (float)(A.bounds->sum_xa[1]) * A.inv3V;
        u2 -= (float)(A.bounds->sum_xa[2]) * A.inv3V;
    }
    if (A.bounds->stale) u0 = u1 = u2 = d0 = d1 = d2 = __builtin_nanf("");  // positions differ from the build's
    const int o = A.perm[i];
    A.ux[o] = (float)u0;
    A.uy[o] = (float)u1;
    A.uz[o] = (float)u2;
    A.dax[o] = (float)d0;
    A.day[o] = (float)d1;
    A.daz[o] = (float)d2;
}

template <class R>
static void finalize(Ctx &c, const P2PArgs &A) {
    sum_parts<float, R>(c);
    k_finalize<R><<<cdiv(c.n_pblocks, 4), 256, 0, c.stream>>>(A, c.near.as<float>());
    VFMM_LAUNCH_CHECK();
}

void finalize_near_far(Ctx &c, float *ux, float *uy, float *uz, float *dax, float *day, float *daz) {
    P2PArgs A = tree_args(c);
    A.far_u = c.far_u.as<float>();
    A.far_da = c.far_da.as<float>();
    A.ux = ux; A.uy = uy; A.uz = uz; A.dax = dax; A.day = day; A.daz = daz;
    if (c.n == 0) return;
    if (compensated(c.prm))
        finalize<double>(c, A);
    else
        finalize<float>(c, A);
}

void p2p_and_finalize(Ctx &c, float *ux, float *uy, float *uz, float *dax, float *day, float *daz) {
    if (c.prm.precision == VFMM_PRECISION_FP64) {
        P2P64Args A{};
        A.rec = c.rec64.as<double4>();
        A.items = c.items.as<int4>();
        A.item_out = c.item_out.as<int>();
        A.blocks = c.pblocks.as<int4>();
        A.ent = c.p2p_ent.as<int4>();
        A.nitems = c.item0[4];
        A.nblocks = c.n_pblocks;
        A.n_long = c.n_long;
        A.near = c.near.as<double>();
        A.B = c.img_B;
        A.len = c.prm.periodic ? c.prm.box_len : 0.0;
        A.far_u = c.far_u.as<double>();
        A.far_da = c.far_da.as<double>();
        A.n = c.n;
        A.perm = c.perm.as<int>();
        A.bounds = c.bres.as<Bounds>();
        A.surface = (c.prm.periodic && c.prm.zero_mean) ? 1 : 0;
        A.inv3V = c.prm.periodic ? 1.0 / (3.0 * c.prm.box_len * c.prm.box_len * c.prm.box_len) : 0.0;
        A.ux = ux; A.uy = uy; A.uz = uz; A.dax = dax; A.day = day; A.daz = daz;
        launch_p2p64(c, A);
        return;
    }
    // the same near-field parts and finalize as the other evaluation orders,
    // so that every order gives bitwise the same results
    p2p_near(c, c.stream);
    finalize_near_far(c, ux, uy, uz, dax, day, daz);
}

// ---------------------------------------------------------------------------
// Direct mode: every target against all N sources (full cutoff form), in the
// caller's order, no tree, no far field.
// ---------------------------------------------------------------------------
__global__ __launch_bounds__(256) void k_direct_setup64(int64_t n, const float *x, const float *y, const float *z,
                                                        const float *ax, const float *ay, const float *az,
                                                        const float *s, double4 *rec, int *perm) {
    const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (i >= n) return;
    const double k = 0.079577471545947667884;  // 1/(4 pi)
    const double c = 0.70710678118654752440 / (double)s[i];  // 1/(sqrt 2 sigma)
    rec[2 * i] = make_double4(x[i], y[i], z[i], c * c);
    rec[2 * i + 1] = make_double4((double)ax[i] * k, (double)ay[i] * k, (double)az[i] * k, c * c * c);
    perm[i] = (int)i;
}

// Records relative to one origin, straight from the caller's arrays.
template <bool VAR>
__global__ __launch_bounds__(256) void k_direct_records(int64_t n, const float *x, const float *y, const float *z,
                                                        const float *ax, const float *ay, const float *az,
                                                        const float *s, double ox, double oy, double oz, double kappa,
                                                        float4 *__restrict__ out) {
    const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (i >= n) return;
    const double k = 0.079577471545947667884;  // 1/(4 pi)
    const double kap = VAR ? kappa / (double)s[i] : kappa;
    const double sc = VAR ? 1.0 : kappa;
    put_record<VAR>(out, i, sc * ((double)x[i] - ox), sc * ((double)y[i] - oy), sc * ((double)z[i] - oz), kap,
                    k * ax[i], k * ay[i], k * az[i], ax[i], ay[i], az[i]);
}

// red[0][k] = the sum over the work-group's W waves of red[w][k], in wave order
template <int W, int K, class T>
__device__ __forceinline__ void sum_waves(T *red) {
    __syncthreads();
    for (int k = threadIdx.x; k < K; k += 64 * W) {
        T v = red[k];
        for (int w = 1; w < W; ++w) v += red[w * K + k];
        red[k] = v;
    }
    __syncthreads();
}

// A work-group of eight waves takes 64 targets; each wave sums an eighth of
// the sources, 64 at a time, as scalar operands, and the waves' sums are added
// in LDS in wave order.  One wave per 64 targets left the chip idle: 65,536
// particles are 1,024 waves, one per SIMD, where the pair loop needs several
// (60,000 particles: 10.6 -> 3.1 ms, 1.15e12 pairs/s).
constexpr int DIRECT_WAVES = 8;
template <int SCHEME, bool KAHAN, bool VAR>
__global__ __launch_bounds__(64 * DIRECT_WAVES) void k_direct(P2PConst k, P2PArgs A) {
    __shared__ Acc<KAHAN> red[DIRECT_WAVES][9][64];
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int n = (int)A.n, i = blockIdx.x * 64 + lane;
    Tgt t;
    const float4 r0 = load_target<VAR>(A, min(i, n - 1), t);
    set_offset<SCHEME>(r0, make_float4(0.f, 0.f, 0.f, 0.f), t);
    float S[9] = {0, 0, 0, 0, 0, 0, 0, 0, 0};
    float Cc[9] = {0, 0, 0, 0, 0, 0, 0, 0, 0};
    const int s0 = (int)((int64_t)wave * n / DIRECT_WAVES), s1 = (int)((int64_t)(wave + 1) * n / DIRECT_WAVES);
    for (int s = s0; s < s1; s += 64) {
        Acc9 p = {0, 0, 0, 0, 0, 0, 0, 0, 0};
        leaf_loop<0, SCHEME, VAR>(k, A.rec, s, min(64, s1 - s), t, p);
        add_leaf<SCHEME, KAHAN>(t, p, S, Cc);  // per 64 sources: |y| spans the domain here
    }
#pragma unroll
    for (int q = 0; q < 9; ++q) red[wave][q][lane] = kahan_value<KAHAN>(S[q], Cc[q]);
    sum_waves<DIRECT_WAVES, 9 * 64>(&red[0][0][0]);
    if (wave != 0 || i >= n) return;
#pragma unroll
    for (int q = 0; q < 9; ++q) S[q] = (float)red[0][q][lane];
    finish<SCHEME>(k, A, i, lane, 64, t, S, nullptr);
}

// Fewer particles: a work-group of sixteen waves takes 16 targets, each wave every
// sixteenth pass of 64 sources (four lane groups that hold the 16 targets, the
// sources staged in LDS as in p2p_group), so that 1,500 particles occupy 94
// CUs with 16 waves each instead of 24 waves in all (the whole call 337 -> 35
// us; 5,000 particles 964 -> 69 us, 16,000 2,930 -> 254 us).
constexpr int DIRECT_SMALL_WAVES = 16, DIRECT_SMALL_T = 16;
template <int SCHEME, bool KAHAN, bool VAR>
__global__ __launch_bounds__(64 * DIRECT_SMALL_WAVES) void k_direct_small(P2PConst k, P2PArgs A) {
    constexpr int RS = VAR ? 4 : 3, T = DIRECT_SMALL_T, NG = 64 / T;
    __shared__ float4 stage[DIRECT_SMALL_WAVES][3 * 64];
    __shared__ Acc<KAHAN> red[DIRECT_SMALL_WAVES][9][T];
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int grp = lane / T, tl = lane % T;
    const int n = (int)A.n, i = blockIdx.x * T + tl;
    Tgt t;
    const float4 r0 = load_target<VAR>(A, min(i, n - 1), t);
    set_offset<SCHEME>(r0, make_float4(0.f, 0.f, 0.f, 0.f), t);
    float S[9] = {0, 0, 0, 0, 0, 0, 0, 0, 0};
    float Cc[9] = {0, 0, 0, 0, 0, 0, 0, 0, 0};
    float4 *L = stage[wave];
    for (int f0 = 64 * wave; f0 < n; f0 += 64 * DIRECT_SMALL_WAVES) {
        const int f = f0 + lane;
        const bool ok = f < n;
        const float4 *src = A.rec + RS * (size_t)min(f, n - 1);
        float4 sp = src[0], sa = src[1], sb = src[2];
        if (!ok) {  // the last source again without its strength
            sa = make_float4(0.f, 0.f, 0.f, sa.w);
            sb = make_float4(0.f, 0.f, 0.f, sb.w);
        }
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");  // LDS order within the wave
        L[3 * lane] = sp;
        L[3 * lane + 1] = sa;
        L[3 * lane + 2] = sb;
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        Acc9 p = {0, 0, 0, 0, 0, 0, 0, 0, 0};
        group_loop<0, SCHEME, VAR>(k, L + 3 * grp, NG, (min(64, n - f0) + 2 * NG - 1) / (2 * NG), t, p);
        add_leaf<SCHEME, KAHAN>(t, p, S, Cc);  // per 64 sources: |y| spans the domain here
    }
#pragma unroll
    for (int q = 0; q < 9; ++q) {
        const Acc<KAHAN> own = kahan_value<KAHAN>(S[q], Cc[q]);
        Acc<KAHAN> v = own;
        for (int g = 1; g < NG; ++g) v += __shfl(own, (lane + g * T) & 63, 64);
        if (lane < T) red[wave][q][lane] = v;
    }
    sum_waves<DIRECT_SMALL_WAVES, 9 * T>(&red[0][0][0]);
    if (wave != 0 || lane >= T || i >= n) return;
#pragma unroll
    for (int q = 0; q < 9; ++q) S[q] = (float)red[0][q][lane];
    finish<SCHEME>(k, A, i, lane, T, t, S, nullptr);
}

// Few targets per work-group keep the last round of work-groups even until the
// scalar form's cheaper pair step outweighs it; measured (scalar / groups):
// 17,000 particles 516 / 280 us, 24,000 724 / 532, 32,768 973 / 926, 40,000
// 1,611 / 1,379, 49,152 1,998 / 2,053, 57,344 2,997 / 2,800, 65,536 3,422 / 3,645.
// The rounds make the two cross more than once; the line lies above the last size at
// which the groups win, for 3 % lost around 49,152, where the scalar form's rounds end evenly.
constexpr int64_t DIRECT_SMALL_N = 61440;

template <int SCHEME, bool KAHAN>
static void launch_direct(const P2PConst &k, const P2PArgs &A, bool var, hipStream_t s) {
    const bool small = A.n < DIRECT_SMALL_N;
    const unsigned g = small ? cdiv(A.n, DIRECT_SMALL_T) : cdiv(A.n, 64);
    if (small && var)
        k_direct_small<SCHEME, KAHAN, true><<<g, 64 * DIRECT_SMALL_WAVES, 0, s>>>(k, A);
    else if (small)
        k_direct_small<SCHEME, KAHAN, false><<<g, 64 * DIRECT_SMALL_WAVES, 0, s>>>(k, A);
    else if (var)
        k_direct<SCHEME, KAHAN, true><<<g, 64 * DIRECT_WAVES, 0, s>>>(k, A);
    else
        k_direct<SCHEME, KAHAN, false><<<g, 64 * DIRECT_WAVES, 0, s>>>(k, A);
    VFMM_LAUNCH_CHECK();
}

// Blocks of 64 targets, entries of 64 sources and np items per block for the
// float64 form.
__global__ __launch_bounds__(256) void k_direct_blocks(int64_t n, int nb, int np, int4 *blocks, int4 *ent, int4 *items,
                                                       int *item_out) {
    const int j = blockIdx.x * 256 + threadIdx.x;
    if (j >= nb * np) return;
    const int b = j / np, p = j % np;
    const int cnt = (int)min<int64_t>(64, n - (int64_t)b * 64);
    const int u0 = b * 64 * np;
    if (p == 0) {
        blocks[b] = make_int4(b * 64, cnt, u0, np);
        ent[b] = make_int4(b * 64, cnt, 0, 0);
    }
    const int e0 = (int)((int64_t)p * nb / np), e1 = (int)((int64_t)(p + 1) * nb / np);
    items[j] = make_int4(b * 64, cnt, e0, e1 - e0);
    item_out[j] = u0 + p * cnt;
}

// The float32 (and mixed) all-pairs evaluation; the near-field kernel's
// interval is timed on tc's events when tc is given.
static void direct_f32_impl(const Ctx &c, Ctx *tc, hipStream_t s, int64_t n, const Bounds &hb, float4 *recp,
                            const Bounds *bounds, const float *x, const float *y, const float *z, const float *ax,
                            const float *ay, const float *az, const float *sigma, float *ux, float *uy, float *uz,
                            float *dax, float *day, float *daz) {
    if (n == 0) return;
    // per-source cores when they differ by more than 1e-6 relative (as a build decides)
    const bool var = hb.sig_max > hb.sig_min * (1.0 + 1e-6);
    const float sig = (float)hb.sig_max;
    const double kap = record_kappa(var, sig);
    // one origin for every record: the centre of the bounding box
    const double org[3] = {0.5 * (hb.lo[0] + hb.hi[0]), 0.5 * (hb.lo[1] + hb.hi[1]), 0.5 * (hb.lo[2] + hb.hi[2])};
    if (var)
        k_direct_records<true><<<cdiv(n, 256), 256, 0, s>>>(n, x, y, z, ax, ay, az, sigma, org[0], org[1], org[2], kap,
                                                            recp);
    else
        k_direct_records<false><<<cdiv(n, 256), 256, 0, s>>>(n, x, y, z, ax, ay, az, sigma, org[0], org[1], org[2],
                                                             kap, recp);
    VFMM_LAUNCH_CHECK();
    const P2PConst k = make_const(sig, var);
    P2PArgs A{};
    A.rec = recp;
    A.n = n;
    A.bounds = bounds;
    A.ux = ux; A.uy = uy; A.uz = uz; A.dax = dax; A.day = day; A.daz = daz;
    if (tc) tc->record(2 * PH_P2P, s);
    const bool kah = compensated(c.prm);
    if (c.prm.scheme == VFMM_SCHEME_TRANSPOSE) {
        if (kah) launch_direct<VFMM_SCHEME_TRANSPOSE, true>(k, A, var, s);
        else launch_direct<VFMM_SCHEME_TRANSPOSE, false>(k, A, var, s);
    } else {
        if (kah) launch_direct<VFMM_SCHEME_CLASSICAL, true>(k, A, var, s);
        else launch_direct<VFMM_SCHEME_CLASSICAL, false>(k, A, var, s);
    }
    if (tc) tc->record(2 * PH_P2P + 1, s);
}

void direct_f32(const Ctx &c, hipStream_t s, int64_t n, const Bounds &hb, float4 *recp, const Bounds *bounds,
                const float *x, const float *y, const float *z, const float *ax, const float *ay, const float *az,
                const float *sigma, float *ux, float *uy, float *uz, float *dax, float *day, float *daz) {
    direct_f32_impl(c, nullptr, s, n, hb, recp, bounds, x, y, z, ax, ay, az, sigma, ux, uy, uz, dax, day, daz);
}

void direct_all_pairs(Ctx &c, const float *x, const float *y, const float *z, const float *ax, const float *ay,
                      const float *az, const float *sigma, float *ux, float *uy, float *uz, float *dax, float *day,
                      float *daz) {
    const int64_t n = c.n;
    const int nb = (int)cdiv(n, 64);
    c.n_blocks = nb;
    c.p2p_pairs = n * n;
    if (c.prm.precision == VFMM_PRECISION_FP64) {
        const int np = std::max(1, std::min(nb, 8192 / nb));  // at least about 8,192 waves
        c.perm.ensure(sizeof(int) * n);
        c.pblocks.ensure(sizeof(int4) * nb);
        c.p2p_ent.ensure(sizeof(int4) * nb);
        c.items.ensure(sizeof(int4) * (size_t)nb * np);
        c.item_out.ensure(sizeof(int) * (size_t)nb * np);
        c.near.ensure(sizeof(double) * 6 * 64 * (size_t)nb * np);
        k_direct_blocks<<<cdiv((size_t)nb * np, 256), 256, 0, c.stream>>>(n, nb, np, c.pblocks.as<int4>(),
                                                                          c.p2p_ent.as<int4>(), c.items.as<int4>(),
                                                                          c.item_out.as<int>());
        VFMM_LAUNCH_CHECK();
        c.rec64.ensure(sizeof(double4) * 2 * n);
        k_direct_setup64<<<cdiv(n, 256), 256, 0, c.stream>>>(n, x, y, z, ax, ay, az, sigma, c.rec64.as<double4>(),
                                                              c.perm.as<int>());
        VFMM_LAUNCH_CHECK();
        P2P64Args A{};
        A.rec = c.rec64.as<double4>();
        A.items = c.items.as<int4>();
        A.item_out = c.item_out.as<int>();
        A.blocks = c.pblocks.as<int4>();
        A.ent = c.p2p_ent.as<int4>();
        A.nitems = nb * np;
        A.nblocks = nb;
        A.near = c.near.as<double>();
        A.n = n;
        A.perm = c.perm.as<int>();
        A.bounds = c.bres.as<Bounds>();
        A.ux = ux; A.uy = uy; A.uz = uz; A.dax = dax; A.day = day; A.daz = daz;
        launch_p2p64(c, A);
        return;
    }
    c.recp.ensure(sizeof(float4) * (c.var_sigma ? 4 : 3) * (size_t)n);
    direct_f32_impl(c, &c, c.stream, n, c.hb, c.recp.as<float4>(), c.bres.as<Bounds>(), x, y, z, ax, ay, az, sigma,
                    ux, uy, uz, dax, day, daz);
}

}  // namespace vfmm
