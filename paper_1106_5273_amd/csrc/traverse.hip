// Dual tree traversal (Sec. 3.3, Algorithms 1 and 2) and interaction-list
// construction ("GPU buffering", Sec. 4.4).
//
// The paper's stack of cell pairs becomes a frontier processed one
// generation at a time: each pair splits its cell of larger radius (the other
// one when that cell is a leaf) and every child pair is classified
//   M2L  if (R_A + R_B) < theta D  and  D - R_A - R_B >= sigma_gap sigma_max,
//   P2P  else if both cells are leaves,
//   push else (next generation).
// Counts, an exclusive scan and a write pass keep the output order fixed, so
// the lists (and every sum built from them) are bit-reproducible.  Periodic
// images enter as an image code on each pair: the source cell is shifted by
// n * box_len.
#include "ctx.h"
#include "cutoff_fits.h"

namespace vfmm {

static constexpr int TPB = 256;

void sort_pairs_u64(Ctx &c, DevBuf &kA, DevBuf &vA, DevBuf &kB, DevBuf &vB, int64_t n, int nbits);

struct TravArgs {
    const int *child, *nchild;
    const float4 *geo;
    const float *rad;
    float theta, gap;  // gap = sigma_gap * sigma_max
    const float4 *hi;  // per-source cores: cell boxes whose .w is the cell's largest core (else null)
    float sgap;        // sigma_gap (with hi)
    float len;         // periodic cube side (0 in free space)
    int B;             // image range |n|_inf <= B
};

__device__ inline void img_shift(int code, int B, float len, float &sx, float &sy, float &sz) {
    const int W = 2 * B + 1;
    const int ix = code % W - B;
    const int iy = (code / W) % W - B;
    const int iz = code / (W * W) - B;
    sx = ix * len;
    sy = iy * len;
    sz = iz * len;
}

// Decisions on distances and radii use a relative margin TIE_TOL: quantities
// that agree to within float32 rounding of the cell coordinates (exact ties
// are common in regular particle layouts) are decided the same way for every
// cell pair, so pairs related by a translation of the tree get equal lists.
static constexpr float TIE_TOL = 1.0f / 65536.0f;

// 0 = M2L, 1 = P2P, 2 = push
__device__ inline int interact(const TravArgs &A, int a, int b, int img) {
    float sx, sy, sz;
    img_shift(img, A.B, A.len, sx, sy, sz);
    const float4 ga = A.geo[a], gb = A.geo[b];
    const float ra = A.rad[a], rb = A.rad[b];
    const int na = A.nchild[a], nb = A.nchild[b];
    const float dx = ga.x - gb.x - sx, dy = ga.y - gb.y - sy, dz = ga.z - gb.z - sz;
    const float D = sqrtf(dx * dx + dy * dy + dz * dz);
    // the MAC and the core gap, both failing on (near-)ties; with per-source
    // cores the gap is measured in the largest core of the source cell b
    const float gap = A.hi ? A.sgap * A.hi[b].w : A.gap;
    const bool far = ra + rb < A.theta * D * (1.0f - TIE_TOL) && D - ra - rb >= gap + TIE_TOL * D;
    return far ? 0 : na == 0 && nb == 0 ? 1 : 2;
}

// Children pairs of a frontier pair (Algorithm 1): split A when its radius is
// larger (radii equal to within TIE_TOL split B), unless the chosen cell is a
// leaf.
__device__ inline void split_pair(const TravArgs &A, int a, int b, bool &splitA, int &first, int &cnt) {
    const float ra = A.rad[a], rb = A.rad[b];
    const bool la = A.nchild[a] == 0, lb = A.nchild[b] == 0;
    splitA = (ra > rb * (1.0f + TIE_TOL) && !la) || lb;
    const int s = splitA ? a : b;
    first = A.child[s];
    cnt = A.nchild[s];
}

// Eight lanes per frontier pair, one per child pair: lane o's cells and decision
// (3: no such child pair), and its lanes' ballots.  With a thread per frontier
// pair the child pairs' loads followed one another and their entries were
// written 16 bytes at a time, 128 bytes apart.
struct ChildPair {
    int a, b, img, kind;
    int sh;                 // first lane of the frontier pair
    unsigned below;         // mask of the lanes before this one among the eight
    unsigned bal[3];        // per kind: which of the eight lanes
};

__device__ inline ChildPair child_pair(const TravArgs &A, const int4 *fr, int nf, int split, int i, int o) {
    ChildPair c;
    c.kind = 3;
    c.a = c.b = c.img = 0;
    if (i < nf) {
        const int4 pr = fr[i];
        c.a = pr.x;
        c.b = pr.y;
        c.img = pr.z;
        int n = 1;
        if (split) {
            bool sa;
            int first;
            split_pair(A, pr.x, pr.y, sa, first, n);
            if (sa) c.a = first + o;
            else c.b = first + o;
        }
        if (o < n) c.kind = interact(A, c.a, c.b, c.img);
    }
    c.sh = (threadIdx.x & 63) & ~7;
    c.below = (1u << o) - 1u;
#pragma unroll
    for (int k = 0; k < 3; ++k) c.bal[k] = (unsigned)(__ballot(c.kind == k) >> c.sh) & 0xffu;
    return c;
}

__global__ __launch_bounds__(TPB) void k_trav_count(TravArgs A, const int4 *fr, int nf, int split, int *cnt) {
    const unsigned g = blockIdx.x * TPB + threadIdx.x;  // below 2^31 + 2^8: frontiers hold at most 2^28 pairs
    const int i = (int)(g >> 3), o = (int)(g & 7u);
    const ChildPair c = child_pair(A, fr, nf, split, i, o);
    if (i < nf && o < 3) cnt[o * nf + i] = __popc(o == 0 ? c.bal[0] : o == 1 ? c.bal[1] : c.bal[2]);
}

__global__ void k_trav_totals(const int *cnt, const int *off, int nf, int *tot) {
    for (int k = 0; k < 3; ++k) tot[k] = off[(k + 1) * nf - 1] + cnt[(k + 1) * nf - 1] - off[k * nf];
}

__global__ __launch_bounds__(TPB) void k_trav_write(TravArgs A, const int4 *fr, int nf, int split, const int *off,
                                                    int4 *m2l, int m2l_base, int4 *p2p, int p2p_base, int4 *next) {
    const unsigned g = blockIdx.x * TPB + threadIdx.x;  // below 2^31 + 2^8: frontiers hold at most 2^28 pairs
    const int i = (int)(g >> 3), o = (int)(g & 7u);
    const ChildPair c = child_pair(A, fr, nf, split, i, o);
    if (c.kind == 3) return;
    const int4 e = make_int4(c.a, c.b, c.img, 0);
    if (c.kind == 0)
        m2l[m2l_base + off[i] - off[0] + __popc(c.bal[0] & c.below)] = e;
    else if (c.kind == 1)
        p2p[p2p_base + off[nf + i] - off[nf] + __popc(c.bal[1] & c.below)] = e;
    else
        next[off[2 * nf + i] - off[2 * nf] + __popc(c.bal[2] & c.below)] = e;
}

// The first generations in one work-group, while the frontier holds at most
// TRAV_GROUP pairs: a generation is otherwise a count, one or two scan launches,
// the totals, a wait and a write, 35 us however few its pairs are.  1,024 pairs at
// a time, a thread each; the entries' order is the same.
static constexpr int TRAV_GROUP = 4096;

struct TravGroupArgs {
    int4 *fr[2];  // frontiers, of 8 TRAV_GROUP pairs
    int4 *m2l, *p2p;
    int m2l_cap, p2p_cap;
    int nroot, ncode;
    int *host;  // pinned: pairs left, their frontier, M2L and P2P entries, whether the pairs are to be split
};

__global__ __launch_bounds__(1024) void k_trav_group(TravArgs A, TravGroupArgs G) {
    __shared__ unsigned long long wsum[16];
    const int t = threadIdx.x, lane = t & 63, w = t >> 6;
    int nf = G.nroot * G.ncode, cur = 0, split = 0, nm = 0, np = 0;
    for (int i = t; i < nf; i += 1024) G.fr[0][i] = make_int4(i / G.ncode, i / G.ncode, i % G.ncode, 0);
    __syncthreads();
    while (nf > 0 && nf <= TRAV_GROUP) {
        const int4 *fr = G.fr[cur];
        int4 *nx = G.fr[cur ^ 1];
        int gm = nm, gp = np, gn = 0;
        bool fits = true;
        for (int base = 0; base < nf; base += 1024) {
            const int i = base + t;
            int4 pr = make_int4(0, 0, 0, 0);
            int first = 0, n = 0;
            bool sa = false;
            if (i < nf) {
                pr = fr[i];
                n = 1;
                if (split) split_pair(A, pr.x, pr.y, sa, first, n);
            }
            auto cell_a = [&](int k) { return split && sa ? first + k : pr.x; };
            auto cell_b = [&](int k) { return split && !sa ? first + k : pr.y; };
            unsigned kinds = 0xffffu;  // two bits per child pair, 3: none
            if (i < nf) {
                kinds = 0;
#pragma unroll
                for (int k = 0; k < 8; ++k) {  // all loads in flight together
                    const int kk = min(k, n - 1);
                    const int v = interact(A, cell_a(kk), cell_b(kk), pr.z);
                    kinds |= (unsigned)(k < n ? v : 3) << (2 * k);
                }
            }
            // counts of the three kinds in 21-bit fields
            unsigned long long mine = 0;
#pragma unroll
            for (int k = 0; k < 8; ++k) {
                const unsigned v = (kinds >> (2 * k)) & 3u;
                if (v < 3u) mine += 1ull << (21 * v);
            }
            unsigned long long incl = mine;
#pragma unroll
            for (int o = 1; o < 64; o <<= 1) {
                const unsigned long long u = __shfl_up(incl, o, 64);
                if (lane >= o) incl += u;
            }
            if (lane == 63) wsum[w] = incl;
            __syncthreads();
            unsigned long long pre = incl - mine, tot = 0;
#pragma unroll
            for (int j = 0; j < 16; ++j) {
                const unsigned long long v = wsum[j];
                pre += j < w ? v : 0;
                tot += v;
            }
            __syncthreads();
            const int f21 = (1 << 21) - 1;
            const int tm = (int)(tot & f21), tp = (int)((tot >> 21) & f21), tn = (int)(tot >> 42);
            if (gm + tm > G.m2l_cap || gp + tp > G.p2p_cap) {  // the caller grows the lists and repeats the generation
                fits = false;
                break;
            }
            int om = gm + (int)(pre & f21), op = gp + (int)((pre >> 21) & f21), on = gn + (int)(pre >> 42);
#pragma unroll
            for (int k = 0; k < 8; ++k) {
                const unsigned v = (kinds >> (2 * k)) & 3u;
                if (v == 3u) continue;
                const int4 e = make_int4(cell_a(k), cell_b(k), pr.z, 0);
                if (v == 0u) G.m2l[om++] = e;
                else if (v == 1u) G.p2p[op++] = e;
                else nx[on++] = e;
            }
            gm += tm;
            gp += tp;
            gn += tn;
        }
        if (!fits) break;
        __syncthreads();  // the new frontier is read by other threads
        nm = gm;
        np = gp;
        nf = gn;
        cur ^= 1;
        split = 1;
    }
    if (t == 0) {
        G.host[0] = nf;
        G.host[1] = cur;
        G.host[2] = nm;
        G.host[3] = np;
        G.host[4] = split;
    }
}

// one (root, root, image) pair per problem and image code
__global__ __launch_bounds__(TPB) void k_trav_init(int4 *fr, int nroot, int ncode) {
    const int i = blockIdx.x * TPB + threadIdx.x;
    if (i < nroot * ncode) fr[i] = make_int4(i / ncode, i / ncode, i % ncode, 0);
}

// ---------------------------------------------------------------------------
// CSR by target cell.  Entries are stably sorted by target, so within a
// target they keep the traversal's (deterministic) order.
// ---------------------------------------------------------------------------
__global__ __launch_bounds__(TPB) void k_list_keys(const int4 *raw, int64_t n, uint64_t *key, uint32_t *val) {
    const int64_t i = (int64_t)blockIdx.x * TPB + threadIdx.x;
    if (i >= n) return;
    key[i] = (uint64_t)(uint32_t)raw[i].x;
    val[i] = (uint32_t)i;
}

// CSR offsets from the sorted targets: off[t] = first position with target >= t
// (t = 0 .. nc), by a binary search per target: a thread per target, so a long
// run of cells without entries (the internal cells) costs no serial loop.
__global__ __launch_bounds__(TPB) void k_csr_bounds(const uint64_t *key, int64_t n, int nc, int *off) {
    const int t = blockIdx.x * TPB + threadIdx.x;
    if (t > nc) return;
    int64_t lo = 0, hi = n;
    while (lo < hi) {
        const int64_t mid = (lo + hi) >> 1;
        if ((int64_t)key[mid] < t) lo = mid + 1;
        else hi = mid;
    }
    off[t] = (int)lo;
}

__global__ __launch_bounds__(TPB) void k_m2l_gather(const int4 *raw, const uint32_t *order, int64_t n, int2 *out,
                                                    int *tgt) {
    const int64_t i = (int64_t)blockIdx.x * TPB + threadIdx.x;
    if (i >= n) return;
    const int4 e = raw[order[i]];
    out[i] = make_int2(e.y, e.z);
    tgt[i] = e.x;
}

struct P2PEntryArgs {
    const int *start, *count;
    const float4 *lo, *hi;
    const float4 *geo;        // cell centres
    float len;
    int B;
    float r2_small, r2_sing;  // thresholds on squared distance for the cutoff branches
    int per_cell;             // per-source cores: thresholds from the source leaf's largest core (hi.w)
    double kappa;             // length scale of the float32 near field
    double len64;             // period (0: free space)
    const int *nsrc;          // partitioned builds: sources in front of each leaf's targets (else null)
    float4 *sh;               // out: kappa (c_t - c_s - image shift) per entry (null: not needed)
};

// entry = (source start, source count, image code, variant) with variant
// 0 = full cutoff (some pair may have s < 1), 1 = s >= 1 for every pair,
// 2 = cutoff equal to 1 in float32 for every pair (singular kernel).  The
// float32 near field also gets the scaled offset between the leaf centres.
__global__ __launch_bounds__(TPB) void k_p2p_gather(P2PEntryArgs A, const int4 *raw, const uint32_t *order,
                                                    int64_t n, int4 *out, unsigned long long *part) {
    const int64_t i = (int64_t)blockIdx.x * TPB + threadIdx.x;
    unsigned long long np = 0, nsrc = 0;
    if (i < n) {
        const int4 e = raw[order[i]];
        const int t = e.x, s = e.y;
        float sx, sy, sz;
        const int W = 2 * A.B + 1;
        sx = (e.z % W - A.B) * A.len;
        sy = ((e.z / W) % W - A.B) * A.len;
        sz = (e.z / (W * W) - A.B) * A.len;
        const float4 tl = A.lo[t], th = A.hi[t], sl = A.lo[s], sh = A.hi[s];
        const float gx = fmaxf(0.f, fmaxf(sl.x + sx - th.x, tl.x - sh.x - sx));
        const float gy = fmaxf(0.f, fmaxf(sl.y + sy - th.y, tl.y - sh.y - sy));
        const float gz = fmaxf(0.f, fmaxf(sl.z + sz - th.z, tl.z - sh.z - sz));
        const float d2 = gx * gx + gy * gy + gz * gz;
        float r2s = A.r2_small, r2g = A.r2_sing;
        if (A.per_cell) {  // every pair's source core is at most the source leaf's largest
            const float s2 = 2.0f * sh.w * sh.w;
            r2s = s2 * VFMM_CUTOFF_XSPLIT * 1.0001f;
            r2g = s2 * 26.0f;
        }
        const int variant = d2 >= r2g ? 2 : (d2 >= r2s ? 1 : 0);
        const int sc = A.nsrc ? A.nsrc[s] : A.count[s];  // only sources enter the near field
        out[i] = make_int4(A.start[s], sc, e.z, variant);
        if (A.sh) {
            const float4 ct = A.geo[t], cs = A.geo[s];
            const double L = A.len64;
            const double Dx = ((double)ct.x - (double)cs.x - (double)(e.z % W - A.B) * L) * A.kappa;
            const double Dy = ((double)ct.y - (double)cs.y - (double)((e.z / W) % W - A.B) * L) * A.kappa;
            const double Dz = ((double)ct.z - (double)cs.z - (double)(e.z / (W * W) - A.B) * L) * A.kappa;
            A.sh[i] = make_float4((float)Dx, (float)Dy, (float)Dz, 0.f);
        }
        np = (unsigned long long)A.count[t] * (unsigned long long)sc;
        nsrc = (unsigned long long)sc;
    }
    // pairs and sources of this work-group's entries, summed by k_sum_u64x2 (no contended atomics)
    __shared__ unsigned long long red[2][TPB / 64];
    unsigned long long ns = nsrc;
    for (int o = 32; o > 0; o >>= 1) {
        np += __shfl_xor(np, o, 64);
        ns += __shfl_xor(ns, o, 64);
    }
    if ((threadIdx.x & 63) == 0) {
        red[0][threadIdx.x >> 6] = np;
        red[1][threadIdx.x >> 6] = ns;
    }
    __syncthreads();
    if (threadIdx.x < 2) {
        unsigned long long t = 0;
        for (int w = 0; w < TPB / 64; ++w) t += red[threadIdx.x][w];
        part[2 * (size_t)blockIdx.x + threadIdx.x] = t;
    }
}

// totals of n pairs of unsigned 64-bit partial counts (one work-group)
__global__ __launch_bounds__(TPB) void k_sum_u64x2(const unsigned long long *part, int n, unsigned long long *out) {
    __shared__ unsigned long long red[2][TPB / 64];
    unsigned long long v0 = 0, v1 = 0;
    for (int i = threadIdx.x; i < n; i += TPB) {
        v0 += part[2 * (size_t)i];
        v1 += part[2 * (size_t)i + 1];
    }
    for (int o = 32; o > 0; o >>= 1) {
        v0 += __shfl_xor(v0, o, 64);
        v1 += __shfl_xor(v1, o, 64);
    }
    if ((threadIdx.x & 63) == 0) {
        red[0][threadIdx.x >> 6] = v0;
        red[1][threadIdx.x >> 6] = v1;
    }
    __syncthreads();
    if (threadIdx.x < 2) {
        unsigned long long t = 0;
        for (int w = 0; w < TPB / 64; ++w) t += red[threadIdx.x][w];
        out[threadIdx.x] = t;
    }
}

// per leaf: its blocks of 64 (Gaussian sums), its near-field blocks, the parts
// by kind (whole waves, lane groups, the same for target points), the float[6]
// outputs of the parts, and the blocks of many parts
constexpr int LEAF_SUMS = 8;

// partials: the work-group's targets times parts, in 64 bits.  The 32-bit sums
// may wrap; they are used only once the total of these is within its limit.
__global__ __launch_bounds__(TPB) void k_leaf_counts(const int *leaves, int nl, const int *count, const int *nsrc,
                                                     const int *loff, const unsigned long long *tot, int64_t nent,
                                                     float stretch, int *out, unsigned long long *partials) {
    const int i = blockIdx.x * TPB + threadIdx.x;
    unsigned long long np64 = 0;
    if (i < nl) {
        const LeafWork W = leaf_work(tot[0], tot[1], nent, stretch);
        const int cell = leaves[i];
        const int cnt = count[cell], lc = loff[cell + 1] - loff[cell];
        unsigned s[LEAF_SUMS] = {(cnt + 63u) / 64u, 0, 0, 0, 0, 0, 0, 0};
        leaf_blocks(cnt, nsrc ? nsrc[cell] : cnt, [&](int, int tc, bool pts) {
            const int np = list_parts(W, tc, lc), kind = (pts ? 2 : 0) + (tc > 32 ? 0 : 1);
            ++s[1];
#pragma unroll
            for (int k = 0; k < 4; ++k) s[2 + k] += k == kind ? np : 0;
            np64 += (unsigned long long)np * (unsigned)tc;
            s[7] += np > LONG_PARTS;
        });
        s[6] = (unsigned)np64;
#pragma unroll
        for (int k = 0; k < LEAF_SUMS; ++k) out[(size_t)k * nl + i] = (int)s[k];
    }
    __shared__ unsigned long long red[TPB / 64];
    for (int o = 32; o > 0; o >>= 1) np64 += __shfl_xor(np64, o, 64);
    if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = np64;
    __syncthreads();
    if (threadIdx.x == 0) {
        for (int w = 1; w < TPB / 64; ++w) np64 += red[w];
        partials[blockIdx.x] = np64;
    }
}

// the totals, the pair count and the targets times parts (np work-groups'), straight to pinned host memory
__global__ __launch_bounds__(TPB) void k_leaf_totals(const int *cnt, const int *off, int nl, const int *tot,
                                                     const unsigned long long *partials, int np, int *out) {
    __shared__ unsigned long long red[TPB / 64];
    unsigned long long v = 0;
    for (int i = threadIdx.x; i < np; i += TPB) v += partials[i];
    for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
    if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = v;
    __syncthreads();
    const int k = threadIdx.x;
    if (k < LEAF_SUMS)
        out[k] = off[(size_t)(k + 1) * nl - 1] + cnt[(size_t)(k + 1) * nl - 1] - off[(size_t)k * nl];
    if (k < 2) out[LEAF_SUMS + k] = tot[k];
    if (k == 0) {
        for (int w = 1; w < TPB / 64; ++w) v += red[w];
        out[LEAF_SUMS + 2] = (int)(unsigned)v;
        out[LEAF_SUMS + 3] = (int)(unsigned)(v >> 32);
    }
}

struct ItemKinds {
    int first[4];
};

// blocks of 64 (target start, targets, first entry, entries); near-field blocks
// (target start, targets, first output, parts and kind) and one work item per
// part (target start, targets, first entry, entries) with its first output, the
// items of kind k from K.first[k] on
__global__ __launch_bounds__(TPB) void k_leaf_items(const int *leaves, int nl, const int *start, const int *count,
                                                    const int *nsrc, const int *loff, const unsigned long long *tot,
                                                    int64_t nent, float stretch, const int *off, ItemKinds K,
                                                    int4 *blocks,
                                                    int4 *pblocks, int *pblong, int4 *items, int *item_out) {
    // one wave per leaf: a leaf may have hundreds of parts
    const int i = blockIdx.x * (TPB / 64) + (threadIdx.x >> 6), lane = threadIdx.x & 63;
    if (i >= nl) return;
    const LeafWork W = leaf_work(tot[0], tot[1], nent, stretch);
    const int cell = leaves[i];
    const int s = start[cell], cnt = count[cell];
    const int l0 = loff[cell], lc = loff[cell + 1] - l0;
    for (int k = 64 * lane, b = off[i] + lane; k < cnt; k += 64 * 64, b += 64)
        blocks[b] = make_int4(s + k, min(64, cnt - k), l0, lc);
    auto before = [&](int k) {  // sum k of the leaves before this one
        const int *o = off + (size_t)k * nl;
        return o[i] - o[0];
    };
    int pb = before(1), u = before(6), ib = before(7);
    int it[4];
#pragma unroll
    for (int k = 0; k < 4; ++k) it[k] = K.first[k] + before(2 + k);
    leaf_blocks(cnt, nsrc ? nsrc[cell] : cnt, [&](int t0, int tc, bool pts) {
        const int np = list_parts(W, tc, lc), kind = (pts ? 2 : 0) + (tc > 32 ? 0 : 1);
        int i0 = it[0];
#pragma unroll
        for (int k = 1; k < 4; ++k) i0 = k == kind ? it[k] : i0;
        if (lane == 0) {
            pblocks[pb] = make_int4(s + t0, tc, u, np | (pts ? PBLOCK_VELOCITY : 0));
            if (np > LONG_PARTS) pblong[ib] = pb;
        }
        ib += np > LONG_PARTS;
        for (int p = lane; p < np; p += 64) {
            const int e0 = (int)((int64_t)p * lc / np), e1 = (int)((int64_t)(p + 1) * lc / np);
            items[i0 + p] = make_int4(s + t0, tc, l0 + e0, e1 - e0);
            item_out[i0 + p] = u + p * tc;
        }
#pragma unroll
        for (int k = 0; k < 4; ++k) it[k] += k == kind ? np : 0;
        ++pb;
        u += np * tc;
    });
}

static int bits_for(int64_t v) {
    int b = 1;
    while ((1LL << b) < v) ++b;
    return b;
}

static void grow_keep4(Ctx &c, DevBuf &b, size_t bytes, size_t used) {
    if (bytes <= b.cap) return;
    DevBuf nb;
    nb.ensure(bytes * 3 / 2);
    if (used) VFMM_HIP(hipMemcpyAsync(nb.ptr, b.ptr, used, hipMemcpyDeviceToDevice, c.stream));
    VFMM_HIP(hipStreamSynchronize(c.stream));
    b.release();
    b = nb;
}

void csr_bounds(Ctx &c, const uint64_t *key, int64_t n, int nc, int *off) {
    k_csr_bounds<<<cdiv(nc + 1, TPB), TPB, 0, c.stream>>>(key, n, nc, off);
    VFMM_LAUNCH_CHECK();
}

// Builds CSR offsets (ncells+1) for a raw (tgt, src, img) list and the
// stable order that sorts it by target.
void csr_by_target(Ctx &c, const int4 *raw, int64_t n, DevBuf &off) {
    hipStream_t s = c.stream;
    const int nc = c.ncells;
    off.ensure(sizeof(int) * ((size_t)nc + 1));
    if (n == 0) {
        VFMM_HIP(hipMemsetAsync(off.ptr, 0, sizeof(int) * ((size_t)nc + 1), s));
        return;
    }
    c.lkey.ensure(sizeof(uint64_t) * n);
    c.lval.ensure(sizeof(uint32_t) * n);
    k_list_keys<<<cdiv(n, TPB), TPB, 0, s>>>(raw, n, c.lkey.as<uint64_t>(), c.lval.as<uint32_t>());
    VFMM_LAUNCH_CHECK();
    sort_pairs_u64(c, c.lkey, c.lval, c.lkey2, c.lval2, n, bits_for(nc));
    csr_bounds(c, c.lkey.as<uint64_t>(), n, nc, off.as<int>());
}

// M2L list in CSR order by target cell (stable: traversal order within a
// target), for the per-pair M2L kernel and for vfmm_copy_lists.
void build_m2l_csr(Ctx &c) {
    hipStream_t s = c.stream;
    const int64_t n_m2l = c.n_m2l;
    csr_by_target(c, c.m2l_raw.as<int4>(), n_m2l, c.m2l_off);
    c.m2l_src.ensure(sizeof(int2) * (size_t)std::max<int64_t>(n_m2l, 1));
    c.m2l_tgt.ensure(sizeof(int) * (size_t)std::max<int64_t>(n_m2l, 1));
    if (n_m2l > 0) {
        k_m2l_gather<<<cdiv(n_m2l, TPB), TPB, 0, s>>>(c.m2l_raw.as<int4>(), c.lval.as<uint32_t>(), n_m2l,
                                                       c.m2l_src.as<int2>(), c.m2l_tgt.as<int>());
        VFMM_LAUNCH_CHECK();
    }
    c.m2l_csr = true;
}

void traverse_and_lists(Ctx &c) {
    hipStream_t s = c.stream;
    TravArgs A{};
    A.child = c.c_child.as<int>();
    A.nchild = c.c_nchild.as<int>();
    A.geo = c.c_geo.as<float4>();
    A.rad = c.c_rad.as<float>();
    A.theta = c.prm.theta;
    A.gap = (float)(c.prm.sigma_gap * c.hb.sig_max);
    if (c.var_sigma) {  // the core gap of each source cell's own largest core
        A.hi = c.c_hi.as<float4>();
        A.sgap = c.prm.sigma_gap;
    }
    A.len = c.prm.periodic ? (float)c.prm.box_len : 0.f;
    A.B = c.img_B;
    const int ncode = c.img_codes;
    c.images_traversed = ncode;

    int nf = ncode * c.nprob, split = 0;
    int64_t n_m2l = 0, n_p2p = 0;
    c.m2l_raw.ensure(sizeof(int4) * (1 << 16));
    c.p2p_raw.ensure(sizeof(int4) * (1 << 16));
    if (nf <= TRAV_GROUP) {
        c.frA.ensure(sizeof(int4) * 8 * TRAV_GROUP);
        c.frB.ensure(sizeof(int4) * 8 * TRAV_GROUP);
        TravGroupArgs G{};
        G.fr[0] = c.frA.as<int4>();
        G.fr[1] = c.frB.as<int4>();
        G.m2l = c.m2l_raw.as<int4>();
        G.p2p = c.p2p_raw.as<int4>();
        G.m2l_cap = (int)std::min<size_t>(c.m2l_raw.cap / sizeof(int4), INT32_MAX / 2);
        G.p2p_cap = (int)std::min<size_t>(c.p2p_raw.cap / sizeof(int4), INT32_MAX / 2);
        G.nroot = c.nprob;
        G.ncode = ncode;
        G.host = pinned_ints(c);
        k_trav_group<<<1, 1024, 0, s>>>(A, G);
        VFMM_LAUNCH_CHECK();
        int h[5];
        sync_ints(c, 5, h);
        nf = h[0];
        if (h[1]) std::swap(c.frA, c.frB);
        n_m2l = h[2];
        n_p2p = h[3];
        split = h[4];
    } else {
        c.frA.ensure(sizeof(int4) * (size_t)nf);
        k_trav_init<<<cdiv(nf, TPB), TPB, 0, s>>>(c.frA.as<int4>(), c.nprob, ncode);
        VFMM_LAUNCH_CHECK();
    }
    int h_tot[4];
    while (nf > 0) {
        c.tcnt.ensure(sizeof(int) * 6 * (size_t)nf + 64);
        int *cnt = c.tcnt.as<int>();
        int *off = cnt + 3 * (size_t)nf;
        k_trav_count<<<cdiv(8 * (int64_t)nf, TPB), TPB, 0, s>>>(A, c.frA.as<int4>(), nf, split, cnt);
        VFMM_LAUNCH_CHECK();
        scan_excl_i32(c, cnt, off, 3LL * nf);
        k_trav_totals<<<1, 1, 0, s>>>(cnt, off, nf, pinned_ints(c));  // straight to pinned host memory
        VFMM_LAUNCH_CHECK();
        sync_ints(c, 3, h_tot);
        const int tm = h_tot[0], tp = h_tot[1], tn = h_tot[2];
        // list positions and frontier counts are 32-bit on the device: refuse before the
        // write pass rather than let an offset wrap (a pair emits at most 8 of each, so
        // a frontier below 2^28 keeps this generation's own totals exact)
        if (tm < 0 || tp < 0 || tn < 0 || n_m2l + tm > INT32_MAX || n_p2p + tp > INT32_MAX || tn > (1 << 28))
            throw Error{VFMM_ENOMEM, "interaction lists exceed 2^31 entries"};
        grow_keep4(c, c.m2l_raw, sizeof(int4) * (size_t)(n_m2l + tm), sizeof(int4) * (size_t)n_m2l);
        grow_keep4(c, c.p2p_raw, sizeof(int4) * (size_t)(n_p2p + tp), sizeof(int4) * (size_t)n_p2p);
        c.frB.ensure(sizeof(int4) * (size_t)std::max(tn, 1));
        k_trav_write<<<cdiv(8 * (int64_t)nf, TPB), TPB, 0, s>>>(A, c.frA.as<int4>(), nf, split, off, c.m2l_raw.as<int4>(),
                                                    (int)n_m2l, c.p2p_raw.as<int4>(), (int)n_p2p,
                                                    c.frB.as<int4>());
        VFMM_LAUNCH_CHECK();
        n_m2l += tm;
        n_p2p += tp;
        std::swap(c.frA, c.frB);
        nf = tn;
        split = 1;
    }
    c.n_m2l = n_m2l;
    c.n_p2p = (int)n_p2p;

    // ---- M2L CSR: only for the per-pair M2L (the batched plan reads the raw list) ----
    c.m2l_csr = false;
    if (!m2l_batched(c.prm)) build_m2l_csr(c);
    // ---- P2P CSR ----
    csr_by_target(c, c.p2p_raw.as<int4>(), n_p2p, c.p2p_off);
    c.p2p_ent.ensure(sizeof(int4) * (size_t)std::max<int64_t>(n_p2p, 1));
    const bool f32 = c.prm.precision != VFMM_PRECISION_FP64;
    if (f32) c.p2p_sh.ensure(sizeof(float4) * (size_t)std::max<int64_t>(n_p2p, 1));
    c.pairs64.ensure(64);
    VFMM_HIP(hipMemsetAsync(c.pairs64.ptr, 0, 16, s));
    if (n_p2p > 0) {
        P2PEntryArgs E{};
        E.start = c.c_start.as<int>();
        E.count = c.c_count.as<int>();
        E.lo = c.c_lo.as<float4>();
        E.hi = c.c_hi.as<float4>();
        E.len = A.len;
        E.B = c.img_B;
        const float s2 = 2.0f * (float)(c.hb.sig_max * c.hb.sig_max);
        E.r2_small = s2 * VFMM_CUTOFF_XSPLIT * 1.0001f;
        E.r2_sing = s2 * 26.0f;
        E.per_cell = c.var_sigma ? 1 : 0;
        E.geo = c.c_geo.as<float4>();
        E.kappa = c.var_sigma ? 1.0 : p2p_kappa(c.sigma_uniform);  // per-source cores: unscaled offsets
        E.len64 = c.prm.periodic ? c.prm.box_len : 0.0;
        E.nsrc = c.parted ? c.c_nsrc.as<int>() : nullptr;
        E.sh = f32 ? c.p2p_sh.as<float4>() : nullptr;
        const int ngb = (int)cdiv(n_p2p, TPB);
        c.gpart.ensure(2 * sizeof(unsigned long long) * (size_t)ngb);
        k_p2p_gather<<<ngb, TPB, 0, s>>>(E, c.p2p_raw.as<int4>(), c.lval.as<uint32_t>(), n_p2p, c.p2p_ent.as<int4>(),
                                         c.gpart.as<unsigned long long>());
        VFMM_LAUNCH_CHECK();
        k_sum_u64x2<<<1, TPB, 0, s>>>(c.gpart.as<unsigned long long>(), ngb, c.pairs64.as<unsigned long long>());
        VFMM_LAUNCH_CHECK();
    }
    // ---- P2P work: blocks of <= 64 targets, their lists in parts ----
    const int nl = c.nleaves;
    c.c_tmp.ensure(sizeof(int) * (2 * LEAF_SUMS * (size_t)nl + 2));
    int *cnt = c.c_tmp.as<int>(), *off = cnt + LEAF_SUMS * (size_t)nl;
    const int *nsrc = c.parted ? c.c_nsrc.as<int>() : nullptr;
    const unsigned long long *tot = c.pairs64.as<unsigned long long>();
    const int ncb = (int)cdiv(nl, TPB);
    c.gpart.ensure(sizeof(unsigned long long) * (size_t)ncb);
    int h[LEAF_SUMS + 4];
    auto count64 = [&](int k) { return (int64_t)((uint64_t)(uint32_t)h[k] | ((uint64_t)(uint32_t)h[k + 1] << 32)); };
    float stretch = 1.f;
    c.n_partial = (int)fit_parts(partials_limit(c.n), [&](float by) {
        k_leaf_counts<<<ncb, TPB, 0, s>>>(c.leaves.as<int>(), nl, c.c_count.as<int>(), nsrc, c.p2p_off.as<int>(), tot,
                                          n_p2p, by, cnt, c.gpart.as<unsigned long long>());
        VFMM_LAUNCH_CHECK();
        scan_excl_i32(c, cnt, off, LEAF_SUMS * (int64_t)nl);
        k_leaf_totals<<<1, TPB, 0, s>>>(cnt, off, nl, c.pairs64.as<int>(), c.gpart.as<unsigned long long>(), ncb,
                                        pinned_ints(c));
        VFMM_LAUNCH_CHECK();
        sync_ints(c, LEAF_SUMS + 4, h);
        return count64(LEAF_SUMS + 2);
    }, stretch);
    c.n_blocks = h[0];
    c.n_pblocks = h[1];
    ItemKinds K{};
    int items = 0;  // at most n_partial
    for (int k = 0; k < 4; ++k) {
        c.item0[k] = K.first[k] = items;
        items += h[2 + k];
    }
    c.item0[4] = items;
    c.n_long = h[7];
    c.p2p_pairs = count64(LEAF_SUMS);
    c.blocks.ensure(sizeof(int4) * (size_t)std::max(c.n_blocks, 1));
    c.pblong.ensure(sizeof(int) * (size_t)std::max(c.n_long, 1));
    c.pblocks.ensure(sizeof(int4) * (size_t)std::max(c.n_pblocks, 1));
    c.items.ensure(sizeof(int4) * (size_t)std::max(items, 1));
    c.item_out.ensure(sizeof(int) * (size_t)std::max(items, 1));
    k_leaf_items<<<cdiv(nl, TPB / 64), TPB, 0, s>>>(c.leaves.as<int>(), nl, c.c_start.as<int>(), c.c_count.as<int>(),
                                                    nsrc, c.p2p_off.as<int>(), tot, n_p2p, stretch, off, K,
                                                    c.blocks.as<int4>(), c.pblocks.as<int4>(), c.pblong.as<int>(),
                                                    c.items.as<int4>(), c.item_out.as<int>());
    VFMM_LAUNCH_CHECK();
}

}  // namespace vfmm
