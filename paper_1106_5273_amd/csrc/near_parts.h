// How the near field is cut into work: a leaf's targets into blocks, a block's
// list into parts, one wave and one set of partial results each.  Plain
// arithmetic on counts, used by the kernels that lay the work out and, compiled
// for the host, by their tests.
#pragma once

#include <algorithm>
#include <cmath>
#include <cstdint>

#ifdef __HIPCC__
#define VFMM_HD __host__ __device__
#else
#define VFMM_HD
#endif

namespace vfmm {

// Lane groups of a near-field block of tc targets: more than 32 targets take the
// wave alone; fewer are held by several groups of tc lanes each (at most 16),
// which take different sources.
VFMM_HD inline int p2p_groups(int tc) { return tc > 32 ? 1 : tc < 4 ? 16 : 64 / tc; }

// ---------------------------------------------------------------------------
// P2P work: every leaf's targets are cut into blocks of at most 64, and every
// block's list into parts of about equal length, one wave each.  The length of
// a part is chosen from the whole build's work: total wave steps / 172,032 (21
// rounds of the 8,192 waves that fill the chip), but at least 48 steps (shorter
// parts cost more in their prologue and partial sums than they spread) and at
// most 1,200.  More than two parts are made a multiple of the four waves of a
// work-group, which then share one block's targets and neighbouring sources: 512
// rings with leaves of 384 take 60.3 ms an evaluation with 8 parts a block, 68.3
// with 4, 68.8 with 6 and 71.6 with 3; 128^3 takes four or eight alike.  A fixed
// four parts per block left one list of 4,849 entries in a clustered tree of
// 100,003 particles to four waves, which alone set the kernel's time.
// Every part writes six values per target, so large leaves, whose lists are long
// (leaves of 512: up to 64 parts a block), are kept within partials_limit of
// them by longer parts (fit_parts).  128^3 in leaves of 512: 60.8 ms with parts
// of that length, 62.2 with parts of 1,200 steps (1.7 GB more), 61.6 with four a block.
// ---------------------------------------------------------------------------
struct LeafWork {
    float src_per_entry;  // mean sources of a list entry
    float part;           // wave steps per part
};

// pairs, srcs: particle pairs and sources of all list entries; stretch >= 1: fit_parts
VFMM_HD inline LeafWork leaf_work(uint64_t pairs, uint64_t srcs, int64_t nent, float stretch) {
    LeafWork w;
    w.src_per_entry = std::max(1.f, (float)srcs / (float)(nent > 0 ? nent : 1));
    w.part = stretch * std::min(1200.f, std::max(48.f, (float)pairs * (1.f / (48.f * 172032.f))));
    return w;
}

// The remainder r = 1 .. 63 of a leaf's targets past its blocks of 64 is cut
// into k blocks of nearly equal size.  A block of more than 32 targets leaves
// the other lanes idle, one of g <= 32 fills the wave with several groups that
// take different list entries (p2p_groups), so the wave rounds per list entry
// are k / p2p_groups(ceil(r / k)); k grows where that saves at least a fifth
// (33 .. 42 targets: two blocks, 2/3; 43 .. 48: three, 3/4).  Leaves of 27, 36
// and 48 (per-particle cores, 50^3): near field 1.28 -> 1.10 ms.
VFMM_HD inline int remainder_blocks(int r) {
    int best = 1;
    float cost = 1.f / (float)p2p_groups(r);
    for (int k = 2; k <= 3 && k <= r; ++k) {
        const float ck = (float)k / (float)p2p_groups((r + k - 1) / k);
        if (ck <= 0.8f * cost) {
            best = k;
            cost = ck;
        }
    }
    return best;
}

// The near-field blocks of a leaf of cnt targets, of which the first ns are
// particles and the rest target points without strength (their blocks compute
// the velocity alone): f(first target, targets, whether target points).
template <class F>
VFMM_HD inline void leaf_blocks(int cnt, int ns, F f) {
    for (int half = 0; half < 2; ++half) {
        const int lo = half ? ns : 0, c = half ? cnt - ns : ns;
        const int full = c / 64, r = c % 64;
        for (int b = 0; b < full; ++b) f(lo + 64 * b, 64, half != 0);
        if (r == 0) continue;
        const int k = remainder_blocks(r);
        for (int q = 0; q < k; ++q) {
            const int a = q * r / k, e = (q + 1) * r / k;
            f(lo + 64 * full + a, e - a, half != 0);
        }
    }
}

// parts of the list (lc entries) of a block of tc targets: whole-wave blocks
// take an entry's sources one per step with a fixed cost of about six steps
// per entry, lane groups take a share of the list's sources; a part of theirs
// holds at least 128 sources (the last pass of 64 is partly empty)
VFMM_HD inline int list_parts(const LeafWork &W, int tc, int lc) {
    const float cap = (float)lc;  // every part keeps an entry
    if (tc > 32) {
        const int np = std::max(1, std::min(lc, (int)std::min(cap, cap * (W.src_per_entry + 6.f) / W.part + 0.5f)));
        return np > 2 ? std::min(lc, (np + 2) / 4 * 4) : np;
    }
    const float srcs = cap * W.src_per_entry;
    const float most = std::min(cap, srcs * (1.f / 128.f));
    return std::max(1, std::min(lc, (int)std::min(most, srcs / ((float)p2p_groups(tc) * W.part) + 0.5f)));
}

// The targets times parts that a build of n targets may have (each holds six
// values, 24 bytes in float32): 12 n, which leaves of 384 with 8 parts a block
// stay below, or 2^25 (0.8 GB) where that is more; from 2^30 on (89 million
// targets) no more than that or four per target, and always a 32-bit count.
VFMM_HD inline int64_t partials_limit(int64_t n) {
    const int64_t most = std::max<int64_t>(std::min<int64_t>(12 * n, int64_t(1) << 30), 4 * n);
    return std::min<int64_t>(std::max<int64_t>(most, int64_t(1) << 25), INT32_MAX);
}

// Lays the work out with longer and longer parts until its targets times parts,
// count(stretch), are within the limit.  Ends: with parts of any length every
// block has one, and that makes n < 2^31 of them.
template <class F>
inline int64_t fit_parts(int64_t limit, F count, float &stretch) {
    stretch = 1.f;
    for (;;) {
        const int64_t total = count(stretch);
        if (total <= limit) return total;
        stretch *= std::max(1.25f, (float)((double)total / (double)limit));
    }
}

}  // namespace vfmm
