// Co-mining kernel for gfx950 (CDNA4, wave64).  This header is included once
// per tree depth by search_d<depth>_t<bits>.hip (one translation unit per tree depth and time width).
//
// What runs here is the co-mining recursion of the paper (Algorithm 3, built
// on the per-motif matcher of Algorithm 1): from every root edge, partial
// matches are extended edge by edge along the search levels of the motif
// group's prefix trie; reaching a trie node credits every motif whose edge
// sequence equals that prefix, and the same partial match then continues into
// all of the node's children.
//
// How it is laid out for the hardware (not the paper's warp-per-candidate
// design):
//   * Every wave is an independent worker.  Root edges are split into eight
//     contiguous (time-ordered) queues, one per XCD; a wave starts with the
//     chunk at its own place, claims more from its XCD's queue and steals from
//     the others when it runs dry, so roots that are close in time, and the
//     adjacency they read, share one L2.  Claims are what bounds small counts
//     (about 20 ns each on one head), so few are made.
//   * Root-level candidates of a chunk beyond a limit are handed on as
//     contexts, which a second launch spreads over the device.
//   * Partial matches are buffered per search level in LDS and expanded 64 at
//     a time, the last ones first, with a live word each: which of the lists
//     it could scan, and of the pairs it could count, hold anything within the
//     window.  It is made of the next codes that come with every list entry,
//     so empty windows (nearly all of them in deep trees) cost nothing.
//   * Children that read the same list (same direction, same anchor vertex)
//     form one group and share one scan of the window: the entries with
//     t_prev < t <= t_first + delta.
//   * Windows are found from other windows where possible: a root's windows
//     in out(a) and in(b) start just past the root edge's own list position,
//     and a deeper window on a list of the root's two vertices lies inside the
//     root's window on that list (kept in LDS), so it needs a short bisection
//     and no search for its end.
//   * A window whose children all end a motif is counted, not expanded.  Where
//     a matched edge joins the list's vertex to the bound vertex that the child
//     ends on, the entries that count are edges of that pair: two positions in
//     the pair order, no scan (before, 99.6 % of all scanned entries lay in
//     such windows; 20M edges and 36 motifs took 6.75 ms, now 2.96).  Other
//     such windows take one equality count per bound vertex, the new-vertex
//     child taking the rest; a short one by its own lane, a long one by the
//     whole wave with ballots.
//   * The other non-empty windows, up to 64 at a time, are expanded as one
//     flat candidate range: lane i takes candidate c + i, finds its window
//     from a 64-bit mask of window ends (LDS flags + ballot + popcount), reads
//     one adjacency entry, finds which bound motif vertex it hits with
//     predicated compares, picks the reached child from the group record
//     (which also carries the child's motif id), credits LDS counters, counts
//     the pairs of a leaf parent, and compacts the survivors that still have
//     something to find into the next level's buffer with ballot + mbcnt.
//   * What bounds it (20M edges): the latency of list lines that miss L2, 403
//     bytes of traffic per root edge, waves waiting 77 % of their cycles at
//     eight waves per SIMD; then VALU issue (59 %).
//   * The level loop nest is unrolled at compile time for the tree depth
//     (1..5 motif edges), one instantiation per depth.
#pragma once
#include <hip/hip_runtime.h>

#include <algorithm>

#include "comine.h"
#include "device_util.h"

namespace mg {
namespace {


constexpr uint32_t kChunkLimit = 0x7fffffffu;   // candidates per window chunk

// Kernel parameters stay in constant memory and are read where they are used:
// there are more of them than scalar registers, and kept there from the start
// they were spilled and fetched back lane by lane in the inner loops.  fresh()
// hides where a reference comes from, so that nothing read through an earlier
// one is kept; pointers read this way are marked as global memory by glb().
template <typename TT>
using ConstParams = const __attribute__((address_space(4))) KParams<TT> *;
template <typename TT>
__device__ __forceinline__ const KParams<TT> &fresh(const KParams<TT> &p) {
    ConstParams<TT> a = (ConstParams<TT>)&p;
    asm volatile("" : "+s"(a));
    return *(const KParams<TT> *)a;
}
template <typename T>
__device__ __forceinline__ T *glb(T *x) {
    return (T *)(__attribute__((address_space(1))) T *)x;
}

// child word of a group for scanned-endpoint index y (0..5 bound, else new)
__device__ __forceinline__ uint32_t child_word(const uint4 &a, const uint4 &b, int y) {
    uint32_t r = b.w;             // new vertex
    r = (y == 0) ? a.y : r;
    r = (y == 1) ? a.z : r;
    r = (y == 2) ? a.w : r;
    r = (y == 3) ? b.x : r;
    r = (y == 4) ? b.y : r;
    r = (y == 5) ? b.z : r;
    return r;
}

// The smaller window j of a multi-window tree (selects, so that the
// parameter array is never indexed at run time: a local copy of it would go
// to scratch memory).
template <typename TT>
__device__ __forceinline__ TT window_lo(const KParams<TT> &p, uint32_t j) {
    TT r = p.dlo[0];
#pragma unroll
    for (int i = 1; i < kMaxDeltas - 1; ++i) r = j == (uint32_t)i ? p.dlo[i] : r;
    return r;
}

// Window slot of a match with first time tf and last time tl: the number of
// smaller windows its span exceeds.
template <typename TT>
__device__ __forceinline__ uint32_t window_slot(const KParams<TT> &p, uint32_t nd, TT tf, TT tl) {
    uint32_t j = 0;
#pragma unroll
    for (int i = 0; i < kMaxDeltas - 1; ++i)
        j += ((uint32_t)i + 1 < nd && tl > sat_add(tf, p.dlo[i])) ? 1u : 0u;
    return j;
}

// c matches of the child in `word`, credited to window slot j of its motif
// (nd slots per motif).  With `move`, the c matches were already credited to
// slot j + 1 (they lie in a larger window too) and move down to slot j: slot
// j + 1 loses them.  The counters are summed over slots modulo 2^64, so a
// slot may hold a negative amount in between.
__device__ __forceinline__ uint32_t credit_child(uint32_t word, uint32_t c,
                                                unsigned long long *cnt, uint32_t nd,
                                                uint32_t j, bool move = false) {
    if (!c || !word) return 0;
    const uint32_t q1 = (word >> 16) & 0x7fffu;
    if (q1) {
        atomicAdd(&cnt[(q1 - 1) * nd + j], (unsigned long long)c);
        if (move) atomicAdd(&cnt[(q1 - 1) * nd + j + 1], 0ull - c);
    }
    return move ? 0u : c;
}

// Counts a leaf-only window [l0, l0 + len) of one adjacency list for one
// partial match: each entry reaches the child of the bound vertex it hits, or
// the new-vertex child.  The bound vertices are distinct, so an entry hits at
// most one of them: one equality count per bound vertex, and the new-vertex
// child gets the rest of the window.  The list's own anchor is left out of
// q[] (no entry equals it: lists hold no self-loops); q[0..K) are the other
// bound vertices (-1 for none) and w[0..K) their child words, wn the
// new-vertex child's word.  Credits go to window slot j of each motif (nd
// slots per motif).  Returns the credits.
template <int U, int K, typename TT, int N>
__device__ __forceinline__ uint32_t leaf_count(const Entry<TT> *__restrict__ adj, uint32_t l0,
                                               uint32_t len, const int32_t (&q)[N],
                                               const uint32_t (&w)[N], uint32_t wn,
                                               unsigned long long *cnt, uint32_t nd,
                                               uint32_t j, bool move = false) {
    static_assert(K <= N, "slots");
    uint32_t c[K];
#pragma unroll
    for (int s = 0; s < K; ++s) c[s] = 0;
    // U independent loads per step, the last step included: there an index
    // past the window reloads its last entry (len >= 1) and counts as no hit,
    // so a window of up to U entries costs one memory trip
    const Entry<TT> *e = adj + l0;
    uint32_t i = 0;
    for (; i + U <= len; i += U) {
        int32_t v[U];
#pragma unroll
        for (int j = 0; j < U; ++j) v[j] = e[i + j].v;
#pragma unroll
        for (int j = 0; j < U; ++j)
#pragma unroll
            for (int s = 0; s < K; ++s) c[s] += v[j] == q[s];
    }
    if (i < len) {
        int32_t v[U];
#pragma unroll
        for (int j = 0; j < U; ++j) v[j] = e[min(i + j, len - 1)].v;
#pragma unroll
        for (int j = 0; j < U; ++j) {
            const int32_t x = i + j < len ? v[j] : -2;   // -2 matches no vertex
#pragma unroll
            for (int s = 0; s < K; ++s) c[s] += x == q[s];
        }
    }
    uint32_t hit = 0, got = 0;
#pragma unroll
    for (int s = 0; s < K; ++s) {
        hit += c[s];
        got += credit_child(w[s], c[s], cnt, nd, j, move);
    }
    return got + credit_child(wn, len - hit, cnt, nd, j, move);
}


// Counts the leaf-only window [l0, l0 + len) of group g for the partial match
// with bound vertices ph[] with the whole wave, 64 entries per pass: one ballot per bound
// vertex counts the entries that hit it, and the new-vertex child gets the
// rest.  All arguments are wave-uniform.  Credits go to window slot j.
// Returns the credits on lane 0 (0 on the other lanes).
template <typename TT, int SA>
__device__ __forceinline__ uint32_t leaf_scan_wave(const KParams<TT> &p, const int32_t (&ph)[SA],
                                                   uint32_t g, uint32_t l0, uint32_t len,
                                                   const int lane, unsigned long long *cnt,
                                                   uint32_t nd, uint32_t j, bool move = false) {
    const uint4 ga = glb(p.tree.grp)[3 * g], gb = glb(p.tree.grp)[3 * g + 1];
    const uint32_t nvp = (ga.x >> 8) & 15;
    const Entry<TT> *__restrict__ e =
        ((ga.x & 15) == kDirOut ? glb(p.g.out_adj) : glb(p.g.in_adj)) + l0;
    int32_t q[SA];
    uint32_t c[SA];
#pragma unroll
    for (int s = 0; s < SA; ++s) {
        q[s] = (uint32_t)s < nvp ? ph[s] : -1;
        c[s] = 0;
    }
    uint32_t i = 0;
    for (; i + 4 * kWave <= len; i += 4 * kWave) {
        int32_t v[4];
#pragma unroll
        for (int j = 0; j < 4; ++j) v[j] = e[i + j * kWave + lane].v;
#pragma unroll
        for (int j = 0; j < 4; ++j)
#pragma unroll
            for (int s = 0; s < SA; ++s) c[s] += (uint32_t)__popcll(__ballot(v[j] == q[s]));
    }
    for (; i < len; i += kWave) {
        const int32_t v = i + lane < len ? e[i + lane].v : -2;   // -2 matches no slot
#pragma unroll
        for (int s = 0; s < SA; ++s) c[s] += (uint32_t)__popcll(__ballot(v == q[s]));
    }
    if (lane != 0) return 0;
    const uint32_t words[6] = {ga.y, ga.z, ga.w, gb.x, gb.y, gb.z};
    uint32_t hit = 0, got = 0;
#pragma unroll
    for (int s = 0; s < SA; ++s) {
        hit += c[s];
        got += credit_child(words[s], c[s], cnt, nd, j, move);
    }
    return got + credit_child(gb.w, len - hit, cnt, nd, j, move);
}

// The same for a tree with several windows: the whole window counts at the
// largest window, and each smaller window, a prefix of it whose length the
// same pass measures (entries with t <= t_first + its delta, one ballot per
// window), moves its matches down one slot with a second, shorter pass.
// tf: the partial match's first time.
template <typename TT, int SA>
__device__ __forceinline__ uint32_t leaf_scan_wave_multi(const KParams<TT> &p,
                                                         const int32_t (&ph)[SA], uint32_t g,
                                                         uint32_t l0, uint32_t len, TT tf,
                                                         const int lane, unsigned long long *cnt,
                                                         uint32_t nd) {
    const uint4 ga = glb(p.tree.grp)[3 * g], gb = glb(p.tree.grp)[3 * g + 1];
    const uint32_t nvp = (ga.x >> 8) & 15;
    const Entry<TT> *__restrict__ e =
        ((ga.x & 15) == kDirOut ? glb(p.g.out_adj) : glb(p.g.in_adj)) + l0;
    int32_t q[SA];
    uint32_t c[SA];
#pragma unroll
    for (int s = 0; s < SA; ++s) {
        q[s] = (uint32_t)s < nvp ? ph[s] : -1;
        c[s] = 0;
    }
    TT thr[kMaxDeltas - 1];
    uint32_t pre[kMaxDeltas - 1];
#pragma unroll
    for (int j = 0; j < kMaxDeltas - 1; ++j) {
        thr[j] = sat_add(tf, p.dlo[j]);
        pre[j] = 0;
    }
    // four independent loads per pass while whole, then one at a time
    uint32_t i = 0;
    for (; i + 4 * kWave <= len; i += 4 * kWave) {
        Entry<TT> en[4];
#pragma unroll
        for (int k = 0; k < 4; ++k) en[k] = e[i + k * kWave + lane];
#pragma unroll
        for (int k = 0; k < 4; ++k) {
#pragma unroll
            for (int s = 0; s < SA; ++s) c[s] += (uint32_t)__popcll(__ballot(en[k].v == q[s]));
#pragma unroll
            for (int j = 0; j < kMaxDeltas - 1; ++j)
                if ((uint32_t)j + 1 < nd) pre[j] += (uint32_t)__popcll(__ballot(en[k].t <= thr[j]));
        }
    }
    for (; i < len; i += kWave) {
        const bool in = i + lane < len;
        Entry<TT> en{};
        if (in) en = e[i + lane];
        const int32_t v = in ? en.v : -2;   // -2 matches no slot
#pragma unroll
        for (int s = 0; s < SA; ++s) c[s] += (uint32_t)__popcll(__ballot(v == q[s]));
#pragma unroll
        for (int j = 0; j < kMaxDeltas - 1; ++j)
            if ((uint32_t)j + 1 < nd) pre[j] += (uint32_t)__popcll(__ballot(in && en.t <= thr[j]));
    }
    uint32_t got = 0;
    if (lane == 0) {
        const uint32_t words[6] = {ga.y, ga.z, ga.w, gb.x, gb.y, gb.z};
        uint32_t hit = 0;
#pragma unroll
        for (int s = 0; s < SA; ++s) {
            hit += c[s];
            got += credit_child(words[s], c[s], cnt, nd, nd - 1);
        }
        got += credit_child(gb.w, len - hit, cnt, nd, nd - 1);
    }
#pragma unroll
    for (int j = kMaxDeltas - 2; j >= 0; --j)
        if ((uint32_t)j + 1 < nd && pre[j] > 0)
            leaf_scan_wave<TT, SA>(p, ph, g, l0, pre[j], lane, cnt, nd, (uint32_t)j, true);
    return got;
}

// Partial matches with L motif edges matched.  Level 1 is the root batch:
// every entry is at the trie root and its last edge is its first, so it keeps
// only the two bound vertices and the root time.
// R: 1 = each partial match also keeps its root edge (the per-root cost log),
// 2 = its root edge and the slot of its parent one level up (enumeration,
// which writes out every matched edge).
// V: vertex slots, the most motif vertices bound at this level (vslots).
template <typename TT, int D, int L, int R, int V>
struct LevelBuf {
    static constexpr int S = V;              // vertex slots
    static constexpr int C = 2 * kWave;      // capacity
    static constexpr bool E2 = L == 3;
    // phi[s - 2][i]: graph vertex of motif vertex s >= 2; motif vertices 0 and
    // 1 and t_first are the root's, kept once in the level-1 batch (slot r1)
    int32_t phi[S - 2][C];
    uint32_t eid[C];       // edge id of its last matched edge
    uint32_t eid2[E2 ? C : 1];   // edge id of its second edge (level 3)
    uint32_t live[C];      // its live word (comine.h), with its root's slot
    uint16_t node[C];      // internal trie node reached
    uint16_t pincl[kWave]; // inclusive prefix of a batch's counts of live lists
    uint32_t root[R ? C : 1];
    uint8_t par[R == 2 && L > 2 ? C : 1];   // slot of its parent at level L - 1
};
template <typename TT, int D, int R, int V>
struct LevelBuf<TT, D, 1, R, V> {
    static constexpr int S = 2;
    static constexpr int C = kWave;
    int32_t phi[2][kWave];
    TT tfirst[kWave];
    uint32_t root[kWave];        // edge id
    uint8_t live[kWave];         // live bits of its lists (0-3) and of its pair (4, 5)
    // how long after the root the last edge of its pair within the window
    // comes (next_code), of the pair against it (room for that at depth 3 only)
    static constexpr int Q = D == 3 ? 2 : 1;
    uint8_t last[Q][kWave];
    uint8_t pair[4 * kWave];     // live (root, list) pairs: slot | list << 6
};

// Vertex slots at level L of a kernel for trees of depth D: two per edge, at
// most kVMax.  Depth-3 kernels keep three at level 2, which holds for trees
// whose buffered two-edge prefixes share a vertex; the host runs trees with a
// four-vertex two-edge prefix on the depth-4 kernel (DevTree::kdepth).  The
// slot saved is registers the compiler no longer spills.
constexpr int vslots(int D, int L) {
    return (D == 3 && L == 2) ? 3 : (2 * L < kVMax ? 2 * L : kVMax);
}

template <typename TT, int D, int R, int L>
struct LevelChain {
    LevelBuf<TT, D, L, R, vslots(D, L)> buf;
    LevelChain<TT, D, R, L + 1> next;
};
template <typename TT, int D, int R>
struct LevelChain<TT, D, R, D> {};

// per-wave LDS: level buffers plus small scratch tables.  Its size is a
// multiple of 16 bytes, so that per-wave blocks laid out back to back (with
// 64-bit counters between them) keep those counters 8-byte aligned, as LDS
// 64-bit atomics require.
//
// Root windows: for each root of the level-1 batch, the windows it found in
// out(a), in(a), out(b), in(b) (index anchor * 2 + direction): first entry and
// length, kNoHint as length when not found yet, kLongHint with the window's
// end (not its first entry) when it has 65534 entries or more.  A deeper
// partial match of that root reads a window of the same
// list with t_prev < t <= t_first + delta, t_prev > t_first: it starts inside
// the root's window and ends where it ends, so a bisection over the root's
// window replaces a bisection over the whole list and the search for the end.
//
// An enumerating wave (R == 2) also keeps the matches it has not written out
// yet: per match its motif and its edges, up to D of them.
template <int D, int R>
struct MatchStage {};
template <int D>
struct MatchStage<D, 2> {
    static constexpr int C = 2 * kWave;
    uint32_t word[1 + D][C];
    uint32_t n;
};
template <typename TT, int D, int R>
struct alignas(16) WaveLds : MatchStage<D, R> {
    static constexpr int H = D > 1 ? 4 : 1;
    uint8_t flag[kWave];          // window-end marks of one pass
    uint32_t hlo[H][kWave];       // root windows (used when D > 2)
    uint16_t hlen[H][kWave];
    LevelChain<TT, D, R, 1> lv;
};

static_assert(sizeof(WaveLds<uint32_t, 1, 0>) % 16 == 0, "per-wave LDS block size");
static_assert(sizeof(WaveLds<uint32_t, 3, 0>) % 16 == 0, "per-wave LDS block size");
static_assert(sizeof(WaveLds<uint32_t, 5, 0>) % 16 == 0, "per-wave LDS block size");
static_assert(sizeof(WaveLds<uint64_t, 5, 1>) % 16 == 0, "per-wave LDS block size");
static_assert(sizeof(WaveLds<uint64_t, 5, 2>) % 16 == 0, "per-wave LDS block size");

constexpr uint16_t kNoHint = 0xffff;
constexpr uint16_t kLongHint = 0xfffe;

// A new root a -> b in level-1 slot `slot`: its root windows are not found
// yet; their first-entry words hold where they start, the first entries
// after the root's time in out(a), in(a), out(b) and in(b).
template <typename TT, int D, int R>
__device__ __forceinline__ void set_root_slot(WaveLds<TT, D, R> &W, uint32_t slot, uint4 gx) {
    W.hlo[0][slot] = gx.x;
    W.hlo[1][slot] = gx.y;
    W.hlo[2][slot] = gx.z;
    W.hlo[3][slot] = gx.w;
#pragma unroll
    for (int k = 0; k < 4; ++k) W.hlen[k][slot] = kNoHint;
}

// Live bits of root edge e, as the level-1 batch keeps them: bits 0-3 out(a),
// in(a), out(b), in(b), bits 4 and 5 its pair a -> b and b -> a.
template <typename TT>
__device__ __forceinline__ uint32_t root_live(const KParams<TT> &p, uint32_t e) {
    const uint2 n = glb(p.g.gn)[e];
    const uint32_t q = next_code(p.delta_sat);
    uint32_t r = 0;
#pragma unroll
    for (int k = 0; k < 4; ++k) r |= ((n.y >> (8 * k)) & 255u) <= q ? 1u << k : 0u;
    r |= (n.x & 255u) <= q ? 16u : 0u;
    r |= ((n.x >> 8) & 255u) <= q ? 32u : 0u;
    return r;
}
// Time of the last entry of a pair, [pos, end) of the pair order, with t <= hi
// (kNever: none).  As pair_count: four at a time, then by galloping.
template <typename TT>
__device__ __forceinline__ TT pair_last(const TT *__restrict__ t, uint32_t pos, uint32_t end, TT hi) {
    TT last = kNever<TT>;
    for (int it = 0; pos < end; ++it) {
        if (it == 2) {
            const uint32_t e = gallop_greater(t, 0, pos, end, hi);
            return e > pos ? t[e - 1] : last;
        }
        TT v[4];
        __builtin_memcpy(v, t + pos, sizeof v);
#pragma unroll
        for (int k = 0; k < 4; ++k)
            if (v[k] <= hi && pos + (uint32_t)k < end) last = v[k];
        if (pos + 4 >= end || v[3] > hi) break;
        pos += 4;
    }
    return last;
}

// The last edges of root e's pairs within its window, into slot `slot` of the
// level-1 batch; returns its live bits without those of pairs that have none.
// (In a burst the edges that repeat the root come right after it, and most of
// the later candidates need not look for more: 3.27 -> 3.08 ms for 20M edges.)
template <typename TT, typename Buf>
__device__ __forceinline__ uint32_t set_pair_ends(const KParams<TT> &p, Buf &A, uint32_t slot,
                                                  uint32_t e, TT t, uint32_t live) {
    const TT thi = sat_add(t, p.delta_sat);
#pragma unroll
    for (int k = 0; k < Buf::Q; ++k) {
        uint32_t q = 0;
        if (live & (p.tree.root_pairs << 4) & (16u << k)) {   // (looked up only if counted)
            const uint2 pr = reinterpret_cast<const uint2 *>(glb(p.g.gp))[2 * (size_t)e + k];
            const TT last = pair_last(glb(p.g.pair_t), pr.x, pr.y, thi);
            if (last == kNever<TT>) live &= ~(16u << k);
            else q = next_code((TT)(last - t));
        }
        A.last[k][slot] = (uint8_t)q;
    }
    return live;
}

// the same as live-word bits
__device__ __forceinline__ uint32_t root_bits(uint32_t r) {
    return (r & 15u) | ((r >> 4) << kLivePair);
}

template <int L, typename TT, int D, int R, int M>
__device__ __forceinline__ LevelBuf<TT, D, L, R, vslots(D, L)> &lvl(LevelChain<TT, D, R, M> &c) {
    if constexpr (L == M) return c.buf;
    else return lvl<L>(c.next);
}

// What the level buffers keep per partial match beyond the search itself
// (the R of LevelBuf) in each kernel MODE.
constexpr int keep_of(int mode) { return mode == 2 ? 1 : mode == 4 ? 2 : 0; }
// MODE 5 and 6 are MODE 0 and 3 with epochs (context offload, KParams::ctx_*)
constexpr bool single_of(int mode) { return mode == 0 || mode == 5; }   // one window
constexpr bool plain_of(int mode) { return mode == 0 || mode == 3 || mode == 5 || mode == 6; }
constexpr bool epochs_of(int mode) { return mode == 5 || mode == 6; }

// Enumeration: the edge ids of partial match i at level L, first edge first,
// into e[0..L), following the parent slots up to the root batch.
template <int L, typename TT, int D>
__device__ __forceinline__ void edge_chain(WaveLds<TT, D, 2> &W, uint32_t i, uint32_t (&e)[kKMax]) {
    if constexpr (L == 1) {
        e[0] = lvl<1>(W.lv).root[i];
    } else {
        auto &A = lvl<L>(W.lv);
        e[L - 1] = A.eid[i];
        if constexpr (L == 2) edge_chain<1>(W, A.live[i] >> kLiveSlot, e);
        else edge_chain<L - 1>(W, A.par[i], e);
    }
}

// Enumeration: the wave's staged matches written out as records (motif, then
// the edges and -1 up to kKMax) at consecutive slots, taken with one atomic.
// Slots past the capacity are dropped.  Returns true once there are any: the
// records are of no use then, and the wave ends its search (22 million matches
// of 2M edges into room for 1,000 took 5.7 ms, of which a count is 0.4).
template <typename TT, int D>
__device__ __forceinline__ bool flush_matches(const KParams<TT> &p, WaveLds<TT, D, 2> &W, int lane) {
    const uint32_t n = uniform(W.n);
    if (!n) return false;
    unsigned long long base = 0;
    if (lane == 0) base = atomicAdd(p.enum_cursor, (unsigned long long)n);
    base = lane0_u64(base);
    constexpr uint32_t kWords = 1 + kKMax;
    if (base < p.enum_cap) {
        const uint32_t fit = (uint32_t)min((unsigned long long)n, (unsigned long long)p.enum_cap - base);
        int32_t *rec = p.enum_out + base * kWords;
        for (uint32_t w = (uint32_t)lane; w < fit * kWords; w += kWave) {
            const uint32_t i = w / kWords, j = w % kWords;
            rec[w] = j <= (uint32_t)D ? (int32_t)W.word[j][i] : -1;
        }
    }
    wave_sync();
    if (lane == 0) W.n = 0;
    wave_sync();
    return base + n > p.enum_cap;
}

// Enumeration: one match per lane with `want` (motif q, edges e[0..k)) staged
// in the wave's LDS, and written out 64 or more at a time.  The cursor is one
// address for the whole device, about 20 ns per atomic: taken once per pass (17
// matches on average) the kernel took 950 us for the 801,489 matches of 36
// three-edge motifs on 200,000 edges, with staged matches 645 us.
template <typename TT, int D>
__device__ __forceinline__ bool write_matches(const KParams<TT> &p, WaveLds<TT, D, 2> &W, int lane,
                                              bool want, uint32_t q, const uint32_t (&e)[kKMax],
                                              uint32_t k) {
    const uint64_t m = __ballot(want);
    if (!m) return false;
    const uint32_t n = uniform(W.n);
    if (want) {
        const uint32_t slot = n + mbcnt(m);
        W.word[0][slot] = q;
#pragma unroll
        for (int i = 0; i < D; ++i) W.word[1 + i][slot] = (uint32_t)i < k ? e[i] : ~0u;
    }
    const uint32_t now = n + (uint32_t)__popcll(m);   // at most 63 + 64
    wave_sync();
    if (lane == 0) W.n = now;
    wave_sync();
    return now >= (uint32_t)kWave && flush_matches<TT, D>(p, W, lane);
}

// Counts the leaf-only window [l0, l0 + len) of group g (header word hdr) for
// one partial match by its own lane: ph[] are its bound vertices, tf its
// first time.  nqm is the largest number of bound vertices compared by the
// lanes counting together (the count loop is compiled for it).  Credits go to
// the largest window, and with several windows each smaller one, a prefix of
// this one, moves its matches down one slot.  Returns the credits.
template <typename TT, int D, int MODE, int S>
__device__ __forceinline__ uint32_t count_leaf_window(const KParams<TT> &p, uint32_t g,
                                                      uint32_t hdr, const int32_t (&ph)[S],
                                                      TT tf, uint32_t l0, uint32_t len,
                                                      uint32_t nqm, unsigned long long *cnt,
                                                      uint32_t nd) {
    constexpr int NQ = S - 1;
    const uint32_t anc = (hdr >> 4) & 15;
    const uint32_t nq = ((hdr >> 8) & 15) - 1u;   // bound vertices, the anchor left out
    const uint4 ga = glb(p.tree.grp)[3 * g], gb = glb(p.tree.grp)[3 * g + 1];
    const uint32_t words[6] = {ga.y, ga.z, ga.w, gb.x, gb.y, gb.z};
    int32_t q[NQ];
    uint32_t w[NQ];
#pragma unroll
    for (int i = 0; i < NQ; ++i) {
        // slot i below the anchor, slot i + 1 from it on
        const bool below = (uint32_t)i < anc, on = (uint32_t)i < nq;
        q[i] = on ? (below ? ph[i] : ph[i + 1]) : -1;
        w[i] = on ? (below ? words[i] : words[i + 1]) : 0u;
    }
    const Entry<TT> *adj = (hdr & 15) == kDirOut ? glb(p.g.out_adj) : glb(p.g.in_adj);
    // loads per step (measured: 8 for trees up to depth 4, 4 deeper)
    constexpr int kLU = D <= 4 ? 8 : 4;
    auto count = [&](uint32_t n, uint32_t j, bool move) -> uint32_t {
        uint32_t c = 0;
        if constexpr (NQ >= 1) if (nqm == 1) c = leaf_count<kLU, 1>(adj, l0, n, q, w, gb.w, cnt, nd, j, move);
        if constexpr (NQ >= 2) if (nqm == 2) c = leaf_count<kLU, 2>(adj, l0, n, q, w, gb.w, cnt, nd, j, move);
        if constexpr (NQ >= 3) if (nqm == 3) c = leaf_count<kLU, 3>(adj, l0, n, q, w, gb.w, cnt, nd, j, move);
        if constexpr (NQ >= 4) if (nqm == 4) c = leaf_count<kLU, 4>(adj, l0, n, q, w, gb.w, cnt, nd, j, move);
        if constexpr (NQ >= 5) if (nqm == 5) c = leaf_count<kLU, 5>(adj, l0, n, q, w, gb.w, cnt, nd, j, move);
        return c;
    };
    // the whole window counts at the largest window
    const uint32_t c = count(len, nd - 1, false);
    if constexpr (!single_of(MODE)) {
        // each smaller window is a prefix of this one: its matches move down
        // one slot (usually it is empty)
        const TT *ta = times_of(adj);
        uint32_t e = l0 + len;
        for (uint32_t j = nd - 1; j-- > 0;) {
            e = gallop_greater(ta, kAdjShift<TT>, l0, e, sat_add(tf, window_lo(p, j)));
            if (e == l0) break;
            count(e - l0, j, true);
        }
    }
    return c;
}

// The number of bound vertices a lane compares in count_leaf_window (0 when it
// counts nothing), maximised over the lanes that run this together.
template <int S>
__device__ __forceinline__ uint32_t leaf_compares(bool counting, uint32_t hdr) {
    const uint32_t nq = counting ? ((hdr >> 8) & 15) - 1u : 0u;
    uint32_t nqm = 0;
#pragma unroll
    for (int k = 1; k < S; ++k) nqm += __ballot(nq >= (uint32_t)k) ? 1u : 0u;
    return nqm;
}

// The window of the root in slot r1 in list k (out(a), in(a), out(b), in(b)),
// a its vertex: [b, e) holds every deeper window on that list, and with true
// they end at e; without, the root had no such window to find.
template <typename TT, int D, int R>
__device__ __forceinline__ bool root_window(const WaveLds<TT, D, R> &W, const uint32_t *off,
                                            int32_t a, uint32_t k, uint32_t r1, uint32_t &b,
                                            uint32_t &e) {
    const uint32_t hl = W.hlen[k][r1], h = W.hlo[k][r1];
    b = h;
    e = h + hl;
    if (hl == kNoHint) {
        e = off[a + 1];   // it starts past the root's time
        return false;
    }
    if (hl == kLongHint) {
        b = off[a];
        e = h;
    }
    return true;
}

// Entries of a pair, [pos, end) of the pair order, with lo < t <= hi.  Most
// pairs have a few in a window, so four are looked at per load without a
// search (lanes stay together; pair_t is padded by four entries); what is left
// after eight is bisected.  (Galloping from the first entry instead: 4.78 ms
// for 3M edges and 756 motifs, against 4.32.)
template <typename TT>
__device__ __forceinline__ uint32_t pair_count(const TT *__restrict__ t, uint32_t pos, uint32_t end,
                                               TT lo, TT hi) {
    uint32_t c = 0;
    for (int it = 0; pos < end; ++it) {
        if (it == 2) {
            const uint32_t a = gallop_greater(t, 0, pos, end, lo);
            return c + gallop_greater(t, 0, a, end, hi) - a;
        }
        TT v[4];
        __builtin_memcpy(v, t + pos, sizeof v);
#pragma unroll
        for (int k = 0; k < 4; ++k)
            c += (v[k] > lo && v[k] <= hi && pos + (uint32_t)k < end) ? 1u : 0u;
        if (pos + 4 >= end || v[3] > hi) break;
        pos += 4;
    }
    return c;
}

// c matches less of the child in `word` at window slot j (the opposite of
// credit_child).
__device__ __forceinline__ void uncredit_child(uint32_t word, uint32_t c, unsigned long long *cnt,
                                               uint32_t nd, uint32_t j, bool move = false) {
    const uint32_t q1 = (word >> 16) & 0x7fffu;
    if (!c || !q1) return;
    atomicAdd(&cnt[(q1 - 1) * nd + j], 0ull - c);
    if (move) atomicAdd(&cnt[(q1 - 1) * nd + j + 1], (unsigned long long)c);
}

// Counts what pairs can count below a leaf parent.  Where every vertex a leaf
// window counts is joined to its anchor by a matched edge, the window needs no
// look at its entries: its edges between the anchor and a bound vertex are the
// later edges of that matched edge's pair, consecutive in the pair order and
// found from the edge.  (On 2M edges and the 36 three-edge motifs, such windows
// held 99.7 % of the entries of all leaf windows, mostly the bursts of a hub
// scanned once per entry of the burst; on 1M edges and 756 motifs of up to four
// edges 98 %.)  A new-vertex child gets the window's length, credited by
// count_leaf_parent, less the pairs, taken off here.  pairs: the live pairs the
// node counts (its edge 2 j, or 2 j + 1 against it), tab: its pair words, has_new:
// some are for new-vertex children,
// pair_of(k): the first later entry and the end of pair k, tp: the last edge's
// time, tf and thi: the window.
template <typename TT, int MODE, typename PairOf>
__device__ __forceinline__ void count_pairs(const KParams<TT> &p, unsigned long long *cnt,
                                            uint32_t pairs, const uint4 *__restrict__ tab,
                                            bool has_new, PairOf pair_of, TT tp, TT tf, TT thi,
                                            uint32_t nd) {
    for (; pairs; pairs &= pairs - 1) {
        const uint32_t k = (uint32_t)__builtin_ctz(pairs);
        const uint2 pr = pair_of(k);
        if constexpr (single_of(MODE)) {
            const uint32_t n = pair_count(glb(p.g.pair_t), pr.x, pr.y, tp, thi);
            if (n) {
                credit_child(tab[k].x, n, cnt, 1u, 0u);
                if (has_new) {
                    const uint2 w = make_uint2(tab[k].y, tab[k].z);
                    uncredit_child(w.x, n, cnt, 1u, 0u);
                    uncredit_child(w.y, n, cnt, 1u, 0u);
                }
            }
        } else {
            const uint32_t lo = gallop_greater(glb(p.g.pair_t), 0, pr.x, pr.y, tp);
            uint32_t e = gallop_greater(glb(p.g.pair_t), 0, lo, pr.y, thi);
            const uint4 w = tab[k];
            for (uint32_t j = nd; j-- > 0 && e != lo;) {
                const bool move = j + 1 < nd;
                if (move) e = first_greater(glb(p.g.pair_t), 0, lo, e, sat_add(tf, window_lo(p, j)));
                credit_child(w.x, e - lo, cnt, nd, j, move);
                uncredit_child(w.y, e - lo, cnt, nd, j, move);
                uncredit_child(w.z, e - lo, cnt, nd, j, move);
            }
        }
    }
}

// A partial match at level L whose trie node has leaf children only (every
// match below it is one more edge): the lane counts the windows of the node's
// lists in `todo` in turn (those that pairs do not count, and the lengths of
// those with a new-vertex child that they do).  A window longer than
// p.leaf_scan entries is left to the whole wave, which counts such windows
// between the lanes' turns.  nw: the node's words, ph[]: the bound vertices,
// eid and tp: the last edge and its time, eid2: the second edge (L 3), tf: the
// first time, live: the live word.
template <typename TT, int D, int MODE, int L, int S>
__device__ __forceinline__ void count_leaf_parent(const KParams<TT> &p,
                                                  WaveLds<TT, D, keep_of(MODE)> &W,
                                                  unsigned long long *cnt, const int lane,
                                                  const uint4 nw, uint32_t todo,
                                                  const int32_t (&ph)[S], uint32_t eid,
                                                  uint32_t eid2, TT tp, TT tf, uint32_t live,
                                                  uint32_t nd) {
    const uint32_t g0 = nw.x & 0xfffffu, lists = nw.y;
    const uint32_t r1 = live >> kLiveSlot;
    const TT thi = sat_add(tf, p.delta_sat);
    for (;;) {
        bool pend = false;     // a window for the whole wave: group pg, [pl0, pl0 + plen)
        uint32_t pg = 0, pl0 = 0, plen = 0;
        while (todo) {
            const uint32_t bit = (uint32_t)__builtin_ctz(todo);
            todo &= todo - 1;
            const uint32_t g = g0 + (uint32_t)__popc(lists & ((1u << bit) - 1u));
            const uint32_t dir = bit & 1u, anc = bit >> 1;
            const uint4 ga = glb(p.tree.grp)[3 * g], gb = glb(p.tree.grp)[3 * g + 1];
            const uint32_t hdr = ga.x, codes = glb(p.tree.grp)[3 * g + 2].x;
            // The out-list of a later vertex x whose children all end on a root
            // vertex (a or b; no new vertex): the edges x -> a and x -> b in the
            // window are also the entries equal to x in the windows of in(a)
            // and in(b), suffixes of the root's own windows.  Those are
            // counted instead when they are shorter than x's window.
            bool swap = false;
            uint32_t sw_lo[2] = {0, 0}, sw_hi[2] = {0, 0}, sw_word[2] = {0, 0}, sw_len = 0;
            int32_t sw_x = 0;
            if constexpr (single_of(MODE) && D == 3) {   // (measured slower for deeper trees)
                if (dir == kDirOut && anc >= 2 && (gb.w | ga.w | gb.x | gb.y | gb.z) == 0) {
                    const uint32_t hla = W.hlen[1][r1], hlb = W.hlen[3][r1];
                    const bool la = ga.y && (live & 2u), lb = ga.z && (live & 8u);
                    if ((!la || hla < kLongHint) && (!lb || hlb < kLongHint)) {
                        swap = true;
#pragma unroll
                        for (int t = 0; t < S; ++t) sw_x |= ph[t] & -(int32_t)(anc == (uint32_t)t);
                        const TT *tin = times_of(glb(p.g.in_adj));
#pragma unroll
                        for (int sv = 0; sv < 2; ++sv) {
                            sw_word[sv] = sv ? ga.z : ga.y;
                            if (!(sv ? lb : la)) continue;
                            const uint32_t k = 2u * (uint32_t)sv + 1u;   // in(a), in(b)
                            const uint32_t hb = W.hlo[k][r1];
                            sw_hi[sv] = hb + (sv ? hlb : hla);
                            sw_lo[sv] = first_greater(tin, kAdjShift<TT>, hb, sw_hi[sv], tp);
                            sw_len += sw_hi[sv] - sw_lo[sv];
                        }
                    }
                }
            }
            auto count_swapped = [&]() {
                constexpr int kLU = D <= 4 ? 8 : 4;
#pragma unroll
                for (int sv = 0; sv < 2; ++sv) {
                    if (sw_hi[sv] > sw_lo[sv]) {
                        const int32_t q1[1] = {sw_x};
                        const uint32_t w1[1] = {sw_word[sv]};
                        leaf_count<kLU, 1>(glb(p.g.in_adj), sw_lo[sv], sw_hi[sv] - sw_lo[sv], q1, w1, 0u,
                                           cnt, 1u, 0u);
                    }
                }
            };
            if (swap && sw_len <= 16u) {   // short enough whatever x's window is
                count_swapped();
                continue;
            }
            const Entry<TT> *adj = dir == kDirOut ? glb(p.g.out_adj) : glb(p.g.in_adj);
            const TT *ta = times_of(adj);
            uint32_t b = 0, e = 0, l0;
            bool hinted = false;
            // the anchor's vertex by masks: a select chain over ph[] would be
            // turned into an indexed load from scratch memory
            int32_t a = 0;
#pragma unroll
            for (int t = 0; t < S; ++t) a |= ph[t] & -(int32_t)(anc == (uint32_t)t);
            const uint32_t *off = dir == kDirOut ? glb(p.g.out_off) : glb(p.g.in_off);
            if (D > 2 && anc < 2) hinted = root_window(W, off, a, bit, r1, b, e);
            else { b = off[a]; e = off[a + 1]; }
            const uint32_t le = (hdr >> 13) & 3u;
            uint32_t be = 0;
            if constexpr (L == 3) be = anc >= 2 ? (hdr >> 15) & 3u : 0u;
            if (le || be) {
                // the list of an endpoint of the last edge: its rank is kept;
                // of the second edge: the window starts no earlier than there
                const uint32_t k = ((le ? le : be) == 1 ? 0u : 2u) + dir;
                l0 = reinterpret_cast<const uint32_t *>(glb(p.g.gx))[4 * (size_t)(le ? eid : eid2) + k];
                if (!le) l0 = gallop_greater(ta, kAdjShift<TT>, l0, e, tp);
            } else {
                l0 = first_greater(ta, kAdjShift<TT>, b, e, tp);
            }
            const uint32_t len = (hinted ? e : gallop_greater(ta, kAdjShift<TT>, l0, e, thi)) - l0;
            if (codes) {
                // the new-vertex child: the window's length (its pairs are off already)
                credit_child(gb.w, len, cnt, nd, nd - 1);
                if constexpr (!single_of(MODE)) {
                    uint32_t x = l0 + len;
                    for (uint32_t k = nd - 1; k-- > 0;) {
                        x = gallop_greater(ta, kAdjShift<TT>, l0, x, sat_add(tf, window_lo(p, k)));
                        if (x == l0) break;
                        credit_child(gb.w, x - l0, cnt, nd, k, true);
                    }
                }
                continue;
            }
            if (swap && sw_len < len) {
                count_swapped();
                continue;
            }
            if (len > p.leaf_scan) {
                pend = true; pg = g; pl0 = l0; plen = len;
                break;
            }
            const uint32_t nqm = leaf_compares<S>(len > 0, hdr);
            if (len > 0) count_leaf_window<TT, D, MODE>(p, g, hdr, ph, tf, l0, len, nqm, cnt, nd);
        }
        for (uint64_t cm = __ballot(pend); cm; cm &= cm - 1) {
            const int src = (int)__builtin_ctzll(cm);
            int32_t wph[S];
#pragma unroll
            for (int t = 0; t < S; ++t) wph[t] = (int32_t)__builtin_amdgcn_readlane(ph[t], src);
            const uint32_t wg = __builtin_amdgcn_readlane(pg, src);
            const uint32_t wl0 = __builtin_amdgcn_readlane(pl0, src);
            const uint32_t wlen = __builtin_amdgcn_readlane(plen, src);
            if (nd == 1)
                leaf_scan_wave<TT, S>(p, wph, wg, wl0, wlen, lane, cnt, 1u, 0u);
            else
                leaf_scan_wave_multi<TT, S>(p, wph, wg, wl0, wlen,
                                            lane_time(tf, src), lane, cnt, nd);
        }
        if (!__ballot(todo != 0)) break;
    }
}

// per-lane statistics (only the STATS instantiation touches them)
struct Stats {
    uint64_t v[kStats];
    bool stopped;   // claim no more work: the wave wrote contexts (an epoch ended), or its
                    // matches have no room left
};

// MODE: 0 plain search (trees with one window), 1 with search statistics, 2
// with the per-root cost log, 3 plain search of a tree with several windows,
// 4 enumeration (every match written out), 5 and 6: 0 and 3 with epochs
// At level 1 with nparts > 1 (one buffered root), only part `part` of the
// root's candidates is expanded: [T * part / nparts, T * (part + 1) / nparts)
// of its T candidates in window order, so that the parts of one root
// partition its search exactly; windows that a single lane counts, and the
// root's window statistics, belong to part 0.
template <typename TT, int D, int MODE, int L>
__device__ __forceinline__ void run_level(const KParams<TT> &p0, WaveLds<TT, D, keep_of(MODE)> &W,
                                          unsigned long long *cnt, const int lane,
                                          const uint32_t base, const uint32_t nA, Stats &st,
                                          const uint32_t part = 0, const uint32_t nparts = 1,
                                          const EpochCtx *ctx = nullptr) {
    constexpr bool STATS = MODE == 1, LOG = MODE == 2;
    const KParams<TT> &p = fresh(p0);
    auto &A = lvl<L>(W.lv);
    constexpr int SA = vslots(D, L);
    auto &R1 = lvl<1>(W.lv);
    // graph vertex of motif vertex s, and t_first, of buffered partial match i
    auto vtx = [&](uint32_t s, uint32_t i) -> int32_t {
        if constexpr (L == 1) return A.phi[s][i];
        else return s < 2 ? R1.phi[s][A.live[i] >> kLiveSlot] : A.phi[s < 2 ? 0 : s - 2][i];
    };
    auto slot_of = [&](uint32_t i) -> uint32_t {
        if constexpr (L == 1) return i;
        else return A.live[i] >> kLiveSlot;
    };
    auto tfirst_of = [&](uint32_t i) -> TT {
        if constexpr (L == 1) return A.tfirst[i];
        else return R1.tfirst[A.live[i] >> kLiveSlot];
    };
    const uint4 *__restrict__ inode = glb(p.tree.inode);
    const uint64_t le_mask = (lane == 63) ? ~0ull : ((2ull << lane) - 1);
    // windows counted at once (MODE 0 serves trees with one window only)
    const uint32_t nd = single_of(MODE) ? 1u : (uint32_t)p.tree.n_d;

    // leaf parents are counted by their lanes, pairs where they were found
    const bool direct = plain_of(MODE) && p.leaf_scan != 0;
    bool counted = false;   // this lane's partial match is a leaf parent, done here
    if constexpr (plain_of(MODE) && L > 1) {
        if (direct) {
            const uint32_t x = base + lane;
            const bool act = (uint32_t)lane < nA;
            uint4 nw = make_uint4(0, 0, 0, 0);
            if (act) nw = inode[A.node[x]];
            counted = (nw.z & kLeafParent) != 0;
            if (__ballot(counted)) {
                int32_t ph[SA];
                uint32_t eid = 0, eid2 = 0, live = 0;
                TT tp = 0, tf = 0;
#pragma unroll
                for (int t = 0; t < SA; ++t) ph[t] = counted ? vtx(t, x) : -1;
                if (counted) {
                    eid = A.eid[x];
                    tp = glb(p.g.gt)[eid];
                    tf = tfirst_of(x);
                    live = A.live[x];
                    if constexpr (L == 3) eid2 = A.eid2[x];
                }
                count_leaf_parent<TT, D, MODE, L, SA>(p, W, cnt, lane, nw,
                                                      counted ? nw.w & live & kLiveLists : 0u, ph,
                                                      eid, eid2, tp, tf, live, nd);
            }
            if (!__ballot(act && !counted)) return;
        }
    }

    // (partial match, list) pairs: the node's lists that are live.  At the root
    // level they are written out, roots in order; deeper, the pairs per
    // partial match become an inclusive prefix.  Lists of motif vertices 0 and
    // 1 come first within a partial match.
    uint32_t P = 0, Pn = 0;
    uint4 node0 = make_uint4(0, 0, 0, 0);
    if constexpr (L == 1) {
        node0 = inode[0];
        if (ctx) {
            P = nA;   // a context is one window of its root
        } else {
            uint32_t act = 0;
            if ((uint32_t)lane < nA) {
                act = A.live[lane] & node0.y & 15u;
                if constexpr (STATS)
                    if (part == 0) st.v[kStatWinList] += (uint32_t)__popc(node0.y & 15u);
            }
            const uint32_t n = (uint32_t)__popc(act);
            const uint32_t incl = incl_scan32(n, lane);
            for (uint32_t at = incl - n; act; act &= act - 1)
                A.pair[at++] = (uint8_t)((uint32_t)lane | ((uint32_t)__builtin_ctz(act) << 6));
            Pn = lane_value(incl, kWave - 1);
            P = Pn + (((node0.y >> kLiveAllBit) & 1u) ? nA : 0u);
            wave_sync();
        }
    } else {
        uint32_t n = 0;
        if ((uint32_t)lane < nA && !counted) {
            const uint32_t lists = inode[A.node[base + lane]].y;
            n = (uint32_t)__popc(lists & A.live[base + lane] & kLiveLists);
            if constexpr (STATS)
                st.v[kStatWinList] += (uint32_t)__popc(lists & ~(1u << kLiveAllBit));
        }
        const uint32_t incl = incl_scan32(n, lane);
        A.pincl[lane] = (uint16_t)incl;
        P = lane_value(incl, kWave - 1);
        wave_sync();
    }

    // window chunk: lane w < nw holds non-empty window w
    //   wrec = {entry | group << 8, first list index, exclusive start, inclusive end}
    uint4 wrec = make_uint4(0, 0, 0, 0);
    uint32_t pc = 0, nw = 0, T = 0, cc = 0;
    uint32_t nB = 0;   // partial matches buffered at level L+1
    // epochs: root-level candidates are written out as contexts instead of
    // expanded once enough waves are idle (polled every 16 passes)
    bool dumping = false, room = true;
    uint32_t polls = 0, used = 0;   // contexts this wave wrote (at most its share of ctx_cap)

    bool done = false;
    for (;;) {
        if constexpr (MODE == 4) if (st.stopped) break;
        const KParams<TT> &p = fresh(p0);
        const uint4 *__restrict__ inode = glb(p.tree.inode);
        if constexpr (L == 1 && epochs_of(MODE)) {
            // (a wave dumps in one batch at most: the later batches of its
            // chunk search on)
            if (p.idle && p.ctx_out && room && !dumping && !st.stopped && (++polls & 15u) == 0) {
                uint32_t v = 0;
                if (lane == 0) v = __hip_atomic_load(p.idle, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                const uint32_t waves = gridDim.x * (blockDim.x / kWave);
                dumping = (uint64_t)lane_value(v, 0) * 100u >= (uint64_t)p.idle_pct * waves;
            }
        }
        bool formed = false;   // a new chunk of windows in this round
        if (cc >= T) {
            if (pc >= P) {
                done = true;
            } else {
                // one (partial match, group) pair per lane -> its window
                const uint32_t pi = pc + lane;
                uint32_t len = 0, x = 0, g = 0, l0 = 0, hdr = 0, bit = 0;
                bool all = false;
                if (pi < P) {
                    uint32_t lo = 0;
                    bool given = false;   // the window comes with a context
                    if constexpr (L == 1) {
                        if (ctx) {
                            const EpochCtx c = ctx[pi];
                            lo = pi;
                            bit = c.bit;
                            g = (node0.x & 0xfffffu) + (uint32_t)__popc(node0.y & ((1u << bit) - 1u));
                            l0 = c.e0;
                            len = c.e1 - c.e0;
                            given = true;
                        } else {
                            bit = kLiveAllBit;
                            if (pi < Pn) {
                                const uint32_t c = A.pair[pi];
                                lo = c & 63u;
                                bit = c >> 6;
                            } else {
                                lo = pi - Pn;
                            }
                            g = (node0.x & 0xfffffu) + (uint32_t)__popc(node0.y & ((1u << bit) - 1u));
                        }
                    } else {
                        uint32_t n = nA;
                        while (n > 0) {
                            const uint32_t h = n >> 1;
                            if (A.pincl[lo + h] <= pi) { lo += h + 1; n -= h + 1; }
                            else n = h;
                        }
                        const uint32_t before = lo ? A.pincl[lo - 1] : 0u;
                        lo += base;
                        const uint4 w = inode[A.node[lo]];
                        uint32_t m = w.y & A.live[lo] & kLiveLists;
                        for (uint32_t k = pi - before; k > 0; --k) m &= m - 1;
                        bit = (uint32_t)__builtin_ctz(m);
                        g = (w.x & 0xfffffu) + (uint32_t)__popc(w.y & ((1u << bit) - 1u));
                    }
                    x = lo;
                    hdr = glb((const uint32_t *)p.tree.grp)[12 * g];
                    if (given) {
                        all = (hdr & 15) == kDirAll;
                    } else {
                        const int dir = hdr & 15, anc = (hdr >> 4) & 15;
                        const TT thi = sat_add(tfirst_of(lo), p.delta_sat);
                        uint32_t b, e, sh;
                        const TT *ta;
                        bool hinted = false, known = false;
                        if (dir == kDirAll) {
                            b = 0; e = p.g.n_edges; ta = glb(p.g.gt); sh = 0;
                            all = true;
                            if constexpr (L > 1) {
                                // the whole-list window starts after the last edge
                                // itself (past the entries with its time)
                                b = A.eid[lo] + 1u;
                            }
                        } else {
                            ta = times_of(dir == kDirOut ? glb(p.g.out_adj) : glb(p.g.in_adj));
                            sh = kAdjShift<TT>;
                            const int32_t a = vtx((uint32_t)anc, lo);
                            const uint32_t *off = dir == kDirOut ? glb(p.g.out_off) : glb(p.g.in_off);
                            if (L > 1 && D > 2 && anc < 2) {
                                hinted = root_window(W, off, a, (uint32_t)anc * 2u + (uint32_t)dir,
                                                     L > 1 ? slot_of(lo) : 0u, b, e);
                            } else {
                                b = off[a];
                                e = off[a + 1];
                            }
                            if constexpr (L == 1) {
                                // the root edge's own entries: its windows start at
                                // the first entry after its time (set with the root)
                                l0 = W.hlo[(uint32_t)anc * 2u + (uint32_t)dir][lo];
                                known = true;
                            } else {
                                // an anchor on the last matched edge: the window
                                // starts where that edge's time ends in its list
                                const uint32_t le = (hdr >> 13) & 3u;
                                if (le) {
                                    const uint4 gx = glb(p.g.gx)[A.eid[lo]];
                                    l0 = le == 1 ? (dir == kDirOut ? gx.x : gx.y)
                                                 : (dir == kDirOut ? gx.z : gx.w);
                                    known = true;
                                }
                            }
                        }
                        if (!known) {
                            TT tp;
                            if constexpr (L == 1) tp = A.tfirst[lo];
                            else tp = glb(p.g.gt)[A.eid[lo]];
                            l0 = all && L > 1 ? gallop_greater(ta, sh, b, e, tp)
                                              : first_greater(ta, sh, b, e, tp);
                        }
                        len = (hinted ? e : gallop_greater(ta, sh, l0, e, thi)) - l0;
                        if constexpr (L == 1 && D > 2) {
                            if (!all && anc < 2) {
                                const uint32_t k = (uint32_t)anc * 2u + (uint32_t)dir;
                                // a long window keeps its end, the list's start
                                // then bounds the deeper bisections
                                const bool lng = len >= kLongHint;
                                W.hlo[k][lo] = lng ? l0 + len : l0;
                                W.hlen[k][lo] = lng ? kLongHint : (uint16_t)len;
                            }
                        }
                    }
                }
                // take the longest prefix of pairs whose candidates stay below 2^31
                // (always all of them when every window is under 2^25 entries;
                // 32-bit sums are exact unless some window has 2^26 entries)
                bool take = pi < P;
                if (__ballot(len >= (1u << 25))) {
                    const uint64_t incl64 = __ballot(len >= (1u << 26))
                                                ? incl_scan64((uint64_t)len, lane)
                                                : (uint64_t)incl_scan32(len, lane);
                    take = take && incl64 <= kChunkLimit;
                }
                pc += uniform((uint32_t)__popcll(__ballot(take)));
                const bool own = part == 0;   // this part keeps the per-window work
                if constexpr (STATS) {
                    // (windows of lists are counted with their partial match)
                    if (take && own) {
                        if (all) st.v[kStatWinAll] += 1;
                        st.v[all ? kStatEntAll : kStatEntList] += len;
                    }
                }
                if constexpr (LOG) {
                    if (take && own && len > 0)
                        atomicAdd(&p.root_cost[A.root[x]], (unsigned long long)len);
                }
                // a window whose children are all leaves is counted without
                // the candidate expansion: a short one by its own lane, a long
                // one by the whole wave
                const bool leaf = take && len > 0 && p.leaf_scan && ((hdr >> 12) & 1);
                const bool scanned = leaf && len <= p.leaf_scan;
                const bool coop = leaf && len > p.leaf_scan;
                const uint32_t nqm = leaf_compares<SA>(scanned && own, hdr);
                if (scanned && own) {
                    int32_t ph[SA];
#pragma unroll
                    for (int t = 0; t < SA; ++t) ph[t] = vtx(t, x);
                    const uint32_t c = count_leaf_window<TT, D, MODE>(p, g, hdr, ph, tfirst_of(x),
                                                                      l0, len, nqm, cnt, nd);
                    if constexpr (STATS) st.v[kStatCredit] += c;
                }
                for (uint64_t cm = __ballot(coop && own); cm; cm &= cm - 1) {
                    const int src = (int)__builtin_ctzll(cm);
                    const uint32_t wx = __builtin_amdgcn_readlane(x, src);
                    int32_t wph[SA];
#pragma unroll
                    for (int t = 0; t < SA; ++t) wph[t] = (int32_t)uniform((uint32_t)vtx(t, wx));
                    const uint32_t wg = __builtin_amdgcn_readlane(g, src);
                    const uint32_t wl0 = __builtin_amdgcn_readlane(l0, src);
                    const uint32_t wlen = __builtin_amdgcn_readlane(len, src);
                    uint32_t c;
                    if (nd == 1)
                        c = leaf_scan_wave<TT, SA>(p, wph, wg, wl0, wlen, lane, cnt, 1u, 0u);
                    else
                        c = leaf_scan_wave_multi<TT, SA>(p, wph, wg, wl0, wlen, tfirst_of(wx), lane,
                                                         cnt, nd);
                    if constexpr (STATS) st.v[kStatCredit] += c;
                }
                // compact the other non-empty windows into lanes 0..nw-1; their
                // candidate ranges are numbered without the leaf-counted ones
                // (the chunk total stays below the limit checked above)
                const bool keep = take && len > 0 && !leaf;
                const uint64_t km = __ballot(keep);
                nw = uniform((uint32_t)__popcll(km));
                wrec = make_uint4(0, 0, 0, 0);
                T = 0;
                if (nw) {
                    const uint32_t lk = keep ? len : 0u;
                    const uint32_t incl = incl_scan32(lk, lane);
                    // every lane sends its window to its place: the kept ones
                    // first, the others behind them
                    const int to = 4 * (int)(keep ? mbcnt(km) : nw + mbcnt(~km));
                    // (a root's list by its bit, a deeper window by its group)
                    wrec.x = (uint32_t)__builtin_amdgcn_ds_permute(to, (int)(x | ((L == 1 ? bit : g) << 8)));
                    wrec.y = (uint32_t)__builtin_amdgcn_ds_permute(to, (int)l0);
                    wrec.z = (uint32_t)__builtin_amdgcn_ds_permute(to, (int)(incl - lk));
                    wrec.w = (uint32_t)__builtin_amdgcn_ds_permute(to, (int)incl);
                    if ((uint32_t)lane >= nw) wrec = make_uint4(0, 0, 0, 0);
                    T = lane_value(wrec.w, nw - 1);
                }
                cc = 0;
                formed = true;
                if (L == 1 && nparts > 1) {
                    // one root, so every window fits this one chunk
                    cc = (uint32_t)(((uint64_t)T * part) / nparts);
                    T = (uint32_t)(((uint64_t)T * (part + 1)) / nparts);
                }
            }
        }
        if constexpr (L == 1 && plain_of(MODE) && (D > 2 || epochs_of(MODE))) if (epochs_of(MODE) || formed) {
            // Candidates [lo, T) of this chunk (in window order; lane w < nw
            // holds window w) as contexts of at most `piece` candidates, where
            // room(total) gives the first slot, or no slot (false) for all.
            auto hand_on = [&](uint32_t lo, uint32_t piece, auto room) -> bool {
                uint32_t c_lo = 0, c_hi = 0;
                if ((uint32_t)lane < nw) {
                    c_lo = max(lo, wrec.z);
                    c_hi = wrec.w;
                }
                const uint32_t n = c_hi > c_lo ? (c_hi - c_lo + piece - 1) / piece : 0u;
                const uint32_t incl = incl_scan32(n, lane);
                unsigned long long slot = 0;
                if (!room(lane_value(incl, kWave - 1), slot)) return false;
                if (n) {
                    const uint32_t ox = wrec.x & 255;
                    const uint64_t tf = (uint64_t)tfirst_of(ox);
                    EpochCtx c;
                    c.a = vtx(0, ox);
                    c.b = vtx(1, ox);
                    c.t_lo = (uint32_t)tf;
                    c.t_hi = (uint32_t)(tf >> 32);
                    c.bit = wrec.x >> 8;
                    c.root = A.root[ox];
#pragma unroll
                    for (int k = 0; k < 4; ++k) {
                        c.hlo[k] = W.hlo[k][ox];
                        c.hlen[k] = W.hlen[k][ox];
                    }
                    c.job = p.job;
                    c.pad2 = 0;
                    slot += incl - n;
                    for (uint32_t k = 0; k < n; ++k) {
                        const uint32_t c0 = c_lo + k * piece;
                        const uint32_t c1 = min(c0 + piece, c_hi);
                        c.e0 = wrec.y + (c0 - wrec.z);
                        c.e1 = wrec.y + (c1 - wrec.z);
                        p.ctx_out[slot + k] = c;
                    }
                }
                return true;
            };
            if constexpr (epochs_of(MODE)) {
                if (!done && cc < T && dumping) {
                    // every wave may write its share of the buffer, so one
                    // atomic add takes the slots and the buffer never overflows
                    const uint64_t share = p.ctx_cap / ((uint64_t)gridDim.x * (blockDim.x / kWave));
                    const bool ok = hand_on(cc, kCtxPiece, [&](uint32_t tot, unsigned long long &slot) {
                        if ((uint64_t)used + tot > share) return false;
                        if (lane == 0 && tot) slot = atomicAdd(p.ctx_count, (unsigned long long)tot);
                        slot = lane0_u64(slot);
                        used += tot;
                        return true;
                    });
                    if (ok) {
                        cc = T;
                    } else {
                        dumping = false;   // its share is used up: this wave searches on
                        room = false;
                    }
                }
            } else {
                // A chunk with far more candidates than most is a long chain
                // for one wave: what is beyond p.hand_on goes to the context
                // launch that follows, spread over the device.
                if (p.hand_on && nparts == 1 && T > p.hand_on + p.hand_on / 2) {
                    const bool ok = hand_on(p.hand_on, p.ctx_piece, [&](uint32_t tot, unsigned long long &slot) {
                        if (lane == 0) slot = atomicAdd(p.ctx_count, (unsigned long long)tot);
                        slot = lane0_u64(slot);
                        if (slot + tot <= p.ctx_cap) return true;
                        // the buffer is full: the slots taken that exist hold
                        // nothing (an empty range of this job's first root: the
                        // next launch looks up the root of every context), and
                        // this wave searches on
                        EpochCtx none{};
                        none.job = p.job;
                        for (unsigned long long k = slot + lane; k < p.ctx_cap; k += kWave) p.ctx_out[k] = none;
                        return false;
                    });
                    if (ok) T = p.hand_on;
                }
            }
        }
        if (!done && cc < T) {
            const KParams<TT> &p = fresh(p0);
            const uint4 *__restrict__ inode = glb(p.tree.inode);
            const uint32_t f = cc + lane;
            // owner window = number of windows that end at or before f
            const uint32_t o0 = (uint32_t)__popcll(__ballot((uint32_t)lane < nw && wrec.w <= cc));
            if ((uint32_t)lane < nw && wrec.w > cc && wrec.w - cc < (uint32_t)kWave)
                W.flag[wrec.w - cc] = 1;
            wave_sync();
            const uint32_t fl = W.flag[lane];
            W.flag[lane] = 0;
            const uint64_t ends = __ballot(fl != 0);
            wave_sync();
            const int oi = (int)((o0 + (uint32_t)__popcll(ends & le_mask)) & 63);
            const uint32_t oxg = __shfl(wrec.x, oi);
            const uint32_t olo = __shfl(wrec.y, oi);
            const uint32_t oex = __shfl(wrec.z, oi);
            const uint32_t oend = __shfl(wrec.w, oi);
            const bool valid = f < T;
            const uint32_t ox = oxg & 255;
            const uint32_t ei = olo + (f - oex);
            const uint32_t *__restrict__ gw = glb((const uint32_t *)p.tree.grp);   // group words

            uint32_t cw = 0;      // child word reached by this candidate
            TT tn = 0;            // its time
            uint32_t nx = 0, en_eid = 0;   // its next codes, its edge id (32-bit times)
            uint32_t dir = 0, anc = 0, g = 0;
            uint32_t nvp = 2, hit_s = 0;   // hit_s: motif vertex of the scanned endpoint
            int32_t nv0 = -1, nv1 = -1;
            int32_t ph[SA];
#pragma unroll
            for (int s = 0; s < SA; ++s) ph[s] = 0;
            if (valid) {
                if constexpr (L == 1) {
                    const uint32_t bit = oxg >> 8;
                    g = (node0.x & 0xfffffu) + (uint32_t)__popc(node0.y & ((1u << bit) - 1u));
                    dir = bit == kLiveAllBit ? (uint32_t)kDirAll : bit & 1u;
                    anc = bit == kLiveAllBit ? 0u : bit >> 1;
                } else {
                    g = oxg >> 8;
                    const uint32_t hdr = gw[12 * g];
                    dir = hdr & 15u;
                    anc = (hdr >> 4) & 15u;
                    nvp = (hdr >> 8) & 15u;
                }
#pragma unroll
                for (int s = 0; s < SA; ++s) ph[s] = vtx(s, ox);
                if (dir != kDirAll) {
                    const Entry<TT> *adj = dir == kDirOut ? glb(p.g.out_adj) : glb(p.g.in_adj);
                    const Entry<TT> en = adj[ei];   // one load: vertex, time, next codes
                    const int32_t v = en.v;
                    tn = en.t;
                    nx = en.nx;
                    if constexpr (sizeof(TT) == 4) en_eid = en.eid;
                    int y = -1;
#pragma unroll
                    for (int s = 0; s < SA; ++s) y = ((uint32_t)s < nvp && ph[s] == v) ? s : y;
                    // in-groups have no bound-target children, so their words are 0
                    cw = gw[12 * g + (y >= 0 ? 1u + (uint32_t)y : 7u)];
                    hit_s = y >= 0 ? (uint32_t)y : nvp;
                    nv0 = v;
                }
            }
            if (__ballot(valid && dir == kDirAll)) {
                if (valid && dir == kDirAll) {
                    const int32_t cs = glb(p.g.gsrc)[ei], cd = glb(p.g.gdst)[ei];
                    bool hit = cs == cd;
#pragma unroll
                    for (int s = 0; s < SA; ++s)
                        hit |= ((uint32_t)s < nvp && (ph[s] == cs || ph[s] == cd));
                    cw = hit ? 0u : gw[12 * g + 7];
                    nv0 = cs;
                    nv1 = cd;
                    tn = glb(p.g.gt)[ei];
                }
            }
            if (cw) {
                const uint32_t q1 = (cw >> 16) & 0x7fffu;
                if (q1) {
                    const uint32_t j = nd > 1 ? window_slot(p, nd, tfirst_of(ox), tn) : 0u;
                    atomicAdd(&cnt[(q1 - 1) * nd + j], 1ull);
                }
                if constexpr (STATS) st.v[kStatCredit] += 1;
            }
            // the edge id of this candidate (pushed along, and written out
            // when enumerating), read only where it is used
            auto cand_eid = [&]() -> uint32_t {
                if (dir == kDirAll) return ei;
                if constexpr (sizeof(TT) == 4) return en_eid;
                else return (dir == kDirOut ? glb(p.g.out_eid) : glb(p.g.in_eid))[ei];
            };
            if constexpr (MODE == 4) {
                const uint32_t q1 = (cw >> 16) & 0x7fffu;
                uint32_t e[kKMax] = {0, 0, 0, 0, 0};
                edge_chain<L>(W, ox, e);
                e[L] = valid ? cand_eid() : 0u;
                st.stopped |= write_matches<TT, D>(p, W, lane, valid && cw && q1, q1 - 1u, e, L + 1);
            }
            if constexpr (L + 1 < D) {
                auto &B = lvl<L + 1>(W.lv);
                constexpr int SB = vslots(D, L + 1);
                bool push = (cw >> 31) != 0;
                // the child's live word: the scanned endpoint's lists and the
                // new edge's pair as their next entries' times say, the list
                // just scanned dead after its last entry, the rest inherited
                uint32_t live = 0;
                if (push) {
                    if constexpr (L == 1) live = root_bits(A.live[ox]) | (1u << kLiveAllBit) | (ox << kLiveSlot);
                    else live = A.live[ox];
                    if (dir == kDirAll) {
                        live |= (15u << (2 * nvp)) | (3u << (kLivePair + 2 * L));
                    } else {
                        const TT tf = tfirst_of(ox), thi = sat_add(tf, p.delta_sat);
                        const uint32_t q = next_code((TT)(thi - tn)), since = next_code((TT)(tn - tf));
#pragma unroll
                        for (int k = 0; k < R1.Q; ++k)   // past the last edge of the root's pair
                            if (since > R1.last[k][L == 1 ? ox : live >> kLiveSlot]) live &= ~(1u << (kLivePair + k));
                        live &= ~(3u << (2 * hit_s));
                        live |= (((nx >> 16) & 255u) <= q ? 1u : 0u) << (2 * hit_s);
                        live |= ((nx >> 24) <= q ? 2u : 0u) << (2 * hit_s);
                        live |= ((nx & 255u) <= q ? 1u : 0u) << (kLivePair + 2 * L);
                        live |= (((nx >> 8) & 255u) <= q ? 2u : 0u) << (kLivePair + 2 * L);
                        if ((L > 1 || !ctx) && f + 1 == oend) live &= ~(1u << (2 * anc + dir));
                    }
                    // nothing below it: not kept (the statistics count it)
                    const uint2 nw = reinterpret_cast<const uint2 *>(inode)[2 * (cw & 0xffffu) + 1];   // z, w
                    if constexpr (LOG) push = (live & inode[cw & 0xffffu].y) != 0;
                    else if constexpr (!STATS) push = (live & nw.x & ~kLeafParent) != 0;
                    // a leaf parent's pairs are counted here, on the full
                    // lanes of the candidate pass; only one with windows left
                    // to look at (2 % of them on a bursty graph) is kept
                    if constexpr (plain_of(MODE)) {
                        if (direct && push && (nw.x & kLeafParent)) {
                            auto pair_of = [&](uint32_t k) -> uint2 {
                                const uint32_t j = k >> 1;
                                uint32_t e = ei;   // record (DevGraph::gp)
                                if (j == (uint32_t)L) {
                                    // (without records per entry the edge id is
                                    // read once more: kept for this it would
                                    // take registers from every search)
                                    if (p.g.gp_out)
                                        e += dir == kDirOut ? p.g.gp_out : dir == kDirIn ? p.g.gp_in : 0u;
                                    else if (dir != kDirAll)
                                        e = sizeof(TT) == 4
                                                ? reinterpret_cast<const uint32_t *>(
                                                      dir == kDirOut ? glb(p.g.out_adj) : glb(p.g.in_adj))[4 * (size_t)ei + 3]
                                                : (dir == kDirOut ? glb(p.g.out_eid) : glb(p.g.in_eid))[ei];
                                } else if constexpr (L == 1) {
                                    e = A.root[ox];
                                } else {
                                    if (j == 0) e = R1.root[A.live[ox] >> kLiveSlot];
                                    else e = A.eid[ox];
                                    if constexpr (L == 3) e = j == 1 ? A.eid2[ox] : e;
                                }
                                return reinterpret_cast<const uint2 *>(glb(p.g.gp))[2 * (size_t)e + (k & 1u)];
                            };
                            const TT tf = tfirst_of(ox);
                            count_pairs<TT, MODE>(p, cnt, (live >> kLivePair) & (nw.y >> 16) & 255u,
                                                  glb(p.tree.pairs) + 8 * (cw & 0xffffu), (nw.y >> 24) & 1u, pair_of, tn, tf,
                                                  sat_add(tf, p.delta_sat), nd);
                            push = (nw.y & live & kLiveLists) != 0;
                        }
                    }
                }
                const uint64_t pm = __ballot(push);
                if (push) {
                    const uint32_t slot = nB + mbcnt(pm);
#pragma unroll
                    for (int s = 2; s < SB; ++s) {
                        int32_t v = (s < SA) ? ph[s < SA ? s : 0] : -1;
                        v = ((uint32_t)s < nvp) ? v
                            : ((uint32_t)s == nvp ? nv0 : ((uint32_t)s == nvp + 1 ? nv1 : -1));
                        B.phi[s - 2][slot] = v;
                    }
                    B.eid[slot] = cand_eid();
                    B.node[slot] = (uint16_t)(cw & 0xffffu);
                    B.live[slot] = live;
                    if constexpr (L == 2) B.eid2[slot] = A.eid[ox];
                    if constexpr (keep_of(MODE) > 0) B.root[slot] = A.root[ox];
                    if constexpr (keep_of(MODE) == 2 && L > 1) B.par[slot] = (uint8_t)ox;
                    if constexpr (STATS) st.v[kStatPush] += 1;
                }
                nB += (uint32_t)__popcll(pm);
            }
            cc += kWave;
        }
        if constexpr (L + 1 < D) {
            // 64 of them at a time, the last ones first (the others stay where
            // they are), so that every batch but the last is full
            if (nB >= kWave || (done && nB > 0)) {
                const uint32_t n = min(nB, (uint32_t)kWave);
                nB -= n;
                wave_sync();
                run_level<TT, D, MODE, L + 1>(p0, W, cnt, lane, nB, n, st);
                wave_sync();
            }
        }
        if (done && nB == 0) break;
    }
    if constexpr (L == 1) {
        if (dumping) st.stopped = true;
    }
}

// A piece of work: roots [pos, end) of the root list (positions, or edge ids
// when p.roots is NULL); with nparts > 1 part `part` of the search from the one
// root `pos`; with ctx contexts [pos, end) of p.ctx_in (at most 64).
struct Piece {
    uint32_t pos, end, part, nparts;
    bool ctx;
};

// Searches the pieces that claim() hands out until it returns false, up to 64
// roots at a time.  Roots with nothing live in their windows take no place in
// the batch.  (Filling the batch across pieces measured no different.)
template <typename TT, int D, int MODE, typename Claim>
__device__ __forceinline__ void search_pieces(const KParams<TT> &p,
                                              WaveLds<TT, D, keep_of(MODE)> &W,
                                              unsigned long long *cnt, const int lane,
                                              Claim claim, Stats &st) {
    constexpr bool STATS = MODE == 1, LOG = MODE == 2;
    Piece w{0, 0, 0, 1, false};
    while (claim(w)) {
        while (w.pos < w.end) {
            uint32_t n1 = 0;   // roots in the level-1 batch
            const EpochCtx *ctx = nullptr;
            if (epochs_of(MODE) && w.ctx) {
                // each context becomes a root of the batch with its window
                // and its root windows given
                if constexpr (D > 1) {
                    auto &A = lvl<1>(W.lv);
                    const uint32_t i = w.pos + (uint32_t)lane;
                    if (i < w.end) {
                        const EpochCtx c = p.ctx_in[i];
                        const TT t = (TT)(((uint64_t)c.t_hi << 32) | c.t_lo);
                        A.phi[0][lane] = c.a;
                        A.phi[1][lane] = c.b;
                        A.tfirst[lane] = t;
                        A.root[lane] = c.root;
                        A.live[lane] = (uint8_t)set_pair_ends(p, A, (uint32_t)lane, c.root, t, root_live(p, c.root));
#pragma unroll
                        for (int k = 0; k < 4; ++k) {
                            W.hlo[k][lane] = c.hlo[k];
                            W.hlen[k][lane] = c.hlen[k];
                        }
                    }
                    ctx = p.ctx_in + w.pos;
                    n1 = w.end - w.pos;
                }
                w.pos = w.end;
            } else {
                const uint32_t i = w.pos + (uint32_t)lane;
                bool ok = i < w.end;
                uint32_t r = 0;
                int32_t s = 0, d = 0;
                if (ok) {
                    r = p.roots ? p.roots[i] : i;
                    s = glb(p.g.gsrc)[r];
                    d = glb(p.g.gdst)[r];
                    ok = s != d;
                }
                uint32_t live = 0;
                TT t = 0;
                bool keep = D > 1 && ok;
                if constexpr (D > 1) {
                    if (ok) {
                        t = glb(p.g.gt)[r];
                        live = root_live(p, r);
                        // a root with nothing in its windows ends here (the
                        // statistics still count its empty windows)
                        if constexpr (!STATS)
                            keep = ((root_bits(live) | (1u << kLiveAllBit)) &
                                    (LOG ? glb(p.tree.inode)[0].y : glb(p.tree.inode)[0].z)) != 0;
                    }
                }
                if (w.part == 0) {
                    const uint64_t all = __ballot(ok);
                    if (p.tree.root_q >= 0 && lane == 0 && all)
                        atomicAdd(&cnt[p.tree.root_q * p.tree.n_d], (unsigned long long)__popcll(all));
                    if constexpr (MODE == 4) {
                        if (p.tree.root_q >= 0) {
                            uint32_t e[kKMax] = {r, 0, 0, 0, 0};
                            st.stopped |= write_matches<TT, D>(p, W, lane, ok, (uint32_t)p.tree.root_q, e, 1);
                        }
                    }
                    if constexpr (STATS) st.v[kStatRoots] += ok ? 1 : 0;
                    if constexpr (LOG) {
                        if (ok) atomicAdd(&p.root_cost[r], 1ull);
                    }
                }
                if constexpr (D > 1) {
                    auto &A = lvl<1>(W.lv);
                    const uint64_t km = __ballot(keep);
                    if (keep) {
                        const uint32_t slot = mbcnt(km);
                        A.phi[0][slot] = s;
                        A.phi[1][slot] = d;
                        A.tfirst[slot] = t;
                        set_root_slot(W, slot, glb(p.g.gx)[r]);
                        A.root[slot] = r;
                        A.live[slot] = (uint8_t)set_pair_ends(p, A, slot, r, t, live);
                    }
                    n1 = uniform((uint32_t)__popcll(km));
                }
                w.pos += kWave;
            }
            if constexpr (D > 1) {
                if (n1 > 0) {
                    wave_sync();
                    run_level<TT, D, MODE, 1>(p, W, cnt, lane, 0u, n1, st, w.part, w.nparts, ctx);
                    wave_sync();
                }
            }
        }
    }
}

// Up to depth 3 the plain search (MODE 0) fits 8 waves per SIMD (at most 64
// VGPRs and 96 SGPRs) without spilling in its loops, and the multi-window
// search (MODE 3) is faster there with a few spills than at 6 waves; the
// compiler is asked for that.  Deeper trees and the instrumented modes keep
// the compiler's own allocation.
template <int D, int MODE>
constexpr int min_waves_per_eu() { return D <= 3 && plain_of(MODE) ? 8 : 1; }

template <typename TT, int D, int MODE>
__global__ void __launch_bounds__(kWave * kMaxWavesPerBlock)
__attribute__((amdgpu_waves_per_eu(min_waves_per_eu<D, MODE>(), 8)))
comine_kernel(const KParams<TT>) {
    const KParams<TT> &p = *(const KParams<TT> *)(ConstParams<TT>)__builtin_amdgcn_kernarg_segment_ptr();
    constexpr bool STATS = MODE == 1;
    extern __shared__ __align__(16) unsigned char smem[];
    const uint32_t wpb = blockDim.x / kWave;
    unsigned long long *cnt = reinterpret_cast<unsigned long long *>(smem);
    const int32_t n_slots = counter_slots(p.tree);
    const size_t cnt_bytes = ((size_t)n_slots * 8 + 15) & ~(size_t)15;
    const int lane = (int)(threadIdx.x & (kWave - 1));
    const int wave = (int)uniform(threadIdx.x / kWave);
    WaveLds<TT, D, keep_of(MODE)> &W = reinterpret_cast<WaveLds<TT, D, keep_of(MODE)> *>(smem + cnt_bytes)[wave];

    __shared__ uint32_t runs_taken;   // context launch: runs this workgroup took
    if (threadIdx.x == 0) runs_taken = 0;
    for (int i = (int)threadIdx.x; i < n_slots; i += (int)blockDim.x) cnt[i] = 0;
    W.flag[lane] = 0;
    if constexpr (MODE == 4) {
        if (lane == 0) W.n = 0;
    }
    __syncthreads();
    Stats st;
#pragma unroll
    for (int i = 0; i < kStats; ++i) st.v[i] = 0;
    st.stopped = false;
    // when each wave starts and ends its search (device real-time clock)
    const uint32_t clock_slot = blockIdx.x * wpb + (uint32_t)wave;
    if (p.wave_clock && lane == 0 && clock_slot < p.n_wave_clock)
        p.wave_clock[2 * clock_slot] = __builtin_amdgcn_s_memrealtime();

    // Scheduled work items first, claimed in order from their own queue; in a
    // later epoch the contexts the last one left, spread over every wave (up to
    // 64 at a time); else the root queues.  Workgroups are dispatched to the
    // XCDs round-robin: a wave starts on its XCD's share of the roots, then
    // takes what is left of the others.  A chunk once claimed is always searched
    // to the end, so after a stop the queue heads (clamped to the queue lengths)
    // mark exactly the roots searched.
    bool items = p.items != nullptr;
    const uint32_t nq = p.n_queues;
    const uint32_t home = blockIdx.x % nq;
    uint32_t qi = 0, ii = 0;
    // The wave's first chunk is its own place in its home queue; claims start
    // behind those (claims on one head take about 20 ns each, one after
    // another: 62,500 chunks of 16 roots were 150 us of a count).  Not where the
    // heads are a resume point or waves may leave early.
    bool first = p.place_first != 0;
    const uint32_t place = (blockIdx.x / nq) * wpb + (uint32_t)wave;
    auto claim = [&](Piece &w) -> bool {
        if (st.stopped) return false;
        if (items) {
            // item i waits in queue i % kQueues, so that the claims of the
            // whole device are not one after another on one head
            const uint32_t n_items = uniform(*p.n_items);
            uint32_t it = n_items;
            for (; ii < (uint32_t)kQueues; ++ii) {
                const uint32_t q = (blockIdx.x + ii) % (uint32_t)kQueues;
                const uint32_t nq_items = (n_items + (uint32_t)kQueues - 1u - q) / (uint32_t)kQueues;
                uint32_t *head = reinterpret_cast<uint32_t *>(&p.queues[q * kQueueStride + kItemWord]);
                uint32_t k = nq_items;
                if (lane == 0) {
                    const uint32_t h = ii ? __hip_atomic_load(head, __ATOMIC_RELAXED,
                                                              __HIP_MEMORY_SCOPE_AGENT) : 0u;
                    if (h < nq_items) k = atomicAdd(head, 1u);
                }
                k = lane_value(k, 0);
                if (k < nq_items) {
                    it = k * (uint32_t)kQueues + q;
                    break;
                }
            }
            if (it < n_items) {
                const uint2 item = p.items[it];
                const uint32_t ix = uniform(item.x), iy = uniform(item.y);
                const bool split = (iy & kItemSplit) != 0;
                w = {ix, split ? ix + 1 : iy, split ? (iy >> 15) & 0x7fffu : 0u,
                     split ? iy & 0x7fffu : 1u, false};
                return true;
            }
            items = false;
        }
        if constexpr (epochs_of(MODE)) {
            if (p.ctx_in && p.ctx_n) {
                // contexts handed on by the launch before: runs of them, one
                // XCD's share in a row (close in time, they read the same
                // lists), dealt to its workgroups in turn and taken by the
                // workgroup's next free wave
                const uint32_t n = (uint32_t)min(*glb(p.ctx_n), p.ctx_cap);
                const uint32_t waves = gridDim.x * wpb;
                const uint32_t per = max(1u, min(16u, n / (4u * waves)));
                const uint32_t runs = (n + per - 1) / per, xcds = min(8u, gridDim.x);
                const uint32_t x = blockIdx.x % xcds;
                const uint32_t r0 = (uint32_t)((uint64_t)runs * x / xcds);
                const uint32_t r1 = (uint32_t)((uint64_t)runs * (x + 1) / xcds);
                uint32_t k = 0;
                if (lane == 0) k = atomicAdd(&runs_taken, 1u);
                k = lane_value(k, 0);
                const uint32_t groups = (gridDim.x - x + xcds - 1) / xcds;
                const uint64_t r = (uint64_t)r0 + blockIdx.x / xcds + (uint64_t)k * groups;
                if (r >= r1) return false;
                const uint32_t b0 = (uint32_t)r * per;
                w = {b0, (uint32_t)min(b0 + per, n), 0u, 1u, true};
                return true;
            }
            if (p.ctx_in) {
                const uint32_t waves = gridDim.x * wpb;
                const uint32_t per = min((uint32_t)kWave, max(1u, (p.n_ctx_in + waves - 1) / waves));
                unsigned long long it = 0;
                if (lane == 0) it = atomicAdd(&p.queues[kItemSlot * kQueueStride], (unsigned long long)per);
                it = lane0_u64(it);
                if (it >= p.n_ctx_in) return false;
                const uint32_t b0 = uniform((uint32_t)it);
                w = {b0, (uint32_t)min(b0 + per, p.n_ctx_in), 0u, 1u, true};
                return true;
            }
        }
        while (qi < nq) {
            const uint32_t q = (home + qi) % nq;
            const uint32_t qbeg = queue_begin(p.n_roots, nq, q);
            const uint32_t qlen = queue_end(p.n_roots, nq, q) - qbeg;
            // chunks of this queue that are some wave's first
            const uint32_t taken = p.place_first ? min(qlen, ((gridDim.x - q + nq - 1) / nq) * wpb * p.chunk) : 0u;
            uint32_t got = qlen;
            if (first) {
                first = false;
                got = min(qlen, place * p.chunk);
                if (got == qlen) continue;
            } else if (taken < qlen) {   // (else nothing is left to claim)
                // Another XCD's queue is looked at before it is claimed from:
                // the failing last claims of 8,192 waves on eight heads were
                // 115 us at the end of every count.  A budget is spent only on a
                // queue that still has roots, so a call makes progress while any
                // root is left: a budget holder's claim fails only when another
                // holder took the last chunk.  A head counts past its queue's
                // end, by one chunk per failing claim: 64 bits, for a caller's
                // 65,536-root chunks on many workgroups pass 2^32.
                unsigned long long *head = &p.queues[q * kQueueStride];
                if (lane == 0) {
                    const bool look = p.max_chunks || qi > 0;
                    const unsigned long long h = look ? __hip_atomic_load(head, __ATOMIC_RELAXED,
                                                                          __HIP_MEMORY_SCOPE_AGENT) : 0ull;
                    if (p.stop && __hip_atomic_load(p.stop, __ATOMIC_RELAXED,
                                                    __HIP_MEMORY_SCOPE_SYSTEM) != 0)
                        got = ~0u;
                    else if (h >= qlen - taken)
                        got = qlen;
                    else if (p.max_chunks &&
                             atomicAdd(&p.queues[kBudgetSlot * kQueueStride], 1ull) >= p.max_chunks)
                        got = ~0u;
                    else
                        got = (uint32_t)min((unsigned long long)qlen,
                                            atomicAdd(head, (unsigned long long)p.chunk) + taken);
                }
                got = lane_value(got, 0);
            }
            if (got == ~0u) {
                qi = nq;
                break;
            }
            if (got >= qlen) {
                ++qi;
                continue;
            }
            const uint32_t b0 = qbeg + got;
            if (p.skip && p.skip[b0 / kWave]) continue;   // searched as an item
            w = {b0, qbeg + (uint32_t)min(got + p.chunk, qlen), 0u, 1u, false};
            return true;
        }
        return false;
    };
    search_pieces<TT, D, MODE>(p, W, cnt, lane, claim, st);
    if constexpr (MODE == 4) flush_matches<TT, D>(p, W, lane);
    if constexpr (epochs_of(MODE)) {
        // out of work: an idle wave, for the epoch limit
        if (p.idle && p.ctx_out && !st.stopped && lane == 0) atomicAdd(p.idle, 1u);
    }

    if (p.wave_clock && lane == 0 && clock_slot < p.n_wave_clock)
        p.wave_clock[2 * clock_slot + 1] = __builtin_amdgcn_s_memrealtime();
    if constexpr (STATS) {
#pragma unroll
        for (int i = 0; i < kStats; ++i)
            if (st.v[i]) atomicAdd(&p.stats[i], (unsigned long long)st.v[i]);
    }
    __syncthreads();
    if (p.part) {
        for (int i = (int)threadIdx.x; i < n_slots; i += (int)blockDim.x)
            p.part[(size_t)blockIdx.x * n_slots + i] = cnt[i];
        return;
    }
    for (int i = (int)threadIdx.x; i < n_slots; i += (int)blockDim.x)
        if (cnt[i]) atomicAdd(&p.counts[i], cnt[i]);
}

// Many (graph, tree) jobs in one persistent launch.  Waves claim work items
// (root ranges of one job) from one queue per XCD; each wave keeps its own LDS
// counters, sized for the largest tree, and flushes them after every item.
template <typename TT, int D, int MODE>
__global__ void __launch_bounds__(kWave * kWavesPerBlock)
__attribute__((amdgpu_waves_per_eu(min_waves_per_eu<D, MODE>(), 8)))
batch_kernel(const BatchParams<TT> bp) {
    extern __shared__ __align__(16) unsigned char smem[];
    const int lane = (int)(threadIdx.x & (kWave - 1));
    const int wave = (int)uniform(threadIdx.x / kWave);
    const size_t cnt_bytes = ((size_t)bp.n_q_max * 8 + 15) & ~(size_t)15;
    unsigned char *mine = smem + (size_t)wave * (cnt_bytes + sizeof(WaveLds<TT, D, 0>));
    unsigned long long *cnt = reinterpret_cast<unsigned long long *>(mine);
    WaveLds<TT, D, 0> &W = *reinterpret_cast<WaveLds<TT, D, 0> *>(mine + cnt_bytes);
    W.flag[lane] = 0;
    Stats st;
    st.stopped = false;
    // search pieces of one job and add its counters to the batch's
    auto search = [&](uint32_t j, auto claim) {
        const BatchJob<TT> &job = bp.jobs[j];
        const KParams<TT> &p = *(const KParams<TT> *)(ConstParams<TT>)&job.p;
        const uint32_t nq = (uint32_t)counter_slots(p.tree);
        for (uint32_t i = (uint32_t)lane; i < nq; i += kWave) cnt[i] = 0;
        wave_sync();
        search_pieces<TT, D, MODE>(p, W, cnt, lane, claim, st);
        wave_sync();
        for (uint32_t i = (uint32_t)lane; i < nq; i += kWave)
            if (cnt[i]) atomicAdd(&bp.counts[job.count_off + i], cnt[i]);
        wave_sync();
    };
    if constexpr (epochs_of(MODE)) {
        // the contexts handed on, dealt to the waves: a context and the ones
        // that follow it in the same job
        const uint32_t n = (uint32_t)min(*glb(bp.ctx_n), bp.ctx_cap);
        const uint32_t wpb = blockDim.x / kWave, waves = gridDim.x * wpb;
        const uint32_t per = max(1u, min(8u, n / (4u * waves)));
        const uint32_t w0 = blockIdx.x * wpb + (uint32_t)wave;
        for (uint32_t r = w0; (uint64_t)r * per < n; r += waves) {
            uint32_t at = r * per;
            const uint32_t end = min(at + per, n);
            while (at < end) {
                const uint32_t j = uniform(glb(bp.ctx)[at].job);
                uint32_t stop = at + 1;
                while (stop < end && uniform(glb(bp.ctx)[stop].job) == j) ++stop;
                bool fresh = true;
                search(j, [&](Piece &w) -> bool {
                    w = {at, stop, 0u, 1u, true};
                    const bool got = fresh;
                    fresh = false;
                    return got;
                });
                at = stop;
            }
        }
    } else {
        // one queue of items per XCD (claims on one head come one after another),
        // then what is left of the others, looked at before it is claimed from
        uint32_t qi = 0;
        while (qi < (uint32_t)kQueues) {
            const uint32_t q = (blockIdx.x + qi) % (uint32_t)kQueues;
            const uint32_t ibeg = (uint32_t)((uint64_t)bp.n_items * q / kQueues);
            const uint32_t iend = (uint32_t)((uint64_t)bp.n_items * (q + 1) / kQueues);
            uint32_t it = iend;
            if (lane == 0) {
                uint32_t *head = reinterpret_cast<uint32_t *>(bp.cursor + q * kQueueStride);
                const uint32_t h =
                    qi ? __hip_atomic_load(head, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) : 0u;
                if (h < iend - ibeg) it = min(ibeg + atomicAdd(head, 1u), iend);
            }
            it = lane_value(it, 0);
            if (it >= iend) {
                ++qi;
                continue;
            }
            BatchItem item;
            if (bp.items) {
                item = bp.items[it];
            } else {
                const uint32_t c = it / bp.n_jobs;
                item.job = it - c * bp.n_jobs;
                item.begin = c * bp.run_roots;
                item.end = min(bp.n_roots - item.begin, bp.run_roots) + item.begin;
                item.part = 0;
            }
            const uint32_t ip = uniform(item.part);
            const bool split = (ip & kItemSplit) != 0;
            bool fresh = true;
            search(uniform(item.job), [&](Piece &w) -> bool {
                w = {uniform(item.begin), uniform(item.end), split ? (ip >> 15) & 0x7fffu : 0u,
                     split ? ip & 0x7fffu : 1u, false};
                const bool got = fresh && w.pos < w.end;
                fresh = false;
                return got;
            });
        }
    }
}


template <typename TT, int D, int MODE>
size_t smem_bytes(int n_q, int wpb) {
    return (((size_t)n_q * 8 + 15) & ~(size_t)15) +
           (size_t)wpb * sizeof(WaveLds<TT, D, keep_of(MODE)>);
}

// Shape of a launch that fills the device: waves per workgroup and workgroups.
// Four waves per workgroup, or eight where sharing one set of counters lets
// more waves onto a compute unit (756 motifs: 6 KB of counters, 16 waves
// instead of 12: 3M edges 5.07 -> 4.73 ms; 48 motifs and three windows on 4M
// edges 2.22 -> 2.07).  The last answer per kernel and thread is kept: asking costs
// more than the rest of a small launch.
constexpr size_t kLdsBytes = 160 * 1024;        // of a compute unit
constexpr size_t kMaxLds = kLdsBytes - 256;   // dynamic part of a workgroup's LDS at most
struct Fill {
    int dev = -1, n_q = -1, wpb = 4, blocks = 0;
};
template <typename TT, int D, int MODE>
hipError_t fill_shape(int n_q, Fill &f) {
    static thread_local Fill last;
    int dev = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return e;
    if (last.dev != dev || last.n_q != n_q) {
        auto kern = comine_kernel<TT, D, MODE>;
        int ncu = 0, most = 0;
        e = hipDeviceGetAttribute(&ncu, hipDeviceAttributeMultiprocessorCount, dev);
        if (e != hipSuccess) return e;
        Fill n{dev, n_q, kWavesPerBlock, ncu};
        for (int wpb = kWavesPerBlock; wpb <= kMaxWavesPerBlock; wpb *= 2) {
            const size_t sm = smem_bytes<TT, D, MODE>(n_q, wpb);
            if (sm > kMaxLds) break;
            if (sm > 65536) {
                e = hipFuncSetAttribute((const void *)kern, hipFuncAttributeMaxDynamicSharedMemorySize,
                                        (int)kMaxLds);   // (one value for every launch)
                if (e != hipSuccess) return e;
            }
            int per = 0;
            e = hipOccupancyMaxActiveBlocksPerMultiprocessor(&per, kern, kWave * wpb, sm);
            if (e != hipSuccess) return e;
            if (per * wpb > most) {
                most = per * wpb;
                n.wpb = wpb;
                n.blocks = ncu * per;
            }
        }
        last = n;
    }
    f = last;
    return hipSuccess;
}

template <typename TT, int D, int MODE>
hipError_t launch_ds(KParams<TT> p, int blocks, hipStream_t stream) {
    auto kern = comine_kernel<TT, D, MODE>;
    const int n_q = counter_slots(p.tree);
    int wpb = kWavesPerBlock;
    if (p.part && (blocks > 0 || p.chunk)) return hipErrorNotSupported;
    if (blocks > 0) {   // the caller's workgroups: four waves each
        if (smem_bytes<TT, D, MODE>(n_q, wpb) > 65536) {
            hipError_t e = hipFuncSetAttribute((const void *)kern,
                                               hipFuncAttributeMaxDynamicSharedMemorySize,
                                               (int)kMaxLds);
            if (e != hipSuccess) return e;
        }
    } else {
        Fill f;
        hipError_t e = fill_shape<TT, D, MODE>(n_q, f);
        if (e != hipSuccess) return e;
        blocks = f.blocks;
        wpb = f.wpb;
        if (p.chunk == 0) {
            // Few roots are spread thinner: a wave's 64 roots are one chain of
            // dependent loads, so a small graph takes as long as its slowest
            // chunk.  Up to 64 roots per wave every wave gets one chunk, of 4
            // roots at least, and there are no more workgroups than chunks
            // (20,000 edges: 150 -> 78 us a call); beyond that, chunks of
            // 64 (of 128: 3.11 ms for 20M edges, of 256: 3.22, against 3.08).
            const uint32_t waves = (uint32_t)(blocks * wpb);
            uint32_t c = 4;
            while (c < (uint32_t)kWave && (uint64_t)c * waves < p.n_roots) c <<= 1;
            p.chunk = c;
            // workgroups that give every chunk of the longest queue its wave
            uint32_t longest = 0;
            for (uint32_t q = 0; q < p.n_queues; ++q)
                longest = std::max(longest, queue_end(p.n_roots, p.n_queues, q) -
                                                queue_begin(p.n_roots, p.n_queues, q));
            const uint32_t need = (longest + c * wpb - 1) / (c * wpb) * p.n_queues;
            const bool one_each = !p.items && !p.ctx_in && need <= (uint32_t)blocks;
            if (one_each) blocks = (int)std::max(1u, need);
            if (p.part) {
                if (!one_each || (uint64_t)need * n_q > p.part_cap) return hipErrorNotSupported;
                *p.part_rows = need;
            }
            p.place_first = !p.items && !p.ctx_in;
        }
    }
    if (p.chunk == 0) p.chunk = kWave;
    if (p.hand_on) {
        p.hand_on = hand_on_limit(p.n_roots, (uint64_t)blocks * (uint32_t)wpb, D > 3);
        p.ctx_piece = hand_on_piece(D > 3);
    }
    const size_t sm = smem_bytes<TT, D, MODE>(n_q, wpb);
    hipLaunchKernelGGL(kern, dim3(blocks), dim3(kWave * wpb), sm, stream, p);
    return hipGetLastError();
}

}  // namespace

template <typename TT, int D>
hipError_t launch_d(const KParams<TT> &p, int blocks, hipStream_t stream) {
    if (p.ctx_in || (p.ctx_out && !p.hand_on))
        return p.tree.n_d > 1 ? launch_ds<TT, D, 6>(p, blocks, stream) : launch_ds<TT, D, 5>(p, blocks, stream);
    if (p.enum_out) return launch_ds<TT, D, 4>(p, blocks, stream);
    if (p.stats) return launch_ds<TT, D, 1>(p, blocks, stream);
    if (p.root_cost) return launch_ds<TT, D, 2>(p, blocks, stream);
    if (p.tree.n_d > 1) return launch_ds<TT, D, 3>(p, blocks, stream);
    return launch_ds<TT, D, 0>(p, blocks, stream);
}

template <typename TT, int D, int MODE>
hipError_t launch_batch_d(const BatchParams<TT> &bp, int blocks, hipStream_t stream) {
    if constexpr (!epochs_of(MODE))
        if (bp.contexts) return launch_batch_d<TT, D, MODE == 0 ? 5 : 6>(bp, blocks, stream);
    // Four waves per workgroup, or as many as fit: each has counters of its own
    // beside its level buffers (depth 5: 12.9 KB, so four up to 3,506 counters
    // and three up to 4,096).
    const size_t per_wave = (((size_t)bp.n_q_max * 8 + 15) & ~(size_t)15) + sizeof(WaveLds<TT, D, 0>);
    int wpb = kWavesPerBlock;
    while (wpb > 1 && wpb * per_wave > kLdsBytes) --wpb;
    const size_t sm = wpb * per_wave;
    auto kern = batch_kernel<TT, D, MODE>;
    if (sm > 65536) {
        hipError_t e = hipFuncSetAttribute((const void *)kern,
                                           hipFuncAttributeMaxDynamicSharedMemorySize, (int)sm);
        if (e != hipSuccess) return e;
    }
    if (blocks <= 0) {
        int dev = 0, ncu = 0, per = 0;
        hipError_t e = hipGetDevice(&dev);
        if (e != hipSuccess) return e;
        e = hipDeviceGetAttribute(&ncu, hipDeviceAttributeMultiprocessorCount, dev);
        if (e != hipSuccess) return e;
        e = hipOccupancyMaxActiveBlocksPerMultiprocessor(&per, kern, kWave * wpb, sm);
        if (e != hipSuccess) return e;
        blocks = ncu * (per > 0 ? per : 1);
        // (one graph's searches: no more waves than items)
        if (!bp.items && !bp.contexts)
            blocks = (int)std::min<uint32_t>((uint32_t)blocks, (bp.n_items + wpb - 1) / wpb);
    }
    hipLaunchKernelGGL(kern, dim3(blocks), dim3(kWave * wpb), sm, stream, bp);
    return hipGetLastError();
}

}  // namespace mg
