// Internal interface between the host code (host.cpp) and the HIP kernels
// (comine.hip).  Not part of the public C ABI.
#pragma once
#include <hip/hip_runtime_api.h>
#include <stdint.h>

namespace mg {

constexpr int kVMax = 6;        // motif vertices
constexpr int kKMax = 5;        // motif edges
constexpr int kWave = 64;
constexpr int kMaxDeltas = 8;   // windows counted in one search
constexpr int kWavesPerBlock = 4;      // 8 where more waves fit so (search.h, fill_shape)
constexpr int kMaxWavesPerBlock = 8;
constexpr int kQueues = 8;      // root queues, one per XCD
constexpr int kQueueStride = 16;  // u64 words between queue heads (own cache line)
// queue words: kQueues root-queue heads, the work-item queue head, the claim
// counter of a chunk budget, each kQueueStride words apart
constexpr int kItemSlot = kQueues;   // contexts of an epoch
constexpr int kItemWord = 8;         // in a root queue's line: head of its share of the items
constexpr int kBudgetSlot = kQueues + 1;
constexpr int kCtxCountWord = (kQueues + 1) * 16 + 8;   // in the budget's line: contexts handed on
constexpr int kQueueSlots = kQueues + 2;
constexpr int kQueueWords = kQueueSlots * kQueueStride;

// Root queue q of n_queues over n_roots roots holds positions [begin, end):
// boundaries on multiples of 64 roots, so that 64-root chunks are the
// scheduler's segments.  Host and device use this one definition.
__host__ __device__ inline uint32_t queue_begin(uint32_t n_roots, uint32_t n_queues, uint32_t q) {
    const uint64_t b = ((uint64_t)n_roots * q) / n_queues + 63;
    const uint32_t r = (uint32_t)(b & ~(uint64_t)63);
    return r < n_roots ? r : n_roots;
}
__host__ __device__ inline uint32_t queue_end(uint32_t n_roots, uint32_t n_queues, uint32_t q) {
    return q + 1 == n_queues ? n_roots : queue_begin(n_roots, n_queues, q + 1);
}
constexpr uint32_t kLeafScanDefault = 256;   // lane-counted leaf window limit

// A partial match's live word: bits 2 s + dir (s < 6: motif vertex, dir as
// below) are clear when the list of that vertex is known to hold no entry
// after the partial match and within its window; kLiveAll stands for the whole
// edge list and is always set; bits kLivePair + 2 j and + 1 are clear when no
// later edge within the window repeats matched edge j or runs against it; the
// root's slot in the level-1 batch sits above.
constexpr uint32_t kLiveAllBit = 12, kLivePair = 13, kLiveSlot = 21;
constexpr uint32_t kLiveLists = (1u << 13) - 1u;
constexpr uint32_t kLeafParent = 1u << 30;

// group direction: which adjacency list holds the candidates
enum : int { kDirOut = 0, kDirIn = 1, kDirAll = 2 };

// Search tables, as uploaded to the device.
//   inode[i]  internal (non-leaf) trie node i:
//     x = first group
//     y = its lists, as live-word bits (2 anchor + dir, kLiveAllBit): one group
//         per bit, in bit order
//     z = the live-word bits of which at least one has to be set for anything
//         to be found below the node when leaf windows are counted from pairs:
//         the lists of its other groups and the pairs of those that are; and
//         kLeafParent: every child a leaf reached through a list of a bound
//         vertex (all groups leaf_only)
//     w = of a leaf parent: the lists whose window has to be found (bits 0-12:
//         not counted from pairs, or with a new-vertex child) and the pairs
//         that are counted (bits 16-23: kLivePair's bits; bit 24: some for
//         new-vertex children too)
//   pairs[8 i + k]  of leaf parent i and pair k (matched edge k / 2, or against
//     it for odd k): x = child reached by an edge of the pair, y and z = the
//     new-vertex children of the out- and of the in-list that hold the pair,
//     for which such an edge does not count
//   grp[3g..3g+2]: twelve words of group g:
//     w0 = dir | anchor << 4 | nv << 8 | leaf_only << 12 | last_end << 13 |
//          bound_by << 15
//          (nv: vertices bound at the owning node; leaf_only: a per-vertex
//          list whose children all end a motif; last_end: the anchor is the
//          source (1) or destination (2) of the owning node's last edge, 0
//          otherwise; bound_by: the same for the node's second edge)
//     w1..w6 = child reached when the scanned endpoint is bound motif vertex 0..5
//     w7 = child reached when the scanned endpoint(s) are new vertices
//     w8 = 1 when the entries that reach bound vertices are counted from pairs:
//         every such vertex (all bound ones with a new-vertex child) is joined
//         to the anchor by a matched edge
//   A child word is 0 when there is no such child, else
//     internal index (bits 0-15, if internal) | (query + 1) << 16 | internal << 31.
// Counters: n_d per distinct motif, counter q * n_d + j holding the matches
// of motif q whose span (last time - first time) fits window j but not
// window j - 1 (windows ascending); the count at window j is the sum of
// slots 0..j.
struct DevTree {
    const uint4 *inode;
    const uint4 *pairs;
    const uint4 *grp;
    uint32_t root_pairs;   // bit 0, 1: some leaf parent counts the root's pair, the one against it
    int32_t n_q;        // distinct motifs
    int32_t root_q;     // query id of the one-edge prefix, -1 if none
    int32_t depth;      // longest motif in edges
    int32_t kdepth;     // kernel instantiation that searches it: depth, or 4
                        // for a depth-3 tree with a buffered two-edge prefix
                        // on four vertices (depth-3 kernels keep three)
    int32_t n_d;        // windows (1..kMaxDeltas), counter slots per motif
};
__host__ __device__ inline int32_t counter_slots(const DevTree &t) { return t.n_q * t.n_d; }

// One adjacency entry, 16 bytes read at once: the other endpoint, the edge time
// (both layouts: the TT-sized word 1 of the entry), next codes, and for 32-bit
// times the edge id (out_eid / in_eid hold it otherwise).  Next codes: four
// bytes, how long after the edge the next one comes in its pair, in the pair
// against it, in out() and in in() of the other endpoint (next_code below).
template <typename TT> struct Entry;
template <> struct alignas(16) Entry<uint32_t> { int32_t v; uint32_t t; uint32_t nx, eid; };
template <> struct alignas(16) Entry<uint64_t> { int32_t v; uint32_t nx; uint64_t t; };
// entry i's time is ((TT *)list)[(i << kAdjShift<TT>) + 1]
template <typename TT> constexpr uint32_t kAdjShift = sizeof(TT) == 4 ? 2 : 1;
template <typename TT> constexpr TT kNever = (TT)~(TT)0;   // past every edge time

template <typename TT>
struct DevGraph {
    const int32_t *gsrc, *gdst;   // time-sorted edge list (all edges)
    const TT *gt;
    const uint4 *gx;              // per edge u -> v at t: the first index with a later
                                  // time in out(u), in(u), out(v), in(v) (self-loops:
                                  // unused)
    const uint2 *gn;              // next codes of the edge: y = of those four lists, x = of
                                  // its pair (byte 0) and of the pair against it (byte 1)
    // Pairs: the edges ordered by (destination, source, time), so that the
    // edges u -> v are consecutive and ascending in time
    const TT *pair_t;             // their times
    const uint4 *gp;              // per edge u -> v at t: the first pair entry with a
                                  // later time and the end of the pair u -> v, then of
                                  // v -> u (self-loops: 0)
    uint32_t gp_out, gp_in;       // the same records once more per out_adj and in_adj entry:
                                  // where they start in gp (both 0: not kept, the
                                  // record is that of the entry's edge id)
    const uint32_t *out_eid;      // edge id of every out_adj entry (64-bit times)
    const uint32_t *in_eid;       // edge id of every in_adj entry (64-bit times)
    const uint32_t *out_off;      // V+1
    const Entry<TT> *out_adj;     // out-lists: destination, time
    const uint32_t *in_off;
    const Entry<TT> *in_adj;      // in-lists: source, time
    uint32_t n_edges;
};

// A piece of search left over when an epoch ends: the candidates of one
// root-level window, entries [e0, e1) of the list `bit` (live-word bit) of the
// root (edge id `root`) a -> b at time t_lo | t_hi << 32, with the root's windows in out(a), in(a),
// out(b), in(b) as far as it had found them (first entry and length, as the
// per-wave root windows keep them).  The root itself was credited when it was
// started.
struct EpochCtx {
    int32_t a, b;
    uint32_t t_lo, t_hi;
    uint32_t bit, e0, e1, root;
    uint32_t hlo[4];
    uint16_t hlen[4];
    uint32_t job, pad2;            // a batch's job
};
static_assert(sizeof(EpochCtx) == 64, "context record");
constexpr uint32_t kCtxPiece = 64;   // candidates per context at most

template <typename TT>
struct KParams {
    DevGraph<TT> g;
    DevTree tree;
    TT delta_sat;                 // the largest window, clamped to the TT range
    TT dlo[kMaxDeltas - 1];       // the smaller windows, ascending (tree.n_d - 1 of them)
    const uint32_t *roots;        // NULL: roots are 0..n_roots-1
    uint32_t n_roots;
    uint32_t chunk;               // roots per chunk (0: chosen at the launch by the number
                                  // of roots; multiple of 64 with items or skip)
    uint32_t n_queues;            // 1..kQueues root queues
    uint32_t place_first;         // 1: every wave's first chunk is its own place in its home
                                  // queue, and claims start behind those (set at the launch)
    unsigned long long *queues;   // kQueueWords: queue heads (zeroed, or a resume
                                  // point) and the claim counter (zeroed)
    const int32_t *stop;          // NULL, or a flag (host-pinned or device memory)
                                  // read before every chunk claim: non-zero = claim
                                  // no more chunks
    uint32_t max_chunks;          // 0, or the launch claims at most this many chunks
    unsigned long long *counts;   // counter_slots(tree), zeroed before launch
    // A small count (every chunk is some wave's first): each workgroup stores
    // its counters in a row of its own, in host memory (mapped, part_cap
    // counters), so nothing is cleared before the launch and nothing copied
    // after it.  launch_comine sets *part_rows to the rows, or returns
    // hipErrorNotSupported, without a launch, for a count that is not small.
    unsigned long long *part;
    uint32_t part_cap;
    uint32_t *part_rows;
    unsigned long long *stats;    // NULL, or kStats totals (zeroed before launch)
    unsigned long long *root_cost;  // NULL, or per root edge id: 1 + window entries
                                    // examined below that root (zeroed before launch)
    const uint2 *items;           // NULL, or work items searched before the queues:
                                  // {first, end} of root positions, or, with
                                  // kItemSplit set in .y, {root, kItemSplit |
                                  // part << 15 | nparts} (part < nparts < 2^15;
                                  // p.roots NULL): one part of one root's search
    const uint32_t *n_items;      // device count of items (with items)
    const uint8_t *skip;          // NULL, or per 64-root segment: 1 = covered by the
                                  // items (needs 64-root chunks and roots NULL)
    int32_t *enum_out;            // NULL, or enumeration: records of 1 + kKMax words
                                  // (distinct motif, edge ids, -1 past the motif's
                                  // length), enum_cap of them, at slots taken from
                                  // *enum_cursor (zeroed); once it is past enum_cap
                                  // the waves end their search, and neither it nor
                                  // the counters are the totals; needs leaf_scan 0
    unsigned long long *enum_cursor;
    unsigned long long enum_cap;
    unsigned long long *wave_clock;  // NULL, or per wave: start and end of its search
                                     // (device real-time clock ticks)
    uint32_t n_wave_clock;           // waves that wave_clock holds
    // epochs (the kernels' MODE 5 and 6, MODE 0 and 3 with epochs): ctx_out
    // and ctx_in NULL = off.  A wave that finds no work
    // left adds one to *idle; once *idle reaches idle_pct percent of the
    // launch's waves, the waves still searching stop expanding root-level
    // candidates, write what is left of their root-level windows as contexts,
    // finish what they already hold and exit.  The next launch searches the
    // contexts (ctx_in) instead of the root queues, claiming them through the
    // item slot of `queues`.
    EpochCtx *ctx_out;            // contexts written (ctx_cap at most; each wave at
                                  // most its share, ctx_cap / waves)
    unsigned long long *ctx_count;  // contexts written so far (zeroed)
    unsigned long long ctx_cap;
    uint32_t *idle;               // idle waves (zeroed)
    uint32_t idle_pct;            // the epoch ends once this percentage of the
                                  // launch's waves is idle (1..100)
    const EpochCtx *ctx_in;       // NULL, or the contexts this launch searches
    uint32_t n_ctx_in;
    // Heavy root-level chunks of the plain search (MODE 0 and 3): with hand_on
    // set (chosen at the launch by the number of roots), the candidates of a
    // chunk beyond that many are written as contexts of ctx_piece candidates
    // into ctx_out, and the launch that follows searches them (ctx_in, with
    // ctx_n their count on the device)
    uint32_t hand_on, ctx_piece;
    uint32_t job;                 // this search's job in a batch
    const unsigned long long *ctx_n;
    uint32_t leaf_scan;           // windows whose children are all leaves are counted
                                  // without the candidate expansion: by one lane up
                                  // to this long, by the whole wave when longer
                                  // (0: never)
};

constexpr uint32_t kItemSplit = 0x80000000u;

// search statistics (schedule independent), filled when KParams::stats is set
enum : int {
    kStatWinList = 0,   // windows on a per-vertex list
    kStatWinAll,        // windows on the whole time-ordered edge list
    kStatEntList,       // entries scanned in per-vertex windows
    kStatEntAll,        // entries scanned in whole-list windows
    kStatPush,          // partial matches buffered for a deeper level
    kStatCredit,        // trie nodes reached below the root (prefix matches)
    kStatRoots,         // roots searched (non-self-loop)
    kStats
};

// Root-level candidates of a chunk beyond which a search of n_roots roots over
// `waves` waves hands the rest on (a multiple of 64): about twice the candidates
// a wave's share of the roots has; deeper trees find far more below each.  Waves
// were busy 50 % of a launch over 2M edges, 49 % with 756 motifs over 3M, before
// chunks were handed on; 20M edges hand nothing on, and the empty second launch
// takes 6 us.
inline uint32_t hand_on_limit(uint64_t n_roots, uint64_t waves, bool deep) {
    const uint64_t share = n_roots / (waves > 0 ? waves : 1);
    const uint64_t n = deep ? (share < 1024 ? 256 : share < 8192 ? share / 4 : 2048)
                            : (share < 256 ? 512 : share < 4096 ? 2 * share : 8192);
    return (uint32_t)n & ~63u;
}
// candidates per context handed on
inline uint32_t hand_on_piece(bool deep) { return deep ? 64u : 256u; }

// Launch the persistent co-mining kernel.  `blocks` <= 0 fills the device.
// Returns a hipError_t value.
template <typename TT>
hipError_t launch_comine(const KParams<TT> &p, int blocks, hipStream_t stream);

// ---- batches: many (graph, tree) jobs in one launch
template <typename TT>
struct BatchJob {
    KParams<TT> p;                // the job's search (roots: every edge, in order)
    uint32_t count_off;           // first counter of this job in BatchParams::counts
};
struct BatchItem {
    uint32_t job, begin, end;   // roots [begin, end) of one job
    uint32_t part;              // 0, or kItemSplit | part << 15 | nparts: that part
                                // of the search from root `begin` (end = begin + 1)
};
template <typename TT>
struct BatchParams {
    const BatchJob<TT> *jobs;
    const BatchItem *items;       // NULL: the jobs are searches of one graph, and item i
                                  // is the chunk i / n_jobs of run_roots roots, of n_roots
                                  // in all, of job i % n_jobs
    uint32_t n_items;
    uint32_t n_jobs, run_roots, n_roots;   // with items NULL
    uint32_t n_q_max;             // largest tree's counter_slots
    unsigned long long *cursor;   // kQueues item queue heads, kQueueStride words apart,
                                  // zeroed before launch; queue q holds items
                                  // [n q / kQueues, n (q + 1) / kQueues)
    unsigned long long *counts;   // every job's counters, zeroed before launch
    uint32_t multi;               // 1 when some job's tree has several windows
    // contexts that the jobs' searches hand on (KParams::hand_on), searched by
    // a second launch when `contexts` is set
    const EpochCtx *ctx;
    const unsigned long long *ctx_n;
    unsigned long long ctx_cap;
    uint32_t contexts;
};

// `depth` = the deepest tree of the batch.
template <typename TT>
hipError_t launch_batch(const BatchParams<TT> &bp, int depth, int blocks, hipStream_t stream);

// The same for one tree depth D (search.h; instantiated in search_d<D>_t<bits>.hip).
// MODE 0 is the plain search, 3 the search of trees with several windows.
template <typename TT, int D>
hipError_t launch_d(const KParams<TT> &p, int blocks, hipStream_t stream);
template <typename TT, int D, int MODE>
hipError_t launch_batch_d(const BatchParams<TT> &bp, int blocks, hipStream_t stream);

// Device scratch of the count that allocates nothing: queue words, then
// kMaxQueries counters, then kStats statistics.  One array per device, held
// until the process ends; *ptr is its address on the current device.
constexpr int kMaxQueries = 4096;
constexpr size_t kStaticWords = (size_t)kQueueWords + kMaxQueries + 8;
hipError_t static_scratch(unsigned long long **ptr);

// p[0..n) = v with a kernel (safe to record into a captured graph)
hipError_t launch_fill_u64(unsigned long long *p, uint32_t n, unsigned long long v,
                           hipStream_t stream);

// Enumeration records (1 + kKMax words each: distinct motif, edge ids) into
// the caller's numbering: motif q becomes first[q], edge e becomes order[e]
// (order NULL: stays).  In place, or motifs to `motif` and edges to `edges`.
hipError_t launch_map_matches(int32_t *rec, uint64_t n, const int32_t *first,
                              const uint32_t *order, int32_t *motif, int32_t *edges,
                              hipStream_t stream);

}  // namespace mg
