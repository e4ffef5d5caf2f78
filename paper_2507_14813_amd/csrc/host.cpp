// Host side of the C ABI declared in include/mayura.h: graph ingest (queued on
// the device; on the host for host-only graphs), motif relabelling, MG-Tree /
// search-trie construction and flattening, and the count dispatch.
#include <hip/hip_runtime_api.h>

#include <algorithm>
#include <chrono>
#include <cmath>
#include <cstdarg>
#include <cstdio>
#include <cstring>
#include <map>
#include <memory>
#include <mutex>
#include <new>
#include <numeric>
#include <string>
#include <thread>
#include <vector>

#include "../../include/mayura.h"
#include "comine.h"
#include "handles.h"
#include "ingest.h"
#include "sched.h"

using mg::kVMax;
using mg::kKMax;
// the learned schedule predicts the cost of one root in this many per segment
constexpr uint32_t kSampleDefault = 1;
// most items one root's search is split into by the learned schedule
constexpr uint32_t kRootParts = 16;
// queue heads (root queues, work items, chunk budget)
constexpr size_t kQueueBytes = sizeof(unsigned long long) * mg::kQueueWords;
static_assert(MG_CURSOR_QUEUES == mg::kQueues, "cursor layout");
static_assert(MG_MAX_QUERIES == mg::kMaxQueries, "query limit");
static_assert(MG_MAX_DELTAS == mg::kMaxDeltas, "window limit");
static_assert(MG_NOALLOC_SCRATCH_BYTES == 8 * mg::kStaticWords, "static scratch size");

namespace mgh {

thread_local std::string g_err;

int fail(int code, const char *fmt, ...) {
    char buf[512];
    va_list ap;
    va_start(ap, fmt);
    vsnprintf(buf, sizeof buf, fmt, ap);
    va_end(ap);
    g_err = buf;
    return code;
}

#define HIP_TRY(expr)                                                              \
    do {                                                                           \
        hipError_t e_ = (expr);                                                    \
        if (e_ != hipSuccess)                                                      \
            return fail(MG_EDEVICE, "%s failed: %s", #expr, hipGetErrorString(e_)); \
    } while (0)

// ---------------------------------------------------------------- allocator
mg_alloc_fn g_alloc = nullptr;
mg_release_fn g_release = nullptr;
void *g_alloc_ctx = nullptr;

int dev_alloc(DevBuf &b, size_t bytes, void *stream) {
    b.bytes = bytes;
    b.stream = stream;
    if (bytes == 0) bytes = 16;
    if (g_alloc) {
        b.ptr = g_alloc(bytes, stream, g_alloc_ctx);
        b.custom = true;
        b.release = g_release;
        b.ctx = g_alloc_ctx;
        if (!b.ptr) return fail(MG_ENOMEM, "device allocator returned NULL for %zu bytes", bytes);
        return MG_OK;
    }
    hipError_t e = hipMalloc(&b.ptr, bytes);
    if (e != hipSuccess) {
        (void)hipGetLastError();
        b.ptr = nullptr;
        return fail(MG_ENOMEM, "hipMalloc(%zu) failed: %s", bytes, hipGetErrorString(e));
    }
    return MG_OK;
}

void dev_free(DevBuf &b) {
    if (!b.ptr) return;
    if (b.part) {
        // (its allocation is released by its own owner)
    } else if (b.custom) {
        if (b.release) b.release(b.ptr, b.stream, b.ctx);
    } else {
        (void)hipFree(b.ptr);
    }
    b.ptr = nullptr;
}

}  // namespace mgh

using namespace mgh;

mg_graph::~mg_graph() {
    for (DevBuf *b : {&gsrc, &gdst, &gt, &gx, &gn, &gp, &pair_t, &out_eid, &in_eid, &out_off,
                      &out_adj, &in_off, &in_adj, &order, &block})
        dev_free(*b);
}

namespace {

// f(begin, end) over [0, n) in contiguous pieces on the host's cores
template <typename F>
void parallel_for(int64_t n, F f) {
    const int64_t nt = std::max<int64_t>(1, std::min<int64_t>(std::thread::hardware_concurrency(),
                                                                n / 65536 + 1));
    std::vector<std::thread> th;
    for (int64_t k = 0; k < nt; ++k)
        th.emplace_back([&, k] { f(n * k / nt, n * (k + 1) / nt); });
    for (auto &x : th) x.join();
}

// Frees a set of device buffers at the end of a scope.
struct Scratch {
    std::vector<DevBuf> bufs;
    ~Scratch() { drop(); }
    void drop() {
        for (DevBuf &b : bufs) dev_free(b);
        bufs.clear();
    }
    int alloc(void **p, size_t bytes, hipStream_t st) {
        bufs.emplace_back();
        const int rc = dev_alloc(bufs.back(), bytes, (void *)st);
        *p = bufs.back().ptr;
        return rc;
    }
    template <typename T>
    int get(T **p, size_t n, hipStream_t st) { return alloc((void **)p, sizeof(T) * n, st); }
};

int bit_width(uint64_t x) {
    int b = 0;
    while (x) { ++b; x >>= 1; }
    return b;
}

#define LAUNCH_TRY(expr)                                                                  \
    do {                                                                                  \
        hipError_t e_ = (expr);                                                           \
        if (e_ != hipSuccess)                                                             \
            return fail(MG_EDEVICE, "graph ingest failed: %s", hipGetErrorString(e_));    \
    } while (0)

template <typename TT>
mg::DevGraph<TT> dev_graph(const mg_graph *g);

// Graphs of this many edges and more do without the pair records per list entry,
// 32 of their 120 bytes per edge (136 with 64-bit times): 2^31 edges hold 189 GB of
// the 288 instead of 258 (223 instead of 292).  Below it the records of the edges
// and of both lists' entries have 32-bit places.
constexpr uint32_t kLeanEdges = 1u << 30;
// Graphs of fewer edges take one allocation for all their arrays (13 or 14 of them
// and the temporaries' were a fifth of the build of 1,000 edges); from this many on
// (16 MB) the uploaded input is released once the edges are placed, at the price of
// a wait for the stream, and the pair records are allocated after that.
constexpr uint32_t kOneBlockEdges = 1u << 20;

// Builds the device graph from checked edge arrays in device memory: sorts
// the edges by time unless they are, then both sides' lists and the per-edge
// list ranks (ingest.hip).  `input` is what holds those arrays, when they are not
// the caller's.  Returns once the stream has finished it.
//
// Memory: what the graph keeps and 16 bytes per edge of temporaries.  The sorts work in arrays that are written
// after them: the time sort in gx and gn, the source and destination sorts in gx,
// the pair sort in the records.
template <typename TT>
int ingest_graph(mg_graph *g, const int32_t *src, const int32_t *dst, const int64_t *t, bool sorted,
                 Scratch &input, hipStream_t st) {
    const uint32_t E = (uint32_t)g->E, V = (uint32_t)g->V;
    const uint32_t A = (uint32_t)(g->E - g->self_loops);   // list entries
    // 32-bit times leave room for the edge id in the list entry
    constexpr size_t kEid = sizeof(TT) == 4 ? 0 : sizeof(uint32_t);
    struct Need { DevBuf *b; size_t n; };
    std::vector<Need> needs = {
        {&g->gsrc, sizeof(int32_t) * (size_t)E}, {&g->gdst, sizeof(int32_t) * (size_t)E},
        {&g->gt, sizeof(TT) * (size_t)E},        {&g->gx, sizeof(uint32_t) * 4 * (size_t)E},
        {&g->gn, sizeof(uint32_t) * 2 * (size_t)E},
        {&g->pair_t, sizeof(TT) * ((size_t)A + 4)},   // read four entries at a time
        {&g->out_eid, kEid * (size_t)A}, {&g->in_eid, kEid * (size_t)A},
        {&g->out_off, sizeof(uint32_t) * ((size_t)V + 1)},
        {&g->out_adj, sizeof(mg::Entry<TT>) * (size_t)A},
        {&g->in_off, sizeof(uint32_t) * ((size_t)V + 1)},
        {&g->in_adj, sizeof(mg::Entry<TT>) * (size_t)A},
    };
    if (!sorted) needs.push_back({&g->order, sizeof(uint32_t) * (size_t)E});
    // The pair records of the edges, and once more (`entries`) in the order of both
    // lists' entries, where a candidate reads them with its neighbours; without
    // memory for those the search takes them by edge id.
    auto gp_bytes = [&](bool entries) {
        return 4 * sizeof(uint32_t) * ((size_t)E + (entries ? 2 * (size_t)A : 0));
    };
    auto up = [](size_t n) { return (std::max<size_t>(n, 16) + 255) & ~(size_t)255; };
    Scratch tmp;
    char *mem = nullptr;
    const size_t sort_bytes = up(mg::sort_scratch_bytes(E));
    int rc = tmp.get(&mem, sort_bytes + 4 * sizeof(uint32_t) * (size_t)E, st);
    if (rc) return rc;
    void *sort_mem = mem;
    uint32_t *opos = (uint32_t *)(mem + sort_bytes);
    uint32_t *ipos = opos + E, *ikey = ipos + E, *oeid = ikey + E;
    g->device_bytes = 0;
    auto keep = [&](DevBuf &b, size_t n) -> int {
        const int rc = dev_alloc(b, n, (void *)st);
        if (!rc) g->device_bytes += (int64_t)n;
        return rc;
    };
    if (E < kOneBlockEdges) {
        rc = MG_ENOMEM;
        for (int lean = 0; lean < 2 && rc; ++lean) {
            size_t all = up(gp_bytes(!lean));
            for (const Need &u : needs) all += up(u.n);
            rc = dev_alloc(g->block, all, (void *)st);
            g->gp_entries = !lean && E > 0;
        }
        if (rc) return rc;
        needs.push_back({&g->gp, gp_bytes(g->gp_entries)});
        char *at = (char *)g->block.ptr;
        for (const Need &u : needs) {
            u.b->ptr = at;
            u.b->bytes = u.n;
            u.b->part = true;
            g->device_bytes += (int64_t)u.n;
            at += up(u.n);
        }
    } else {
        for (const Need &u : needs) {
            rc = keep(*u.b, u.n);
            if (rc) return rc;
        }
    }
    // on an error the kernels already queued still use all of this memory
    struct Wait {
        hipStream_t st;
        bool done;
        ~Wait() { if (!done) (void)hipStreamSynchronize(st); }
    } wait{st, false};
    auto part = [&](const DevBuf &b, size_t i) { return (uint32_t *)b.ptr + i * E; };
    int at = 0;
    if (!sorted) {
        TT *tk[2] = {(TT *)g->gx.ptr, (TT *)g->gx.ptr + E};
        uint32_t *v[2] = {part(g->gn, 0), part(g->gn, 1)};
        LAUNCH_TRY(mg::launch_time_keys<TT>(t, g->t_min, E, tk[0], st));
        LAUNCH_TRY(mg::sort_pairs<TT>(tk, v, true, E, bit_width((uint64_t)(g->t_max - g->t_min)),
                                      sort_mem, &at, st));
        HIP_TRY(hipMemcpyAsync(g->order.ptr, v[at], sizeof(uint32_t) * (size_t)E,
                               hipMemcpyDeviceToDevice, st));
    }
    uint32_t *okey = part(g->gx, 0), *v[2] = {part(g->gx, 2), part(g->gx, 3)};
    auto *gsrc = (int32_t *)g->gsrc.ptr, *gdst = (int32_t *)g->gdst.ptr;
    TT *gt = (TT *)g->gt.ptr;
    if (E)
        LAUNCH_TRY(mg::launch_place_edges<TT>(src, dst, t, g->t_min, (const uint32_t *)g->order.ptr,
                                              E, V, gsrc, gdst, gt, okey, ikey, st));
    if (!input.bufs.empty() && E >= kOneBlockEdges) {
        HIP_TRY(hipStreamSynchronize(st));
        input.drop();
    }
    const int vb = bit_width(V);   // vertices and V itself (self-loops)
    for (int side = 0; side < 2; ++side) {
        uint32_t *k[2] = {side ? ikey : okey, part(g->gx, 1)};
        LAUNCH_TRY(mg::sort_pairs<uint32_t>(k, v, true, E, vb, sort_mem, &at, st));
        DevBuf &eid = side ? g->in_eid : g->out_eid;
        if (A && kEid)
            HIP_TRY(hipMemcpyAsync(eid.ptr, v[at], kEid * (size_t)A, hipMemcpyDeviceToDevice, st));
        if (A && side == 0)   // the pair order starts from this one
            HIP_TRY(hipMemcpyAsync(oeid, v[at], sizeof(uint32_t) * (size_t)A,
                                   hipMemcpyDeviceToDevice, st));
        LAUNCH_TRY(mg::launch_lists<TT>(k[at], v[at], A, V, side ? gsrc : gdst, gt,
                                        (uint32_t *)(side ? g->in_off : g->out_off).ptr,
                                        (mg::Entry<TT> *)(side ? g->in_adj : g->out_adj).ptr,
                                        side ? ipos : opos, st));
    }
    LAUNCH_TRY(mg::launch_ranks<TT>(dev_graph<TT>(g), opos, ipos, (uint4 *)g->gx.ptr,
                                    (uint2 *)g->gn.ptr, st));
    if (!g->gp.ptr) {
        g->gp_entries = E < kLeanEdges && !keep(g->gp, gp_bytes(true));
        if (!g->gp_entries) rc = keep(g->gp, gp_bytes(false));
        if (rc) return rc;
    }
    // pair order: the out-lists' order (source, time) sorted by destination
    uint32_t *pv[2] = {oeid, ikey}, *pk[2] = {part(g->gp, 0), part(g->gp, 1)};
    if (A) {
        LAUNCH_TRY(mg::launch_gather(pv[0], gdst, A, pk[0], st));
        LAUNCH_TRY(mg::sort_pairs<uint32_t>(pk, pv, false, A, vb, sort_mem, &at, st));
    }
    // self-loops are in no pair: their records are zero
    if (g->self_loops) HIP_TRY(hipMemsetAsync(g->gp.ptr, 0, gp_bytes(false), st));
    if (A)
        LAUNCH_TRY(mg::launch_pairs<TT>(dev_graph<TT>(g), pv[at], A, opos, ipos, (int32_t *)pv[at ^ 1],
                                        (TT *)g->pair_t.ptr, (uint4 *)g->gp.ptr,
                                        (uint2 *)g->gn.ptr, (mg::Entry<TT> *)g->out_adj.ptr,
                                        (mg::Entry<TT> *)g->in_adj.ptr, st));
    wait.done = true;
    HIP_TRY(hipStreamSynchronize(st));
    return MG_OK;
}

}  // namespace

// ---------------------------------------------------------------- tree
mg_tree::~mg_tree() {
    dev_free(d_tab);
    release_cpu_code(this);
}

namespace {

// First-appearance relabelling: vertices are numbered in the order they are
// first seen, source before destination.  Two motifs are the same ordered
// edge sequence up to relabelling iff their relabelled forms are equal.
int canonical(const int32_t *uv, int k, Motif &out) {
    std::vector<std::pair<int32_t, int>> seen;
    auto id = [&](int32_t x) {
        for (auto &p : seen) if (p.first == x) return p.second;
        seen.push_back({x, (int)seen.size()});
        return (int)seen.size() - 1;
    };
    out.clear();
    for (int j = 0; j < k; ++j) {
        int32_t a = uv[2 * j], b = uv[2 * j + 1];
        if (a < 0 || b < 0) return fail(MG_EINVAL, "motif vertex label < 0");
        if (a == b) return fail(MG_EINVAL, "motif edge %d is a self-loop", j);
        int ia = id(a), ib = id(b);
        out.push_back({ia, ib});
    }
    if ((int)seen.size() > kVMax)
        return fail(MG_EUNSUPPORTED, "motif has %d vertices (limit %d)", (int)seen.size(), kVMax);
    return MG_OK;
}

// Build the prefix trie, then the flat tables the kernel reads.
int build_tree(mg_tree *tr) {
    tr->nodes.clear();
    TrieNode root;
    root.u = 0; root.v = 1; root.depth = 1; root.nv = 2;
    tr->nodes.push_back(root);
    for (size_t q = 0; q < tr->distinct.size(); ++q) {
        const Motif &m = tr->distinct[q];
        int cur = 0;
        for (size_t j = 1; j < m.size(); ++j) {
            int found = -1;
            for (int c : tr->nodes[cur].kids)
                if (tr->nodes[c].u == m[j].first && tr->nodes[c].v == m[j].second) found = c;
            if (found < 0) {
                TrieNode n;
                n.parent = cur;
                n.u = m[j].first; n.v = m[j].second;
                n.depth = tr->nodes[cur].depth + 1;
                int hi = std::max(n.u, n.v);
                n.nv = std::max(tr->nodes[cur].nv, hi + 1);
                found = (int)tr->nodes.size();
                tr->nodes.push_back(n);
                tr->nodes[cur].kids.push_back(found);
            }
            cur = found;
        }
        tr->nodes[cur].q = (int)q;
    }
    // flat tables (see comine.h): internal nodes get dense indices, the
    // root (node 0) being internal index 0 whenever it has children
    const int N = (int)tr->nodes.size();
    std::vector<int> iidx(N, -1);
    int n_int = 0;
    for (int n = 0; n < N; ++n)
        if (!tr->nodes[n].kids.empty()) iidx[n] = n_int++;
    if (n_int > 0xffff) return fail(MG_EUNSUPPORTED, "%d internal search nodes (limit 65535)", n_int);
    auto child_word = [&](int c) -> int32_t {
        const TrieNode &ch = tr->nodes[c];
        uint32_t w = ((uint32_t)(ch.q + 1) & 0x7fffu) << 16;
        if (iidx[c] >= 0) w |= (uint32_t)iidx[c] | 0x80000000u;
        return (int32_t)w;
    };
    tr->node_tab.assign(4 * (size_t)std::max(n_int, 1), 0);
    tr->grp_tab.clear();
    tr->root_pairs = 0;
    tr->pair_tab.assign(32 * (size_t)std::max(n_int, 1), 0);
    tr->depth = 0;
    bool wide2 = false;   // an internal two-edge prefix on four vertices
    for (int n = 0; n < N; ++n) {
        const TrieNode &nd = tr->nodes[n];
        tr->depth = std::max(tr->depth, nd.depth);
        if (nd.depth == 2 && nd.nv > 3 && !nd.kids.empty()) wide2 = true;
        if (nd.kids.empty()) continue;
        // the matched edges of the prefix, first edge first
        std::vector<std::pair<int, int>> path;
        for (int c = n; c >= 0; c = tr->nodes[c].parent)
            path.insert(path.begin(), {tr->nodes[c].u, tr->nodes[c].v});
        // group the children by the list they scan, in live-word bit order
        std::map<int, std::vector<int>> groups;
        for (int c : nd.kids) {
            const TrieNode &ch = tr->nodes[c];
            const int bit = ch.u < nd.nv   ? 2 * ch.u + mg::kDirOut
                            : ch.v < nd.nv ? 2 * ch.v + mg::kDirIn
                                           : (int)mg::kLiveAllBit;
            groups[bit].push_back(c);
        }
        const int g0 = (int)tr->grp_tab.size() / 12;
        if (g0 + (int)groups.size() > (1 << 20))
            return fail(MG_EUNSUPPORTED, "too many child groups");
        uint32_t lists = 0, gate = 0, pairs = 0, by_window = 0;
        bool news = false;   // a new-vertex child whose window is counted from pairs
        for (auto &kv : groups) {
            const bool all = kv.first == (int)mg::kLiveAllBit;
            const int dir = all ? mg::kDirAll : kv.first & 1, anc = all ? 0 : kv.first >> 1;
            bool leaf_only = !all;
            for (int c : kv.second) leaf_only = leaf_only && tr->nodes[c].kids.empty();
            // the anchor is the source (1) or destination (2) of the node's
            // own last edge: the window then starts where that edge's time
            // ends in the anchor's list, known per edge; likewise, no earlier
            // than there, for its second edge
            auto end_of = [&](size_t j) {
                return all || j >= path.size() || j == 0 ? 0
                       : anc == path[j].first            ? 1
                       : anc == path[j].second           ? 2
                                                         : 0;
            };
            const int last_end = all ? 0 : anc == nd.u ? 1 : anc == nd.v ? 2 : 0;
            int32_t rec[12] = {dir | (anc << 4) | (nd.nv << 8) | ((leaf_only ? 1 : 0) << 12) |
                                   (last_end << 13) | (end_of(1) << 15)};
            bool counted[kVMax] = {};
            for (int c : kv.second) {
                const TrieNode &ch = tr->nodes[c];
                // out-group: the scanned endpoint is the destination; a bound
                // destination selects word 1+v, a new one word 7.  In- and
                // whole-list groups only ever reach new vertices (word 7).
                if (dir == mg::kDirOut && ch.v < nd.nv) {
                    rec[1 + ch.v] = child_word(c);
                    counted[ch.v] = true;
                } else {
                    rec[7] = child_word(c);
                }
            }
            // a leaf window's count is known from the pairs of its anchor with
            // the counted vertices (with a new-vertex child, all bound ones)
            // when each is joined to the anchor by a matched edge
            std::vector<std::pair<int, int>> by;   // (pair, vertex) counted
            bool known = leaf_only;
            for (int y = 0; y < nd.nv && known; ++y) {
                if (y == anc || !(counted[y] || rec[7])) continue;
                int pair = -1;
                for (size_t j = 0; j < path.size(); ++j) {   // the latest such edge
                    // the list's entries run from the anchor (out) or to it (in)
                    const std::pair<int, int> with =
                        dir == mg::kDirOut ? std::make_pair(anc, y) : std::make_pair(y, anc);
                    if (path[j] == with) pair = 2 * (int)j;
                    else if (path[j].first == with.second && path[j].second == with.first)
                        pair = 2 * (int)j + 1;
                }
                known = pair >= 0;
                by.push_back({pair, y});
            }
            uint32_t codes = 0;   // the pairs, when all are known
            for (auto &x : by) codes |= known ? 1u << x.first : 0u;
            rec[8] = codes ? 1 : 0;
            pairs |= codes;
            if (codes)
                for (auto &x : by) {
                    // each pair is in the out-list of its source and the
                    // in-list of its destination
                    int32_t *w = &tr->pair_tab[32 * (size_t)iidx[n] + 4 * x.first];
                    if (dir == mg::kDirOut) {
                        w[0] = rec[1 + x.second];
                        w[1] = rec[7];
                    } else {
                        w[2] = rec[7];
                    }
                }
            lists |= 1u << kv.first;
            if (!codes || rec[7]) by_window |= 1u << kv.first;
            news = news || (codes && rec[7]);
            gate |= codes && !rec[7] ? codes << mg::kLivePair : 1u << kv.first;
            tr->grp_tab.insert(tr->grp_tab.end(), rec, rec + 12);
        }
        // a leaf parent: every match below it is one more edge on a list of
        // a bound vertex
        bool leaf_parent = true;
        for (int c : nd.kids) {
            const TrieNode &ch = tr->nodes[c];
            leaf_parent = leaf_parent && ch.kids.empty() && (ch.u < nd.nv || ch.v < nd.nv);
        }
        int32_t *w = &tr->node_tab[4 * (size_t)iidx[n]];
        w[0] = g0;
        if (leaf_parent) tr->root_pairs |= pairs & 3u;
        w[1] = (int32_t)lists;
        w[2] = (int32_t)(leaf_parent ? gate | mg::kLeafParent : lists);
        w[3] = (int32_t)(leaf_parent ? by_window | pairs << 16 | (news ? 1u << 24 : 0u) : 0u);
    }
    if (tr->grp_tab.empty()) tr->grp_tab.assign(12, 0);
    tr->root_q = tr->nodes[0].q;
    tr->kdepth = (tr->depth == 3 && wide2) ? 4 : tr->depth;

    // MG-Tree view: the root is the longest prefix shared by every motif;
    // below it a node exists where a prefix is a query or branches.
    int r = 0;
    while (tr->nodes[r].q < 0 && tr->nodes[r].kids.size() == 1) r = tr->nodes[r].kids[0];
    int mg_nodes = 0;
    std::vector<int> stack{r};
    while (!stack.empty()) {
        int n = stack.back();
        stack.pop_back();
        const TrieNode &nd = tr->nodes[n];
        if (n == r || nd.q >= 0 || nd.kids.size() != 1) mg_nodes++;
        for (int c : nd.kids) stack.push_back(c);
    }
    long total_edges = 0;
    for (auto &m : tr->distinct) total_edges += (long)m.size();
    mg_tree_info_t &in = tr->info;
    in.n_motifs = tr->n_motifs;
    in.n_distinct = (int32_t)tr->distinct.size();
    in.n_prefixes = N;
    in.n_nodes = mg_nodes;
    in.depth = tr->depth;
    in.root_edges = tr->nodes[r].depth;
    in.similarity = total_edges ? 1.0 - (double)N / (double)total_edges : 0.0;
    in.delta = tr->delta;
    in.n_deltas = (int32_t)tr->delta_slot.size();
    return MG_OK;
}

int make_tree(const std::vector<Motif> &canon, const std::vector<int64_t> &windows,
              mg_tree **out) {
    std::unique_ptr<mg_tree> tr(new (std::nothrow) mg_tree);
    if (!tr) return fail(MG_ENOMEM, "out of host memory");
    tr->n_motifs = (int32_t)canon.size();
    tr->deltas = windows;
    std::sort(tr->deltas.begin(), tr->deltas.end());
    tr->deltas.erase(std::unique(tr->deltas.begin(), tr->deltas.end()), tr->deltas.end());
    for (int64_t w : windows)
        tr->delta_slot.push_back(
            (int32_t)(std::lower_bound(tr->deltas.begin(), tr->deltas.end(), w) - tr->deltas.begin()));
    tr->delta = tr->deltas.back();
    std::map<Motif, int> ids;
    for (const Motif &m : canon) {
        auto it = ids.find(m);
        int q;
        if (it == ids.end()) {
            q = (int)tr->distinct.size();
            ids[m] = q;
            tr->distinct.push_back(m);
        } else {
            q = it->second;
        }
        tr->motif_q.push_back(q);
    }
    if ((int)tr->distinct.size() > MG_MAX_QUERIES)
        return fail(MG_EUNSUPPORTED, "%d distinct motifs (limit %d)", (int)tr->distinct.size(),
                    MG_MAX_QUERIES);
    if (tr->distinct.size() * tr->deltas.size() > (size_t)MG_MAX_QUERIES)
        return fail(MG_EUNSUPPORTED, "%d distinct motifs x %d windows exceed %d counters",
                    (int)tr->distinct.size(), (int)tr->deltas.size(), MG_MAX_QUERIES);
    int rc = build_tree(tr.get());
    if (rc) return rc;
    *out = tr.release();
    return MG_OK;
}

// Caller-visible counts of one tree from its counters (n_d slots per
// distinct motif; slot j holds the matches whose span fits window j but not
// window j - 1): out[i * n_motifs + m] for the caller's window i and motif m.
void map_counts(const mg_tree *tr, const uint64_t *slots, uint64_t *out) {
    const size_t nd = tr->deltas.size();
    for (size_t i = 0; i < tr->delta_slot.size(); ++i)
        for (int32_t m = 0; m < tr->n_motifs; ++m) {
            const uint64_t *c = slots + (size_t)tr->motif_q[m] * nd;
            uint64_t sum = 0;
            for (int32_t j = 0; j <= tr->delta_slot[i]; ++j) sum += c[j];
            out[i * (size_t)tr->n_motifs + m] = sum;
        }
}

// Host memory that small counts' kernels store their counters in: one buffer
// per thread (a call returns after its stream is done with it), allocated by
// the thread's first small mg_count and kept until the thread ends.
constexpr uint32_t kPartCounters = 8192;
struct PartBuf {
    uint64_t *host = nullptr;
    ~PartBuf() { if (host) (void)hipHostFree(host); }
    uint64_t *get(bool may_allocate) {
        if (!host && may_allocate && hipHostMalloc((void **)&host, 8 * (size_t)kPartCounters,
                                   hipHostMallocPortable | hipHostMallocMapped) != hipSuccess) {
            (void)hipGetLastError();
            host = nullptr;
        }
        return host;
    }
};
thread_local PartBuf g_part;
constexpr int64_t kPartRoots = 1 << 16;   // counts of more roots are not small

size_t n_slots(const mg_tree *tr) { return tr->distinct.size() * tr->deltas.size(); }

int upload_tree(mg_tree *tr, int device, hipStream_t st) {
    if (tr->device == device && tr->d_tab.ptr) return MG_OK;
    dev_free(tr->d_tab);
    std::vector<int32_t> all;
    for (const std::vector<int32_t> *t : {&tr->node_tab, &tr->grp_tab, &tr->pair_tab})
        all.insert(all.end(), t->begin(), t->end());
    int rc = dev_alloc(tr->d_tab, all.size() * 4, (void *)st);
    if (rc) return rc;
    HIP_TRY(hipMemcpyAsync(tr->d_tab.ptr, all.data(), all.size() * 4, hipMemcpyHostToDevice, st));
    HIP_TRY(hipStreamSynchronize(st));   // `all` is released on return
    tr->device = device;
    return MG_OK;
}

// The search of one tree; counts land in d_counts.  Queue heads, counters and
// statistics are zero already.
template <typename TT>
int learned_search(const mg_graph *g, mg_tree *tr, const mg_model *model,
                   const mg::KParams<TT> &base, int blocks, uint32_t stride, hipStream_t st);

template <typename TT>
mg::DevGraph<TT> dev_graph(const mg_graph *g);
mg::DevTree dev_tree(const mg_tree *tr);
template <typename TT>
TT delta_sat(int64_t delta);

// Kernel parameters of a count over every root of g (the caller may then
// restrict the roots).
template <typename TT>
void fill_params(mg::KParams<TT> &p, const mg_graph *g, const mg_tree *tr, const mg_count_opts &o,
                 unsigned long long *d_queues, unsigned long long *d_counts,
                 unsigned long long *d_stats, unsigned long long *d_cost) {
    p.g = dev_graph<TT>(g);
    p.tree = dev_tree(tr);
    p.delta_sat = delta_sat<TT>(tr->delta);
    for (size_t i = 0; i + 1 < tr->deltas.size(); ++i) p.dlo[i] = delta_sat<TT>(tr->deltas[i]);
    p.roots = nullptr;
    p.n_roots = (uint32_t)g->E;
    // a stopped count's chunks are part of its resume point
    p.chunk = (uint32_t)(o.chunk > 0 ? o.chunk : (o.stop || o.max_chunks || o.cursor || o.epoch_idle) ? 64 : 0);
    p.n_queues = (uint32_t)(o.queues > 0 ? o.queues : mg::kQueues);
    p.leaf_scan = o.leaf_scan < 0 ? 0u : (o.leaf_scan == 0 ? mg::kLeafScanDefault
                                                           : (uint32_t)o.leaf_scan);
    p.queues = d_queues;
    p.counts = d_counts;
    p.stats = d_stats;
    p.root_cost = d_cost;
    p.stop = o.stop;
    p.max_chunks = (uint32_t)o.max_chunks;
}

// A small co-mining count in one launch (KParams::part): true when it was taken
// (*rc: its status, counts in slots[0..n_slots)), false when it is not small or
// there is no buffer for it yet and none may be allocated.  A count of 1,000
// edges is all launches and waits: fill, search and copy back took 78 us a
// call, one launch that stores to mapped host memory takes 33.
template <typename TT>
bool small_count(const mg_graph *g, const mg_tree *tr, const mg_count_opts &o, bool may_allocate,
                 uint64_t *slots, hipStream_t st, int *rc) {
    uint64_t *part = g->E > 0 && g->E <= kPartRoots ? g_part.get(may_allocate) : nullptr;
    if (!part) return false;
    mg::KParams<TT> p{};
    uint32_t rows = 0;
    fill_params<TT>(p, g, tr, o, nullptr, nullptr, nullptr, nullptr);
    void *dev = nullptr;
    if (hipHostGetDevicePointer(&dev, part, 0) != hipSuccess) {
        (void)hipGetLastError();
        return false;
    }
    p.part = (unsigned long long *)dev;
    p.part_cap = kPartCounters;
    p.part_rows = &rows;
    hipError_t e = mg::launch_comine<TT>(p, o.blocks, st);
    if (e == hipErrorNotSupported) return false;
    if (e == hipSuccess) e = hipStreamSynchronize(st);
    *rc = e == hipSuccess ? MG_OK : fail(MG_EDEVICE, "co-mining launch failed: %s", hipGetErrorString(e));
    const size_t n = n_slots(tr);
    std::fill(slots, slots + n, 0);
    for (size_t r = 0; e == hipSuccess && r < rows; ++r)
        for (size_t i = 0; i < n; ++i) slots[i] += part[r * n + i];
    return true;
}

constexpr uint32_t kHandOnRoots = 1u << 17;   // counts of fewer roots hand nothing on: a
                                              // wave has 16 roots or fewer there
constexpr uint64_t kHandOnCap = 1u << 18;     // contexts one count can hand on (16 MB)
constexpr uint64_t kCtxCap = 1u << 20;   // contexts one epoch can hand on (64 MB)

// Whether the heavy chunks of a count over n_roots roots may be handed on.  Its
// context buffer is allocated for the call and only for such a call (12 us of a
// hipMalloc, less from a caching allocator); without memory for it nothing is
// handed on.
bool hands_on(const mg_count_opts &o, uint32_t n_roots) {
    return n_roots >= kHandOnRoots && o.sched == MG_SCHED_PLAIN && !o.epoch_idle && !o.stop &&
           !o.max_chunks && !o.stats && !o.root_cost && !o.wave_clock;
}

// Epochs (paper, section 4.5): launch after launch, each ending once
// o.epoch_idle percent of its waves are idle; the root-level candidates the
// busy waves had not reached yet come back as contexts, which the next launch
// spreads over all of its waves.  The last of max_epochs launches runs to the
// end.  Counts accumulate in p.counts; p.queues is cleared before each launch.
template <typename TT>
int epoch_search(mg::KParams<TT> p, const mg_count_opts &o, hipStream_t st) {
    const int max_epochs = o.max_epochs > 0 ? o.max_epochs : 16;
    struct Free {
        DevBuf *b;
        ~Free() { dev_free(b[0]); dev_free(b[1]); dev_free(b[2]); }
    };
    DevBuf all[3];
    Free fr{all};
    for (int i = 0; i < 2; ++i) {
        int rc = dev_alloc(all[i], sizeof(mg::EpochCtx) * kCtxCap, (void *)st);
        if (rc) return rc;
    }
    int rc = dev_alloc(all[2], 16, (void *)st);
    if (rc) return rc;
    p.ctx_count = (unsigned long long *)all[2].ptr;
    p.idle = (uint32_t *)((char *)all[2].ptr + 8);
    p.ctx_cap = kCtxCap;
    p.idle_pct = (uint32_t)o.epoch_idle;
    for (int ep = 0; ep < max_epochs; ++ep) {
        const bool last = ep + 1 == max_epochs;
        p.ctx_out = last ? nullptr : (mg::EpochCtx *)all[ep & 1].ptr;
        HIP_TRY(hipMemsetAsync(all[2].ptr, 0, 16, st));
        if (ep > 0) HIP_TRY(hipMemsetAsync(p.queues, 0, kQueueBytes, st));
        // (the first launch with neither contexts in nor out is the plain search)
        hipError_t e = mg::launch_comine<TT>(p, o.blocks, st);
        if (e != hipSuccess)
            return fail(MG_EDEVICE, "co-mining launch failed: %s", hipGetErrorString(e));
        unsigned long long n = 0;
        if (p.ctx_out) {
            HIP_TRY(hipMemcpyAsync(&n, p.ctx_count, sizeof n, hipMemcpyDeviceToHost, st));
            HIP_TRY(hipStreamSynchronize(st));
        }
        if (o.epoch_contexts) o.epoch_contexts[ep] = (int64_t)n;
        if (n == 0) {
            for (int k = ep + 1; o.epoch_contexts && k < max_epochs; ++k) o.epoch_contexts[k] = 0;
            break;
        }
        p.ctx_in = (const mg::EpochCtx *)all[ep & 1].ptr;
        p.n_ctx_in = (uint32_t)n;
    }
    return MG_OK;
}

template <typename TT>
int launch_tree(const mg_graph *g, mg_tree *tr, const uint32_t *d_roots, uint32_t n_roots,
                unsigned long long *d_queues, unsigned long long *d_counts,
                unsigned long long *d_stats, unsigned long long *d_cost,
                unsigned long long *d_clock, mg::EpochCtx *ctx, const mg_count_opts &o,
                hipStream_t st, float *ms) {
    mg::KParams<TT> p{};
    fill_params<TT>(p, g, tr, o, d_queues, d_counts, d_stats, d_cost);
    p.roots = d_roots;
    p.n_roots = n_roots;
    p.wave_clock = d_clock;
    p.n_wave_clock = d_clock ? (uint32_t)std::min<int64_t>(o.wave_clock_len / 2, 0x7fffffff) : 0u;

    if (o.cursor && o.cursor->started) {
        // resume: every root queue starts where the last call stopped
        std::vector<unsigned long long> q(mg::kQueueWords, 0ull);
        for (int i = 0; i < mg::kQueues; ++i) q[(size_t)i * mg::kQueueStride] = o.cursor->head[i];
        HIP_TRY(hipMemcpyAsync(d_queues, q.data(), kQueueBytes, hipMemcpyHostToDevice, st));
        HIP_TRY(hipStreamSynchronize(st));   // q is released on return
    }
    hipEvent_t e0 = nullptr, e1 = nullptr;
    if (ms) {
        HIP_TRY(hipEventCreate(&e0));
        HIP_TRY(hipEventCreate(&e1));
        HIP_TRY(hipEventRecord(e0, st));
    }
    if (n_roots > 0 && o.sched == MG_SCHED_LEARNED) {
        int rc = learned_search<TT>(g, tr, o.model, p, o.blocks,
                                    o.sample > 0 ? (uint32_t)o.sample : kSampleDefault, st);
        if (rc) return rc;
    } else if (n_roots > 0 && o.epoch_idle > 0) {
        int rc = epoch_search<TT>(p, o, st);
        if (rc) return rc;
    } else if (n_roots > 0) {
        // Deep trees over many roots: the candidates of the heaviest root
        // chunks are searched by a second launch, spread over the device (one
        // wave's 64 roots inside a burst took as long as everything else: half
        // of a count of 3M edges with 756 motifs).
        const bool two = ctx && tr->kdepth > 2;
        if (two) {
            p.hand_on = 1;
            p.ctx_out = ctx;
            p.ctx_cap = kHandOnCap;
            p.ctx_count = d_queues + mg::kCtxCountWord;
        }
        hipError_t e = mg::launch_comine<TT>(p, o.blocks, st);
        if (e == hipSuccess && two) {
            p.hand_on = 0;
            p.ctx_in = p.ctx_out;
            p.ctx_out = nullptr;
            p.ctx_n = p.ctx_count;
            e = mg::launch_comine<TT>(p, o.blocks, st);
        }
        if (e != hipSuccess)
            return fail(MG_EDEVICE, "co-mining launch failed: %s", hipGetErrorString(e));
    }
    if (ms) {
        HIP_TRY(hipEventRecord(e1, st));
        HIP_TRY(hipEventSynchronize(e1));
        HIP_TRY(hipEventElapsedTime(ms, e0, e1));
        (void)hipEventDestroy(e0);
        (void)hipEventDestroy(e1);
    }
    return MG_OK;
}

}  // namespace

int mgh::chain_trees(mg_tree *tr) {
    if (!tr->singles.empty()) return MG_OK;
    for (const Motif &m : tr->distinct) {
        mg_tree *one = nullptr;
        int rc = make_tree({m}, tr->deltas, &one);
        if (rc) return rc;
        tr->singles.emplace_back(one);
    }
    return MG_OK;
}


// ---------------------------------------------------------------- cost model
static_assert(mg::kParams == MG_MODEL_PARAMS, "parameter layout");
static_assert(mg::kFeat == MG_NFEATURES, "feature count");

struct mg_model {
    int device = 0;
    DevBuf params, adam_m, adam_v;
    ~mg_model() {
        dev_free(params);
        dev_free(adam_m);
        dev_free(adam_v);
    }
};

namespace {

uint64_t splitmix(uint64_t &s) {
    uint64_t z = (s += 0x9e3779b97f4a7c15ull);
    z = (z ^ (z >> 30)) * 0xbf58476d1ce4e5b9ull;
    z = (z ^ (z >> 27)) * 0x94d049bb133111ebull;
    return z ^ (z >> 31);
}
double uniform01(uint64_t &s) { return ((splitmix(s) >> 11) + 0.5) * (1.0 / 9007199254740992.0); }
double normal(uint64_t &s) {   // Box-Muller
    const double u = uniform01(s), v = uniform01(s);
    return std::sqrt(-2.0 * std::log(u)) * std::cos(6.283185307179586 * v);
}

template <typename TT>
mg::DevGraph<TT> dev_graph(const mg_graph *g) {
    mg::DevGraph<TT> d{};
    d.gsrc = (const int32_t *)g->gsrc.ptr;
    d.gdst = (const int32_t *)g->gdst.ptr;
    d.gt = (const TT *)g->gt.ptr;
    d.gx = (const uint4 *)g->gx.ptr;
    d.gn = (const uint2 *)g->gn.ptr;
    d.gp = (const uint4 *)g->gp.ptr;
    d.gp_out = g->gp_entries ? (uint32_t)g->E : 0u;
    d.gp_in = g->gp_entries ? (uint32_t)(2 * g->E - g->self_loops) : 0u;
    d.pair_t = (const TT *)g->pair_t.ptr;
    d.out_eid = (const uint32_t *)g->out_eid.ptr;
    d.in_eid = (const uint32_t *)g->in_eid.ptr;
    d.out_off = (const uint32_t *)g->out_off.ptr;
    d.out_adj = (const mg::Entry<TT> *)g->out_adj.ptr;
    d.in_off = (const uint32_t *)g->in_off.ptr;
    d.in_adj = (const mg::Entry<TT> *)g->in_adj.ptr;
    d.n_edges = (uint32_t)g->E;
    return d;
}

mg::DevTree dev_tree(const mg_tree *tr) {
    mg::DevTree t{};
    t.inode = (const uint4 *)tr->d_tab.ptr;
    t.grp = t.inode + tr->node_tab.size() / 4;
    t.pairs = t.grp + tr->grp_tab.size() / 4;
    t.n_q = (int32_t)tr->distinct.size();
    t.root_pairs = tr->root_pairs;
    t.root_q = tr->root_q;
    t.depth = tr->depth;
    t.kdepth = tr->kdepth;
    t.n_d = (int32_t)tr->deltas.size();
    return t;
}

template <typename TT>
TT delta_sat(int64_t delta) {
    return sizeof(TT) == 4 ? (TT)std::min<uint64_t>((uint64_t)delta, 0xffffffffull)
                           : (TT)(uint64_t)delta;
}

// Learned schedule + search on stream st: predicted segment costs -> items ->
// item-driven search kernel.
template <typename TT>
int learned_search(const mg_graph *g, mg_tree *tr, const mg_model *model,
                   const mg::KParams<TT> &base, int blocks, uint32_t stride, hipStream_t st) {
    const uint32_t E = (uint32_t)g->E;
    const uint32_t n_seg = (E + mg::kSeg - 1) / mg::kSeg;
    DevBuf d;
    const size_t off_total = 4 * (size_t)n_seg;
    const size_t off_work = off_total + 16;
    const size_t off_nitems = off_work + 4 * (size_t)mg::kBinWords;
    const size_t off_items = (off_nitems + 16 + 15) & ~(size_t)15;
    const size_t off_feat = (off_items + 8 * (size_t)std::max<uint32_t>(E, 1) + 15) & ~(size_t)15;
    const size_t off_skip = off_feat + 32 * (size_t)std::max<uint32_t>((E + stride - 1) / stride, 1);
    int rc = dev_alloc(d, off_skip + n_seg + 16, (void *)st);
    if (rc) return rc;
    struct G { DevBuf *b; ~G() { dev_free(*b); } } guard{&d};
    char *p0 = (char *)d.ptr;
    float *seg_cost = (float *)p0, *total = (float *)(p0 + off_total);
    uint32_t *work = (uint32_t *)(p0 + off_work), *n_items = (uint32_t *)(p0 + off_nitems);
    uint2 *items = (uint2 *)(p0 + off_items);
    uint4 *feat = (uint4 *)(p0 + off_feat);
    uint8_t *skip = (uint8_t *)(p0 + off_skip);
    hipError_t e = mg::launch_fill_f32_zero(total, 1, st);
    if (e == hipSuccess)
        e = mg::launch_predict_roots<TT>(base.g, base.tree, base.delta_sat,
                                         (const float *)model->params.ptr, stride, seg_cost, total,
                                         feat, st);
    // segments predicted at more than 8x the mean go first (one root per item
    // above ~1/(4 * resident waves) of the total, heavy roots in up to
    // kRootParts parts); the rest keep time order
    if (e == hipSuccess)
        e = mg::launch_bin(seg_cost, n_seg, E, total, 8.0f, 1.0f / 32768.0f, kRootParts, work,
                           items, std::max<uint32_t>(E, 1), n_items, skip, st);
    if (e != hipSuccess) return fail(MG_EDEVICE, "learned schedule failed: %s", hipGetErrorString(e));
    mg::KParams<TT> p = base;
    p.items = items;
    p.n_items = n_items;
    p.skip = skip;
    p.roots = nullptr;
    p.chunk = mg::kSeg;      // one chunk is one segment
    e = mg::launch_comine<TT>(p, blocks, st);
    if (e != hipSuccess) return fail(MG_EDEVICE, "co-mining launch failed: %s", hipGetErrorString(e));
    // the buffer is released after the caller synchronises the stream
    HIP_TRY(hipStreamSynchronize(st));
    return MG_OK;
}

}  // namespace

// ---------------------------------------------------------------- batches
constexpr uint32_t kBatchQueueWords = mg::kQueues * mg::kQueueStride;
constexpr uint32_t kBatchCtxWord = 8;      // in the first head's line: contexts handed on
constexpr uint32_t kBatchWaves = 4096;     // waves of a batch launch, about

struct mg_batch {
    std::vector<const mg_graph *> graphs;
    std::vector<mg_tree *> trees;
    int time_bytes = 4;
    int device = 0;
    int depth = 1;
    uint32_t n_q_max = 1;
    uint32_t total_q = 0;         // device counters (distinct motifs per job)
    int32_t total_motifs = 0;     // caller-visible counts
    int64_t total_roots = 0;
    std::vector<uint32_t> count_off;
    mg_batch_opts opts{};
    int32_t item_roots = 0;
    float tuned_ms = 0.f;
    float predict_ms = 0.f;       // features + MLP + ordering at plan creation
    bool learned = false;
    std::vector<mg::BatchItem> items;
    DevBuf d_jobs, d_items, d_work;   // d_work: item queue heads, then counters
    DevBuf d_ctx;                     // contexts a step hands on between its two launches
    uint64_t *h_counts = nullptr;     // pinned
    hipGraph_t graph = nullptr;
    hipGraphExec_t exec = nullptr;
    hipStream_t cap_stream = nullptr;
    ~mg_batch() {
        if (exec) (void)hipGraphExecDestroy(exec);
        if (graph) (void)hipGraphDestroy(graph);
        if (cap_stream) (void)hipStreamDestroy(cap_stream);
        if (h_counts) (void)hipHostFree(h_counts);
        dev_free(d_jobs);
        dev_free(d_items);
        dev_free(d_work);
        dev_free(d_ctx);
    }
};

namespace {

// The heavy chunks of a batch's job handed on as in a single count (launch_ds),
// with the batch's roots per wave.
template <typename TT>
void hand_on_to(mg::KParams<TT> &p, const mg_tree *tr, uint64_t total_roots, mg::EpochCtx *ctx,
                unsigned long long *ctx_count) {
    const bool deep = tr->depth > 3;
    p.hand_on = mg::hand_on_limit(total_roots, kBatchWaves, deep);
    p.ctx_piece = mg::hand_on_piece(deep);
    p.ctx_out = ctx;
    p.ctx_in = ctx;
    p.ctx_cap = kHandOnCap;
    p.ctx_count = ctx_count;
}

template <typename TT>
int upload_jobs(mg_batch *b, hipStream_t st) {
    std::vector<mg::BatchJob<TT>> jobs(b->graphs.size());
    mg_count_opts o;
    mg_count_opts_init(&o);
    for (size_t j = 0; j < jobs.size(); ++j) {
        mg::BatchJob<TT> &J = jobs[j];
        std::memset(&J, 0, sizeof J);
        fill_params<TT>(J.p, b->graphs[j], b->trees[j], o, nullptr, nullptr, nullptr, nullptr);
        J.count_off = b->count_off[j];
        J.p.job = (uint32_t)j;
        if (b->d_ctx.ptr && b->trees[j]->kdepth > 2)
            hand_on_to(J.p, b->trees[j], b->total_roots, (mg::EpochCtx *)b->d_ctx.ptr,
                       (unsigned long long *)b->d_work.ptr + kBatchCtxWord);
    }
    int rc = dev_alloc(b->d_jobs, sizeof(mg::BatchJob<TT>) * jobs.size(), (void *)st);
    if (rc) return rc;
    HIP_TRY(hipMemcpyAsync(b->d_jobs.ptr, jobs.data(), sizeof(mg::BatchJob<TT>) * jobs.size(),
                           hipMemcpyHostToDevice, st));
    return MG_OK;
}

// The searches of several trees over one graph (per-motif mode) as one batch per
// kernel depth, its items the chunks of the graph's roots, each for every tree
// in turn: the waves go from tree to tree without waiting for each other, and
// the roots' rows and lists are read from L2 by all trees but one.  Launched one
// after another, 36 searches of 1M edges filled and drained the device 72
// times: 4.23 ms, here 2.20 (of 20M edges: 35.5 ms, here 20.5).  Counters come back in `slots`, tree after tree; *taken stays false for
// more items than a batch can number.
template <typename TT>
int count_runs(const mg_graph *g, const std::vector<mg_tree *> &runs, const mg_count_opts &o,
               uint64_t *slots, bool *taken, hipStream_t st, float *ms) {
    const uint32_t E = (uint32_t)g->E;
    // about 16 items per wave, of at most 2048 roots (a claim on one queue head
    // takes about 20 ns)
    uint32_t len = 4;
    while (len < 2048 && (uint64_t)len * 16 * 2 * kBatchWaves < (uint64_t)E * runs.size()) len <<= 1;
    const uint32_t chunks = (E + len - 1) / len;
    if ((uint64_t)chunks * runs.size() >> 31) return MG_OK;
    std::vector<uint32_t> order(runs.size()), off(runs.size());
    std::iota(order.begin(), order.end(), 0u);
    std::stable_sort(order.begin(), order.end(),
                     [&](uint32_t a, uint32_t b) { return runs[a]->kdepth < runs[b]->kdepth; });
    uint32_t n_out = 0, depths = 0;
    for (size_t i = 0; i < runs.size(); ++i) {
        int rc = upload_tree(runs[i], g->device, st);
        if (rc) return rc;
        off[i] = n_out;
        n_out += (uint32_t)n_slots(runs[i]);
        depths += i == 0 || runs[order[i]]->kdepth != runs[order[i - 1]]->kdepth;
    }
    const bool deep = runs[order.back()]->kdepth > 2 && E >= kHandOnRoots;
    Scratch own;
    mg::BatchJob<TT> *d_jobs;
    unsigned long long *d_work;
    mg::EpochCtx *d_ctx = nullptr;
    int rc = own.get(&d_jobs, runs.size(), st);
    if (!rc) rc = own.get(&d_work, (size_t)depths * kBatchQueueWords + n_out, st);
    if (rc) return rc;
    if (deep) (void)own.get(&d_ctx, kHandOnCap, st);   // (NULL: nothing is handed on)
    unsigned long long *d_out = d_work + (size_t)depths * kBatchQueueWords;
    std::vector<mg::BatchJob<TT>> jobs(runs.size());
    for (size_t i = 0, at = 0, d = 0; i < runs.size(); ++i) {
        const mg_tree *t = runs[order[i]];
        if (i && t->kdepth != runs[order[i - 1]]->kdepth) at = i, ++d;
        mg::BatchJob<TT> &J = jobs[i];
        std::memset(&J, 0, sizeof J);
        fill_params<TT>(J.p, g, t, o, nullptr, nullptr, nullptr, nullptr);
        J.count_off = off[order[i]];
        J.p.job = (uint32_t)(i - at);
        if (d_ctx && t->kdepth > 2)
            hand_on_to(J.p, t, (uint64_t)E * runs.size(), d_ctx,
                       d_work + d * kBatchQueueWords + kBatchCtxWord);
    }
    HIP_TRY(hipMemcpyAsync(d_jobs, jobs.data(), sizeof(mg::BatchJob<TT>) * jobs.size(),
                           hipMemcpyHostToDevice, st));
    HIP_TRY(mg::launch_fill_u64(d_work, depths * kBatchQueueWords + n_out, 0ull, st));
    struct Events {
        hipEvent_t a = nullptr, b = nullptr;
        ~Events() {
            if (a) (void)hipEventDestroy(a);
            if (b) (void)hipEventDestroy(b);
        }
    } ev;
    if (ms) {
        HIP_TRY(hipEventCreate(&ev.a));
        HIP_TRY(hipEventCreate(&ev.b));
        HIP_TRY(hipEventRecord(ev.a, st));
    }
    for (size_t i = 0, d = 0; i < runs.size(); ++d) {
        const mg_tree *t = runs[order[i]];
        size_t end = i;
        mg::BatchParams<TT> bp{};
        for (; end < runs.size() && runs[order[end]]->kdepth == t->kdepth; ++end)
            bp.n_q_max = std::max<uint32_t>(bp.n_q_max, (uint32_t)n_slots(runs[order[end]]));
        bp.jobs = d_jobs + i;
        bp.n_jobs = (uint32_t)(end - i);
        bp.run_roots = len;
        bp.n_roots = E;
        bp.n_items = chunks * bp.n_jobs;
        bp.cursor = d_work + d * kBatchQueueWords;
        bp.counts = d_out;
        bp.multi = t->deltas.size() > 1 ? 1u : 0u;
        hipError_t e = mg::launch_batch<TT>(bp, t->kdepth, 0, st);
        if (e == hipSuccess && d_ctx && t->kdepth > 2) {
            bp.contexts = 1;
            bp.ctx = d_ctx;
            bp.ctx_n = bp.cursor + kBatchCtxWord;
            bp.ctx_cap = kHandOnCap;
            e = mg::launch_batch<TT>(bp, t->kdepth, 0, st);
        }
        if (e != hipSuccess)
            return fail(MG_EDEVICE, "per-motif launch failed: %s", hipGetErrorString(e));
        i = end;
    }
    if (ms) HIP_TRY(hipEventRecord(ev.b, st));
    HIP_TRY(hipMemcpyAsync(slots, d_out, 8 * (size_t)n_out, hipMemcpyDeviceToHost, st));
    HIP_TRY(hipStreamSynchronize(st));
    if (ms) HIP_TRY(hipEventElapsedTime(ms, ev.a, ev.b));
    *taken = true;
    return MG_OK;
}

// Work items: root ranges of item_roots roots, largest graphs first.
int make_items(mg_batch *b, int32_t item_roots, hipStream_t st) {
    std::vector<uint32_t> order(b->graphs.size());
    std::iota(order.begin(), order.end(), 0u);
    std::stable_sort(order.begin(), order.end(), [&](uint32_t x, uint32_t y) {
        return b->graphs[x]->E > b->graphs[y]->E;
    });
    b->items.clear();
    for (uint32_t j : order) {
        const uint32_t E = (uint32_t)b->graphs[j]->E;
        for (uint32_t r = 0; r < E; r += (uint32_t)item_roots)
            b->items.push_back({j, r, std::min<uint32_t>(E, r + (uint32_t)item_roots), 0u});
    }
    dev_free(b->d_items);
    int rc = dev_alloc(b->d_items, sizeof(mg::BatchItem) * std::max<size_t>(1, b->items.size()),
                       (void *)st);
    if (rc) return rc;
    if (!b->items.empty())
        HIP_TRY(hipMemcpyAsync(b->d_items.ptr, b->items.data(),
                               sizeof(mg::BatchItem) * b->items.size(), hipMemcpyHostToDevice, st));
    b->item_roots = item_roots;
    return MG_OK;
}

// Predicted segment costs of one job (learned_items orders the items).
template <typename TT>
int predict_job_segments(const mg_graph *g, mg_tree *tr, const mg_model *m, float *d_seg,
                         float *d_total, uint4 *d_feat, hipStream_t st) {
    hipError_t e = mg::launch_fill_f32_zero(d_total, 1, st);
    if (e == hipSuccess)
        e = mg::launch_predict_roots<TT>(dev_graph<TT>(g), dev_tree(tr), delta_sat<TT>(tr->delta),
                                         (const float *)m->params.ptr, kSampleDefault, d_seg,
                                         d_total, d_feat, st);
    if (e != hipSuccess) return fail(MG_EDEVICE, "cost prediction failed: %s", hipGetErrorString(e));
    return MG_OK;
}

int learned_items(mg_batch *b, const mg_model *m, hipStream_t st) {
    const auto t0 = std::chrono::steady_clock::now();
    struct Seg { float cost; uint32_t job, first, end; };
    std::vector<Seg> segs;
    double total = 0.0;
    for (size_t j = 0; j < b->graphs.size(); ++j) {
        const mg_graph *g = b->graphs[j];
        const uint32_t E = (uint32_t)g->E, n_seg = (E + mg::kSeg - 1) / mg::kSeg;
        if (!n_seg) continue;
        DevBuf d;
        const size_t off_feat = (4 * (size_t)n_seg + 16 + 15) & ~(size_t)15;
        int rc = dev_alloc(d, off_feat + 32 * (size_t)((E + kSampleDefault - 1) / kSampleDefault),
                           (void *)st);
        if (rc) return rc;
        struct G { DevBuf *b; ~G() { dev_free(*b); } } guard{&d};
        float *d_seg = (float *)d.ptr, *d_total = d_seg + n_seg;
        uint4 *d_feat = (uint4 *)((char *)d.ptr + off_feat);
        rc = b->time_bytes == 4
                 ? predict_job_segments<uint32_t>(g, b->trees[j], m, d_seg, d_total, d_feat, st)
                 : predict_job_segments<uint64_t>(g, b->trees[j], m, d_seg, d_total, d_feat, st);
        if (rc) return rc;
        std::vector<float> h(n_seg);
        HIP_TRY(hipMemcpyAsync(h.data(), d_seg, 4 * (size_t)n_seg, hipMemcpyDeviceToHost, st));
        HIP_TRY(hipStreamSynchronize(st));
        for (uint32_t sg = 0; sg < n_seg; ++sg) {
            const uint32_t r0 = sg * mg::kSeg;
            segs.push_back({h[sg], (uint32_t)j, r0, std::min<uint32_t>(E, r0 + mg::kSeg)});
            total += h[sg];
        }
    }
    int dev = 0, ncu = 0;
    HIP_TRY(hipGetDevice(&dev));
    HIP_TRY(hipDeviceGetAttribute(&ncu, hipDeviceAttributeMultiprocessorCount, dev));
    // heavy segments (above 8x the mean) first, heaviest first; one root per
    // item above a quarter of one wave's fair share (~32 resident waves per
    // CU), a root still above that in up to kRootParts parts of its
    // first-level candidates; then every other segment in job order (largest
    // graph first) and time order, as the plain schedule runs them
    const double split = total / (4.0 * 32.0 * std::max(ncu, 1));
    const double heavy = segs.empty() ? 0.0 : 8.0 * total / (double)segs.size();
    std::vector<std::pair<float, mg::BatchItem>> it;
    std::vector<uint8_t> is_heavy(segs.size(), 0);
    for (size_t i = 0; i < segs.size(); ++i) {
        const Seg &sg = segs[i];
        if (!(total > 0.0 && sg.cost > heavy)) continue;
        is_heavy[i] = 1;
        const uint32_t nr = sg.end - sg.first;
        if (sg.cost > split && nr > 1) {
            const double c = (double)sg.cost / nr;
            const uint32_t k =
                (uint32_t)std::min<double>(kRootParts, std::max(1.0, std::ceil(c / split)));
            for (uint32_t r = sg.first; r < sg.end; ++r)
                for (uint32_t q = 0; q < k; ++q)
                    it.push_back({(float)(c / k), {sg.job, r, r + 1,
                                                   k > 1 ? (mg::kItemSplit | (q << 15) | k) : 0u}});
        } else {
            it.push_back({sg.cost, {sg.job, sg.first, sg.end, 0u}});
        }
    }
    std::stable_sort(it.begin(), it.end(),
                     [](const auto &x, const auto &y) { return x.first > y.first; });
    std::vector<uint32_t> order(b->graphs.size());
    std::iota(order.begin(), order.end(), 0u);
    std::stable_sort(order.begin(), order.end(), [&](uint32_t x, uint32_t y) {
        return b->graphs[x]->E > b->graphs[y]->E;
    });
    std::vector<size_t> seg0(b->graphs.size() + 1, 0);   // first segment of each job
    for (const Seg &sg : segs) seg0[sg.job + 1]++;
    for (size_t j = 0; j < b->graphs.size(); ++j) seg0[j + 1] += seg0[j];
    for (uint32_t j : order)
        for (size_t i = seg0[j]; i < seg0[j + 1]; ++i)
            if (!is_heavy[i]) it.push_back({0.f, {j, segs[i].first, segs[i].end, 0u}});
    b->items.clear();
    for (auto &x : it) b->items.push_back(x.second);
    dev_free(b->d_items);
    int rc = dev_alloc(b->d_items, sizeof(mg::BatchItem) * std::max<size_t>(1, b->items.size()),
                       (void *)st);
    if (rc) return rc;
    if (!b->items.empty())
        HIP_TRY(hipMemcpyAsync(b->d_items.ptr, b->items.data(),
                               sizeof(mg::BatchItem) * b->items.size(), hipMemcpyHostToDevice, st));
    b->item_roots = mg::kSeg;
    b->learned = true;
    HIP_TRY(hipStreamSynchronize(st));
    b->predict_ms = std::chrono::duration<float, std::milli>(std::chrono::steady_clock::now() - t0).count();
    return MG_OK;
}

// Enqueue one step on st: zero, search, copy the counters to pinned memory.
template <typename TT>
int enqueue_step(mg_batch *b, hipStream_t st) {
    mg::BatchParams<TT> bp{};
    bp.jobs = (const mg::BatchJob<TT> *)b->d_jobs.ptr;
    bp.items = (const mg::BatchItem *)b->d_items.ptr;
    bp.n_items = (uint32_t)b->items.size();
    bp.n_q_max = b->n_q_max;
    bp.cursor = (unsigned long long *)b->d_work.ptr;
    bp.counts = bp.cursor + kBatchQueueWords;
    bp.multi = 0;
    for (const mg_tree *tr : b->trees) bp.multi |= tr->deltas.size() > 1 ? 1u : 0u;
    hipError_t e = mg::launch_fill_u64(bp.cursor, kBatchQueueWords + b->total_q, 0ull, st);
    if (e != hipSuccess) return fail(MG_EDEVICE, "fill launch failed: %s", hipGetErrorString(e));
    if (bp.n_items) {
        e = mg::launch_batch<TT>(bp, b->depth, b->opts.blocks, st);
        if (e == hipSuccess && b->d_ctx.ptr) {
            // the heaviest chunks' candidates, spread over the device
            bp.contexts = 1;
            bp.ctx = (const mg::EpochCtx *)b->d_ctx.ptr;
            bp.ctx_n = bp.cursor + kBatchCtxWord;
            bp.ctx_cap = kHandOnCap;
            e = mg::launch_batch<TT>(bp, b->depth, b->opts.blocks, st);
        }
        if (e != hipSuccess) return fail(MG_EDEVICE, "batch launch failed: %s", hipGetErrorString(e));
    }
    HIP_TRY(hipMemcpyAsync(b->h_counts, bp.counts, 8 * (size_t)std::max<uint32_t>(1, b->total_q),
                           hipMemcpyDeviceToHost, st));
    return MG_OK;
}

int run_step(mg_batch *b, hipStream_t st, float *ms) {
    hipEvent_t e0 = nullptr, e1 = nullptr;
    if (ms) {
        HIP_TRY(hipEventCreate(&e0));
        HIP_TRY(hipEventCreate(&e1));
        HIP_TRY(hipEventRecord(e0, st));
    }
    int rc;
    if (b->exec) {
        HIP_TRY(hipGraphLaunch(b->exec, st));
        rc = MG_OK;
    } else {
        rc = b->time_bytes == 4 ? enqueue_step<uint32_t>(b, st) : enqueue_step<uint64_t>(b, st);
    }
    if (rc) return rc;
    if (ms) {
        HIP_TRY(hipEventRecord(e1, st));
        HIP_TRY(hipEventSynchronize(e1));
        HIP_TRY(hipEventElapsedTime(ms, e0, e1));
        (void)hipEventDestroy(e0);
        (void)hipEventDestroy(e1);
    }
    HIP_TRY(hipStreamSynchronize(st));
    return MG_OK;
}

int capture(mg_batch *b) {
    if (!b->cap_stream) HIP_TRY(hipStreamCreateWithFlags(&b->cap_stream, hipStreamNonBlocking));
    HIP_TRY(hipStreamBeginCapture(b->cap_stream, hipStreamCaptureModeThreadLocal));
    int rc = b->time_bytes == 4 ? enqueue_step<uint32_t>(b, b->cap_stream)
                                : enqueue_step<uint64_t>(b, b->cap_stream);
    hipGraph_t gr = nullptr;
    hipError_t e = hipStreamEndCapture(b->cap_stream, &gr);
    if (rc) { if (gr) (void)hipGraphDestroy(gr); return rc; }
    if (e != hipSuccess) return fail(MG_EDEVICE, "graph capture failed: %s", hipGetErrorString(e));
    b->graph = gr;
    HIP_TRY(hipGraphInstantiate(&b->exec, gr, nullptr, nullptr, 0));
    return MG_OK;
}

}  // namespace

// ---------------------------------------------------------------- C ABI
extern "C" {

int mg_set_allocator(mg_alloc_fn alloc, mg_release_fn release, void *ctx) {
    if ((alloc == nullptr) != (release == nullptr))
        return fail(MG_EINVAL, "alloc and release must both be set or both be NULL");
    g_alloc = alloc;
    g_release = release;
    g_alloc_ctx = ctx;
    return MG_OK;
}

const char *mg_last_error(void) { return g_err.c_str(); }

int mg_model_create(uint64_t seed, mg_model **out) {
    try {
        if (!out) return fail(MG_EINVAL, "out is NULL");
        std::unique_ptr<mg_model> m(new (std::nothrow) mg_model);
        if (!m) return fail(MG_ENOMEM, "out of host memory");
        HIP_TRY(hipGetDevice(&m->device));
        std::vector<float> w(mg::kParams, 0.f);
        uint64_t s = seed;
        auto he = [&](int off, int fan_in, int rows, int cols) {
            const double sd = std::sqrt(2.0 / fan_in);
            for (int i = 0; i < rows * cols; ++i) w[off + i] = (float)(normal(s) * sd);
        };
        he(mg::kOffW1, mg::kFeat, mg::kFeat, mg::kHid);    // rows 16..31 stay zero
        he(mg::kOffW2, mg::kHid, mg::kHid, mg::kHid);
        he(mg::kOffW3, mg::kHid, mg::kHid, mg::kHid);
        he(mg::kOffW4, mg::kHid, 1, mg::kHid);
        for (DevBuf *b : {&m->params, &m->adam_m, &m->adam_v}) {
            int rc = dev_alloc(*b, sizeof(float) * mg::kParams, nullptr);
            if (rc) return rc;
        }
        HIP_TRY(hipMemcpy(m->params.ptr, w.data(), sizeof(float) * w.size(), hipMemcpyHostToDevice));
        HIP_TRY(hipMemset(m->adam_m.ptr, 0, sizeof(float) * mg::kParams));
        HIP_TRY(hipMemset(m->adam_v.ptr, 0, sizeof(float) * mg::kParams));
        *out = m.release();
        return MG_OK;
    } catch (...) {
        return fail(MG_EINTERNAL, "unexpected exception");
    }
}

int mg_model_get_weights(const mg_model *m, float *w) {
    if (!m || !w) return fail(MG_EINVAL, "NULL argument");
    HIP_TRY(hipMemcpy(w, m->params.ptr, sizeof(float) * mg::kParams, hipMemcpyDeviceToHost));
    return MG_OK;
}

int mg_model_set_weights(mg_model *m, const float *w) {
    if (!m || !w) return fail(MG_EINVAL, "NULL argument");
    for (int i = 0; i < mg::kParams; ++i)
        if (!std::isfinite(w[i])) return fail(MG_EINVAL, "weight %d is not finite", i);
    for (int r = mg::kFeat; r < 32; ++r)
        for (int c = 0; c < mg::kHid; ++c)
            if (w[mg::kOffW1 + r * mg::kHid + c] != 0.f)
                return fail(MG_EINVAL, "W1 rows %d..31 must be zero", mg::kFeat);
    HIP_TRY(hipMemcpy(m->params.ptr, w, sizeof(float) * mg::kParams, hipMemcpyHostToDevice));
    HIP_TRY(hipMemset(m->adam_m.ptr, 0, sizeof(float) * mg::kParams));
    HIP_TRY(hipMemset(m->adam_v.ptr, 0, sizeof(float) * mg::kParams));
    return MG_OK;
}

int mg_model_get_moments(const mg_model *m, float *m1, float *m2) {
    if (!m) return fail(MG_EINVAL, "NULL model");
    if (m1) HIP_TRY(hipMemcpy(m1, m->adam_m.ptr, sizeof(float) * mg::kParams, hipMemcpyDeviceToHost));
    if (m2) HIP_TRY(hipMemcpy(m2, m->adam_v.ptr, sizeof(float) * mg::kParams, hipMemcpyDeviceToHost));
    return MG_OK;
}

void mg_model_destroy(mg_model *m) { delete m; }

int mg_root_features(const mg_graph *g, const mg_tree *tr_c, const int64_t *roots, int64_t n,
                     float *feats) {
    try {
        if (!g || !tr_c || !feats || n < 0) return fail(MG_EINVAL, "bad argument");
        if (g->host_only) return fail(MG_EINVAL, "the graph is on the host only (MG_HOST_ONLY)");
        if (!roots && n != g->E) return fail(MG_EINVAL, "without roots, n must be n_edges");
        mg_tree *tr = const_cast<mg_tree *>(tr_c);
        int rc = upload_tree(tr, g->device, nullptr);
        if (rc) return rc;
        std::vector<uint32_t> r;
        if (roots) {
            r.resize(n);
            for (int64_t i = 0; i < n; ++i) {
                if (roots[i] < 0 || roots[i] >= g->E) return fail(MG_EINVAL, "root out of range");
                r[i] = (uint32_t)roots[i];
            }
        }
        DevBuf d_r, d_f;
        struct G { DevBuf *a, *b; ~G() { dev_free(*a); dev_free(*b); } } guard{&d_r, &d_f};
        if (roots) {
            rc = dev_alloc(d_r, 4 * std::max<size_t>(1, r.size()), nullptr);
            if (rc) return rc;
            if (n) HIP_TRY(hipMemcpy(d_r.ptr, r.data(), 4 * r.size(), hipMemcpyHostToDevice));
        }
        rc = dev_alloc(d_f, sizeof(float) * mg::kFeat * std::max<int64_t>(1, n), nullptr);
        if (rc) return rc;
        hipError_t e = g->time_bytes == 4
            ? mg::launch_features<uint32_t>(dev_graph<uint32_t>(g), dev_tree(tr),
                                            delta_sat<uint32_t>(tr->delta),
                                            (const uint32_t *)d_r.ptr, (uint32_t)n,
                                            (float *)d_f.ptr, nullptr)
            : mg::launch_features<uint64_t>(dev_graph<uint64_t>(g), dev_tree(tr),
                                            delta_sat<uint64_t>(tr->delta),
                                            (const uint32_t *)d_r.ptr, (uint32_t)n,
                                            (float *)d_f.ptr, nullptr);
        if (e != hipSuccess) return fail(MG_EDEVICE, "features launch failed: %s", hipGetErrorString(e));
        if (n) HIP_TRY(hipMemcpy(feats, d_f.ptr, sizeof(float) * mg::kFeat * n, hipMemcpyDeviceToHost));
        return MG_OK;
    } catch (...) {
        return fail(MG_EINTERNAL, "unexpected exception");
    }
}

int mg_model_predict(const mg_model *m, const float *feats, int64_t n, float *out) {
    try {
        if (!m || !feats || !out || n < 0 || n >= (int64_t)1 << 31)
            return fail(MG_EINVAL, "bad argument");
        DevBuf d_f, d_o;
        struct G { DevBuf *a, *b; ~G() { dev_free(*a); dev_free(*b); } } guard{&d_f, &d_o};
        int rc = dev_alloc(d_f, sizeof(float) * mg::kFeat * std::max<int64_t>(1, n), nullptr);
        if (rc) return rc;
        rc = dev_alloc(d_o, sizeof(float) * std::max<int64_t>(1, n), nullptr);
        if (rc) return rc;
        if (n) HIP_TRY(hipMemcpy(d_f.ptr, feats, sizeof(float) * mg::kFeat * n, hipMemcpyHostToDevice));
        hipError_t e = mg::launch_predict_feats((const float *)m->params.ptr, (const float *)d_f.ptr,
                                                (uint32_t)n, (float *)d_o.ptr, nullptr);
        if (e != hipSuccess) return fail(MG_EDEVICE, "predict launch failed: %s", hipGetErrorString(e));
        if (n) HIP_TRY(hipMemcpy(out, d_o.ptr, sizeof(float) * n, hipMemcpyDeviceToHost));
        return MG_OK;
    } catch (...) {
        return fail(MG_EINTERNAL, "unexpected exception");
    }
}

int mg_model_train(mg_model *m, const float *feats, const float *labels, int64_t n,
                   int32_t epochs, float lr, uint64_t seed, float *loss) {
    try {
        if (!m || !feats || !labels || n < 0 || n >= (int64_t)1 << 31 || epochs < 0 ||
            !(lr > 0.f))
            return fail(MG_EINVAL, "bad argument");
        std::vector<uint32_t> perm(n);
        std::iota(perm.begin(), perm.end(), 0u);
        uint64_t s = seed;
        for (int64_t i = n - 1; i > 0; --i) std::swap(perm[i], perm[splitmix(s) % (uint64_t)(i + 1)]);
        DevBuf d_f, d_y, d_p, d_l;
        struct G {
            DevBuf *a, *b, *c, *d;
            ~G() { dev_free(*a); dev_free(*b); dev_free(*c); dev_free(*d); }
        } guard{&d_f, &d_y, &d_p, &d_l};
        int rc = dev_alloc(d_f, sizeof(float) * mg::kFeat * std::max<int64_t>(1, n), nullptr);
        if (!rc) rc = dev_alloc(d_y, sizeof(float) * std::max<int64_t>(1, n), nullptr);
        if (!rc) rc = dev_alloc(d_p, sizeof(uint32_t) * std::max<int64_t>(1, n), nullptr);
        if (!rc) rc = dev_alloc(d_l, sizeof(float) * std::max(1, epochs), nullptr);
        if (rc) return rc;
        if (n) {
            HIP_TRY(hipMemcpy(d_f.ptr, feats, sizeof(float) * mg::kFeat * n, hipMemcpyHostToDevice));
            HIP_TRY(hipMemcpy(d_y.ptr, labels, sizeof(float) * n, hipMemcpyHostToDevice));
            HIP_TRY(hipMemcpy(d_p.ptr, perm.data(), sizeof(uint32_t) * n, hipMemcpyHostToDevice));
        }
        hipError_t e = mg::launch_train((float *)m->params.ptr, (float *)m->adam_m.ptr,
                                        (float *)m->adam_v.ptr, (const float *)d_f.ptr,
                                        (const float *)d_y.ptr, (uint32_t)n,
                                        (const uint32_t *)d_p.ptr, (uint32_t)epochs, lr,
                                        (float *)d_l.ptr, nullptr);
        if (e != hipSuccess) return fail(MG_EDEVICE, "train launch failed: %s", hipGetErrorString(e));
        HIP_TRY(hipDeviceSynchronize());
        if (loss && epochs)
            HIP_TRY(hipMemcpy(loss, d_l.ptr, sizeof(float) * epochs, hipMemcpyDeviceToHost));
        return MG_OK;
    } catch (...) {
        return fail(MG_EINTERNAL, "unexpected exception");
    }
}

void mg_batch_opts_init(mg_batch_opts *o) {
    if (!o) return;
    std::memset(o, 0, sizeof *o);
    o->use_graph = 1;
}

int mg_batch_create(const mg_graph *const *graphs, const mg_tree *const *trees, int32_t n,
                    const mg_batch_opts *opts, mg_batch **out) {
    try {
        if (!out || !graphs || !trees || n < 1) return fail(MG_EINVAL, "empty batch");
        mg_batch_opts o;
        mg_batch_opts_init(&o);
        if (opts) o = *opts;
        if (o.item_roots < 0 || o.item_roots % 64 || o.item_roots > (1 << 24))
            return fail(MG_EINVAL, "item_roots must be a multiple of 64 in [0, 2^24]");
        int dev = 0;
        HIP_TRY(hipGetDevice(&dev));
        if (o.model && o.model->device != dev) return fail(MG_EINVAL, "model on another device");
        std::unique_ptr<mg_batch> b(new (std::nothrow) mg_batch);
        if (!b) return fail(MG_ENOMEM, "out of host memory");
        b->opts = o;
        b->device = dev;
        hipStream_t st = (hipStream_t)o.stream;
        for (int32_t j = 0; j < n; ++j) {
            if (!graphs[j] || !trees[j]) return fail(MG_EINVAL, "job %d has a NULL handle", j);
            if (graphs[j]->host_only) return fail(MG_EINVAL, "job %d: graph on the host only", j);
            if (graphs[j]->device != dev) return fail(MG_EINVAL, "job %d: graph on another device", j);
            if (j && graphs[j]->time_bytes != graphs[0]->time_bytes)
                return fail(MG_EUNSUPPORTED, "graphs of one batch must share the time width");
            mg_tree *tr = const_cast<mg_tree *>(trees[j]);
            int rc = upload_tree(tr, dev, st);
            if (rc) return rc;
            b->graphs.push_back(graphs[j]);
            b->trees.push_back(tr);
            b->count_off.push_back(b->total_q);
            b->total_q += (uint32_t)n_slots(tr);
            b->total_motifs += tr->n_motifs * (int32_t)tr->delta_slot.size();
            b->total_roots += graphs[j]->E;
            b->n_q_max = std::max<uint32_t>(b->n_q_max, (uint32_t)n_slots(tr));
            b->depth = std::max(b->depth, tr->kdepth);
        }
        b->time_bytes = graphs[0]->time_bytes;
        int rc = dev_alloc(b->d_work, 8 * (size_t)(kBatchQueueWords + std::max<uint32_t>(1, b->total_q)),
                           (void *)st);
        if (rc) return rc;
        if (b->depth > 2 && b->total_roots >= kHandOnRoots)   // (without it nothing is handed on)
            (void)dev_alloc(b->d_ctx, sizeof(mg::EpochCtx) * kHandOnCap, (void *)st);
        rc = b->time_bytes == 4 ? upload_jobs<uint32_t>(b.get(), st)
                                : upload_jobs<uint64_t>(b.get(), st);
        if (rc) return rc;
        HIP_TRY(hipHostMalloc((void **)&b->h_counts, 8 * (size_t)std::max<uint32_t>(1, b->total_q),
                              hipHostMallocDefault));
        if (o.model) {
            rc = learned_items(b.get(), o.model, st);
            if (rc) return rc;
        } else if (o.item_roots > 0) {
            rc = make_items(b.get(), o.item_roots, st);
            if (rc) return rc;
        } else {
            // autotune the item size: one timed step per candidate, from small
            // to large, stopping at the first one that is clearly slower
            float best = -1.f;
            int32_t best_ir = 64;
            bool warm = false;
            for (int32_t ir : {64, 128, 256, 512, 1024}) {
                rc = make_items(b.get(), ir, st);
                if (rc) return rc;
                if (!warm) {
                    rc = run_step(b.get(), st, nullptr);
                    if (rc) return rc;
                    warm = true;
                }
                float ms = 0.f;
                rc = run_step(b.get(), st, &ms);
                if (rc) return rc;
                if (best < 0.f || ms < best) { best = ms; best_ir = ir; }
                else if (ms > 1.05f * best) break;
            }
            b->tuned_ms = best;
            if (b->item_roots != best_ir) {
                rc = make_items(b.get(), best_ir, st);
                if (rc) return rc;
            }
        }
        HIP_TRY(hipStreamSynchronize(st));
        *out = b.release();
        return MG_OK;
    } catch (const std::bad_alloc &) {
        return fail(MG_ENOMEM, "out of host memory");
    } catch (...) {
        return fail(MG_EINTERNAL, "unexpected exception");
    }
}

int mg_batch_count(mg_batch *b, uint64_t *counts, float *elapsed_ms) {
    try {
        if (!b || !counts) return fail(MG_EINVAL, "NULL argument");
        int dev = 0;
        HIP_TRY(hipGetDevice(&dev));
        if (dev != b->device) return fail(MG_EINVAL, "batch lives on device %d", b->device);
        hipStream_t st = (hipStream_t)b->opts.stream;
        int rc;
        if (b->opts.use_graph && !b->exec) {
            rc = capture(b);
            if (rc) return rc;
        }
        rc = run_step(b, st, elapsed_ms);
        if (rc) return rc;
        size_t k = 0;
        for (size_t j = 0; j < b->trees.size(); ++j) {
            const mg_tree *tr = b->trees[j];
            map_counts(tr, b->h_counts + b->count_off[j], counts + k);
            k += (size_t)tr->n_motifs * tr->delta_slot.size();
        }
        return MG_OK;
    } catch (...) {
        return fail(MG_EINTERNAL, "unexpected exception");
    }
}

int mg_batch_info(const mg_batch *b, mg_batch_info_t *out) {
    if (!b || !out) return fail(MG_EINVAL, "NULL argument");
    out->n_jobs = (int32_t)b->trees.size();
    out->total_motifs = b->total_motifs;
    out->total_roots = b->total_roots;
    out->n_items = (int64_t)b->items.size();
    out->item_roots = b->item_roots;
    out->blocks = b->opts.blocks;
    out->graph_captured = b->exec ? 1 : 0;
    out->depth = b->depth;
    out->tuned_ms = b->tuned_ms;
    out->learned = b->learned ? 1 : 0;
    out->predict_ms = b->predict_ms;
    return MG_OK;
}

void mg_batch_destroy(mg_batch *b) { delete b; }

int mg_count_batch(const mg_graph *const *graphs, const mg_tree *const *trees, int32_t n,
                   const mg_batch_opts *opts, uint64_t *counts) {
    if (!counts) return fail(MG_EINVAL, "NULL counts");
    mg_batch_opts o;
    mg_batch_opts_init(&o);
    if (opts) o = *opts;
    o.use_graph = 0;
    if (o.item_roots == 0) o.item_roots = 64;
    mg_batch *b = nullptr;
    int rc = mg_batch_create(graphs, trees, n, &o, &b);
    if (rc) return rc;
    rc = mg_batch_count(b, counts, nullptr);
    mg_batch_destroy(b);
    return rc;
}

int mg_graph_create(const int32_t *src, const int32_t *dst, const int64_t *t, int64_t n_edges,
                    int32_t n_nodes, uint32_t flags, void *stream, mg_graph **out) {
    try {
        if (!out) return fail(MG_EINVAL, "out is NULL");
        if (n_edges < 0 || n_nodes < 0) return fail(MG_EINVAL, "negative size");
        if (n_edges > 0 && (!src || !dst || !t)) return fail(MG_EINVAL, "NULL edge array");
        if (n_edges >= (int64_t)1 << 31)
            return fail(MG_EUNSUPPORTED, "n_edges %lld >= 2^31", (long long)n_edges);
        if (n_nodes >= INT32_MAX) return fail(MG_EUNSUPPORTED, "n_nodes too large");
        if (flags & ~(MG_SORTED_BY_T | MG_DEVICE_INPUT | MG_HOST_ONLY))
            return fail(MG_EINVAL, "unknown flags");
        if ((flags & MG_DEVICE_INPUT) && (flags & MG_HOST_ONLY))
            return fail(MG_EINVAL, "MG_DEVICE_INPUT and MG_HOST_ONLY exclude each other");
        hipStream_t st = (hipStream_t)stream;
        const bool on_device = (flags & MG_DEVICE_INPUT) && n_edges > 0;
        // what the arrays hold: the first bad edge, order, self-loops, times
        int64_t bad = -1, loops = 0, t_min = 0, t_max = 0;
        bool sorted = true;
        if (on_device) {
            DevBuf d_f;
            struct G { DevBuf *b; ~G() { dev_free(*b); } } guard{&d_f};
            int rc = dev_alloc(d_f, sizeof(mg::EdgeFacts), stream);
            if (rc) return rc;
            LAUNCH_TRY(mg::launch_edge_facts(src, dst, t, (uint32_t)n_edges, n_nodes,
                                             (mg::EdgeFacts *)d_f.ptr, st));
            mg::EdgeFacts f;
            HIP_TRY(hipMemcpyAsync(&f, d_f.ptr, sizeof f, hipMemcpyDeviceToHost, st));
            HIP_TRY(hipStreamSynchronize(st));
            bad = f.first_bad == ~0ull ? -1 : (int64_t)f.first_bad;
            sorted = f.unsorted == 0;
            loops = (int64_t)f.loops;
            t_min = mg::unbias_time(f.t_min);
            t_max = mg::unbias_time(f.t_max);
        } else if (n_edges > 0) {
            std::mutex mu;
            t_min = t_max = t[0];
            parallel_for(n_edges, [&](int64_t i0, int64_t i1) {
                int64_t b = -1, l = 0, lo = t[i0 < n_edges ? i0 : 0], hi = lo;
                bool so = true;
                for (int64_t i = i0; i < i1; ++i) {
                    if (b < 0 && (src[i] < 0 || src[i] >= n_nodes || dst[i] < 0 || dst[i] >= n_nodes))
                        b = i;
                    l += src[i] == dst[i];
                    so = so && (i == 0 || t[i] >= t[i - 1]);
                    lo = std::min(lo, t[i]);
                    hi = std::max(hi, t[i]);
                }
                std::lock_guard<std::mutex> lock(mu);
                if (b >= 0 && (bad < 0 || b < bad)) bad = b;
                loops += l;
                sorted = sorted && so;
                if (i1 > i0) { t_min = std::min(t_min, lo); t_max = std::max(t_max, hi); }
            });
        }
        if (bad >= 0)
            return fail(MG_EINVAL, "edge %lld has a vertex outside [0, %d)", (long long)bad, n_nodes);
        if ((flags & MG_SORTED_BY_T) && !sorted)
            return fail(MG_EINVAL, "MG_SORTED_BY_T given but t is not non-decreasing");
        if ((uint64_t)t_max - (uint64_t)t_min >= 1ull << 63)
            return fail(MG_EUNSUPPORTED, "time span >= 2^63");
        std::unique_ptr<mg_graph> g(new (std::nothrow) mg_graph);
        if (!g) return fail(MG_ENOMEM, "out of host memory");
        g->E = n_edges;
        g->V = n_nodes;
        g->self_loops = loops;
        g->t_min = t_min;
        g->t_max = t_max;
        g->time_bytes = (uint64_t)t_max - (uint64_t)t_min < 0xffffffffull ? 4 : 8;
        if (flags & MG_HOST_ONLY) {
            std::vector<int32_t> s(n_edges), d(n_edges);
            std::vector<int64_t> tt(n_edges);
            if (sorted) {
                std::copy(src, src + n_edges, s.begin());
                std::copy(dst, dst + n_edges, d.begin());
                std::copy(t, t + n_edges, tt.begin());
            } else {
                std::vector<int64_t> ord(n_edges);
                std::iota(ord.begin(), ord.end(), 0);
                std::stable_sort(ord.begin(), ord.end(),
                                 [&](int64_t a, int64_t b) { return t[a] < t[b]; });
                for (int64_t i = 0; i < n_edges; ++i) {
                    s[i] = src[ord[i]]; d[i] = dst[ord[i]]; tt[i] = t[ord[i]];
                }
            }
            g->host_only = true;
            g->device = -1;
            build_host(g.get(), std::move(s), std::move(d), std::move(tt));
            *out = g.release();
            return MG_OK;
        }
        HIP_TRY(hipGetDevice(&g->device));
        Scratch in;   // the input on the device
        if (!on_device && n_edges > 0) {
            int64_t *dt;
            int rc = in.get(&dt, 2 * (size_t)n_edges, st);
            if (rc) return rc;
            int32_t *ds = (int32_t *)(dt + n_edges), *dd = ds + n_edges;
            HIP_TRY(hipMemcpyAsync(ds, src, 4 * (size_t)n_edges, hipMemcpyHostToDevice, st));
            HIP_TRY(hipMemcpyAsync(dd, dst, 4 * (size_t)n_edges, hipMemcpyHostToDevice, st));
            HIP_TRY(hipMemcpyAsync(dt, t, 8 * (size_t)n_edges, hipMemcpyHostToDevice, st));
            src = ds;
            dst = dd;
            t = dt;
        }
        int rc = g->time_bytes == 4 ? ingest_graph<uint32_t>(g.get(), src, dst, t, sorted, in, st)
                                    : ingest_graph<uint64_t>(g.get(), src, dst, t, sorted, in, st);
        if (rc) return rc;
        *out = g.release();
        return MG_OK;
    } catch (const std::bad_alloc &) {
        return fail(MG_ENOMEM, "out of host memory");
    } catch (...) {
        return fail(MG_EINTERNAL, "unexpected exception");
    }
}

int mg_graph_info(const mg_graph *g, mg_graph_info_t *out) {
    if (!g || !out) return fail(MG_EINVAL, "NULL argument");
    out->n_edges = g->E;
    out->n_nodes = g->V;
    out->self_loops = g->self_loops;
    out->t_min = g->t_min;
    out->t_max = g->t_max;
    out->time_bytes = g->time_bytes;
    out->device_bytes = g->device_bytes;
    return MG_OK;
}

void mg_graph_destroy(mg_graph *g) { delete g; }

int mg_tree_create(const int32_t *motif_uv, const int32_t *motif_k, int32_t n_motifs,
                   int64_t delta, mg_tree **out) {
    return mg_tree_create_multi(motif_uv, motif_k, n_motifs, &delta, 1, out);
}

int mg_tree_create_multi(const int32_t *motif_uv, const int32_t *motif_k, int32_t n_motifs,
                         const int64_t *deltas, int32_t n_deltas, mg_tree **out) {
    try {
        if (!out) return fail(MG_EINVAL, "out is NULL");
        if (n_motifs < 1 || !motif_uv || !motif_k) return fail(MG_EINVAL, "no motifs");
        if (!deltas || n_deltas < 1) return fail(MG_EINVAL, "no window");
        if (n_deltas > MG_MAX_DELTAS)
            return fail(MG_EUNSUPPORTED, "%d windows (limit %d)", n_deltas, MG_MAX_DELTAS);
        for (int32_t i = 0; i < n_deltas; ++i)
            if (deltas[i] < 0) return fail(MG_EINVAL, "delta < 0");
        std::vector<Motif> canon(n_motifs);
        int64_t off = 0;
        for (int32_t i = 0; i < n_motifs; ++i) {
            const int k = motif_k[i];
            if (k < 1) return fail(MG_EINVAL, "motif %d has %d edges", i, k);
            if (k > kKMax)
                return fail(MG_EUNSUPPORTED, "motif %d has %d edges (limit %d)", i, k, kKMax);
            int rc = canonical(motif_uv + 2 * off, k, canon[i]);
            if (rc) return rc;
            off += k;
        }
        return make_tree(canon, std::vector<int64_t>(deltas, deltas + n_deltas), out);
    } catch (const std::bad_alloc &) {
        return fail(MG_ENOMEM, "out of host memory");
    } catch (...) {
        return fail(MG_EINTERNAL, "unexpected exception");
    }
}

int mg_tree_info(const mg_tree *tr, mg_tree_info_t *out) {
    if (!tr || !out) return fail(MG_EINVAL, "NULL argument");
    *out = tr->info;
    return MG_OK;
}

void mg_tree_destroy(mg_tree *tr) { delete tr; }

}  // extern "C"

namespace {

// mg_enumerate and mg_enumerate_arrays: records in `out`, or motif indices in
// `motif` and edges in `edges`.
int enumerate(const mg_graph *g, const mg_tree *tr_c, void *stream, mg_match *out, int32_t *motif,
              int32_t *edges, int64_t capacity, int64_t *n_matches) {
    const bool arrays = motif && edges;
    try {
        if (!g || !tr_c || !n_matches || capacity < 0) return fail(MG_EINVAL, "bad argument");
        if (g->host_only) return fail(MG_EINVAL, "the graph is on the host only (MG_HOST_ONLY)");
        mg_tree *tr = const_cast<mg_tree *>(tr_c);
        if (tr->deltas.size() != 1)
            return fail(MG_EUNSUPPORTED, "enumeration takes a tree with one window");
        static_assert(sizeof(mg_match) == 4 * (1 + mg::kKMax), "record layout");
        std::vector<int32_t> first(tr->distinct.size(), -1);   // first caller motif per distinct one
        for (int32_t m = 0; m < tr->n_motifs; ++m)
            if (first[tr->motif_q[m]] < 0) first[tr->motif_q[m]] = m;
        mg_count_opts o;
        mg_count_opts_init(&o);
        o.stream = stream;
        mg_count_opts all = o;
        all.leaf_scan = -1;   // every match goes through the candidate expansion
        // The count sizes the output, unless the caller's own capacity is small
        // enough to be taken as it is and there is memory for it: then the search
        // writes into that much, and a count follows only if it was too little.
        constexpr uint64_t kDirectBytes = 256u << 20;
        hipStream_t st = (hipStream_t)stream;
        DevBuf d_work, d_rec;
        struct G { DevBuf *a, *b; ~G() { dev_free(*a); dev_free(*b); } } guard{&d_work, &d_rec};
        bool direct = (out || arrays) && capacity > 0 && (uint64_t)capacity * sizeof(mg_match) <= kDirectBytes;
        uint64_t room = 0, total = 0;
        auto count_all = [&]() -> int {
            std::vector<uint64_t> cnt(tr->n_motifs);
            int rc = mg_count(g, tr, &o, cnt.data());
            if (rc) return rc;
            total = 0;
            for (size_t q = 0; q < first.size(); ++q) total += cnt[first[q]];
            return MG_OK;
        };
        if (direct) {
            int dev = 0;
            HIP_TRY(hipGetDevice(&dev));
            if (dev != g->device)
                return fail(MG_EINVAL, "graph lives on device %d, current is %d", g->device, dev);
            int rc = upload_tree(tr, dev, st);
            if (rc) return rc;
            room = (uint64_t)capacity;
            direct = dev_alloc(d_rec, sizeof(mg_match) * room, (void *)st) == MG_OK;
        }
        if (!direct) {
            int rc = count_all();
            if (rc) return rc;
            if (!(out || arrays) || (uint64_t)capacity < total) {
                *n_matches = (int64_t)total;
                return MG_OK;
            }
            room = total;
            rc = dev_alloc(d_rec, sizeof(mg_match) * std::max<uint64_t>(room, 1), (void *)st);
            if (rc) return rc;
        }
        const size_t cnt_off = kQueueBytes, cur_off = cnt_off + 8 * n_slots(tr), first_off = cur_off + 8;
        int rc = dev_alloc(d_work, first_off + 4 * first.size(), (void *)st);
        if (rc) return rc;
        unsigned long long *w = (unsigned long long *)d_work.ptr;
        HIP_TRY(mg::launch_fill_u64(w, (uint32_t)(first_off / 8), 0ull, st));
        hipError_t e = hipSuccess;
        if (g->E > 0) {
            if (g->time_bytes == 4) {
                mg::KParams<uint32_t> p{};
                fill_params<uint32_t>(p, g, tr, all, w, w + cnt_off / 8, nullptr, nullptr);
                p.enum_out = (int32_t *)d_rec.ptr;
                p.enum_cursor = w + cur_off / 8;
                p.enum_cap = room;
                e = mg::launch_comine<uint32_t>(p, 0, st);
            } else {
                mg::KParams<uint64_t> p{};
                fill_params<uint64_t>(p, g, tr, all, w, w + cnt_off / 8, nullptr, nullptr);
                p.enum_out = (int32_t *)d_rec.ptr;
                p.enum_cursor = w + cur_off / 8;
                p.enum_cap = room;
                e = mg::launch_comine<uint64_t>(p, 0, st);
            }
        }
        if (e != hipSuccess) return fail(MG_EDEVICE, "enumeration launch failed: %s", hipGetErrorString(e));
        // the search's own counters, then the records written
        std::vector<uint64_t> h(n_slots(tr) + 1);
        HIP_TRY(hipMemcpyAsync(h.data(), w + cnt_off / 8, 8 * h.size(), hipMemcpyDeviceToHost, st));
        HIP_TRY(hipStreamSynchronize(st));
        const uint64_t written = h.back();
        if (direct && written > room) {
            dev_free(d_rec);
            rc = count_all();
            if (rc) return rc;
            if (total <= room)
                return fail(MG_EINTERNAL, "enumeration found more than %llu matches, the count is %llu",
                            (unsigned long long)room, (unsigned long long)total);
            *n_matches = (int64_t)total;
            return MG_OK;
        }
        const uint64_t counted = std::accumulate(h.begin(), h.end() - 1, (uint64_t)0);
        if (direct) total = counted;
        if (written != total || counted != total)
            return fail(MG_EINTERNAL, "enumeration wrote %llu matches, the count is %llu",
                        (unsigned long long)written, (unsigned long long)total);
        if (total) {
            // motifs in the caller's numbering (a duplicate's first occurrence),
            // edges in the caller's input order
            HIP_TRY(hipMemcpyAsync((char *)d_work.ptr + first_off, first.data(), 4 * first.size(),
                                   hipMemcpyHostToDevice, st));
            const int32_t *d_first = (const int32_t *)((char *)d_work.ptr + first_off);
            const uint32_t *order = (const uint32_t *)g->order.ptr;
            int32_t *rec = (int32_t *)d_rec.ptr;
            if (arrays) {
                // split into two arrays a piece at a time, so that the records need
                // no second copy of themselves (a piece: 96 MiB)
                constexpr uint64_t kPiece = 1u << 22;
                const uint64_t most = std::min(total, kPiece);
                Scratch split;
                int32_t *d_m, *d_e;
                rc = split.get(&d_m, most, st);
                if (!rc) rc = split.get(&d_e, mg::kKMax * most, st);
                if (rc) return rc;
                for (uint64_t i = 0; i < total; i += most) {
                    const uint64_t n = std::min(total - i, most);
                    HIP_TRY(mg::launch_map_matches(rec + i * (1 + mg::kKMax), n, d_first, order, d_m,
                                                   d_e, st));
                    HIP_TRY(hipMemcpyAsync(motif + i, d_m, 4 * n, hipMemcpyDeviceToHost, st));
                    HIP_TRY(hipMemcpyAsync(edges + i * mg::kKMax, d_e, 4 * mg::kKMax * n,
                                           hipMemcpyDeviceToHost, st));
                }
                HIP_TRY(hipStreamSynchronize(st));
            } else {
                HIP_TRY(mg::launch_map_matches(rec, total, d_first, order, nullptr, nullptr, st));
                HIP_TRY(hipMemcpyAsync(out, rec, sizeof(mg_match) * total, hipMemcpyDeviceToHost, st));
                HIP_TRY(hipStreamSynchronize(st));
            }
        }
        *n_matches = (int64_t)total;
        return MG_OK;
    } catch (const std::bad_alloc &) {
        return fail(MG_ENOMEM, "out of host memory");
    } catch (...) {
        return fail(MG_EINTERNAL, "unexpected exception");
    }
}

}  // namespace

extern "C" {

int mg_enumerate(const mg_graph *g, const mg_tree *tr, void *stream, mg_match *out,
                 int64_t capacity, int64_t *n_matches) {
    return enumerate(g, tr, stream, out, nullptr, nullptr, capacity, n_matches);
}

int mg_enumerate_arrays(const mg_graph *g, const mg_tree *tr, void *stream, int32_t *motif,
                        int32_t *edges, int64_t capacity, int64_t *n_matches) {
    if ((motif == nullptr) != (edges == nullptr))
        return fail(MG_EINVAL, "motif and edges must both be given or both be NULL");
    return enumerate(g, tr, stream, nullptr, motif, edges, capacity, n_matches);
}

int mg_count_noalloc(const mg_graph *g, const mg_tree *tr, const mg_count_opts *opts,
                     uint64_t *counts) {
    try {
        if (!g || !tr || !counts) return fail(MG_EINVAL, "NULL argument");
        if (g->host_only) return fail(MG_EINVAL, "the graph is on the host only (MG_HOST_ONLY)");
        mg_count_opts o;
        mg_count_opts_init(&o);
        if (opts) o = *opts;
        if (o.mode != MG_MODE_COMINE || o.sched != MG_SCHED_PLAIN || o.roots || o.root_cost ||
            o.elapsed_ms || o.cursor || o.wave_clock || o.epoch_idle)
            return fail(MG_EINVAL, "mg_count_noalloc takes co-mining with the plain schedule over "
                                   "every root; roots, root_cost, elapsed_ms, cursor and epochs "
                                   "need memory");
        if (o.chunk < 0 || (o.chunk % 64) != 0 || o.chunk > (1 << 16))
            return fail(MG_EINVAL, "chunk must be a multiple of 64 in [0, 65536]");
        if (o.queues < 0 || o.queues > mg::kQueues)
            return fail(MG_EINVAL, "queues must be in [0, %d]", mg::kQueues);
        if (o.max_chunks < 0 || o.max_chunks > 0xffffffffll)
            return fail(MG_EINVAL, "max_chunks must be in [0, 2^32)");
        const size_t nq = n_slots(tr);
        if (nq > (size_t)mg::kMaxQueries)
            return fail(MG_EUNSUPPORTED, "%zu counters; the static array holds %d", nq,
                        mg::kMaxQueries);
        int dev = 0;
        HIP_TRY(hipGetDevice(&dev));
        if (dev != g->device) return fail(MG_EINVAL, "graph lives on device %d, current is %d",
                                          g->device, dev);
        if (tr->device != dev || !tr->d_tab.ptr)
            return fail(MG_EINVAL, "the tree has no device tables on device %d yet (count it "
                                   "with mg_count there once)", dev);
        hipStream_t st = (hipStream_t)o.stream;
        if (!o.stats && !o.stop && !o.max_chunks) {
            uint64_t h[mg::kMaxQueries];
            int rc = MG_OK;
            if (g->time_bytes == 4 ? small_count<uint32_t>(g, tr, o, false, h, st, &rc)
                                   : small_count<uint64_t>(g, tr, o, false, h, st, &rc)) {
                if (!rc) map_counts(tr, h, counts);
                return rc;
            }
        }
        unsigned long long *scr = nullptr;
        HIP_TRY(mg::static_scratch(&scr));
        unsigned long long *d_queues = scr;
        unsigned long long *d_counts = scr + mg::kQueueWords;
        unsigned long long *d_stats = o.stats ? d_counts + mg::kMaxQueries : nullptr;
        // queue heads, claim counter, counters and statistics start at zero
        // (a fill kernel, no memset node if the caller captures the stream)
        HIP_TRY(mg::launch_fill_u64(scr, (uint32_t)mg::kStaticWords, 0ull, st));
        const uint32_t n_roots = (uint32_t)g->E;
        if (n_roots > 0) {
            hipError_t e;
            if (g->time_bytes == 4) {
                mg::KParams<uint32_t> p{};
                fill_params<uint32_t>(p, g, tr, o, d_queues, d_counts, d_stats, nullptr);
                e = mg::launch_comine<uint32_t>(p, o.blocks, st);
            } else {
                mg::KParams<uint64_t> p{};
                fill_params<uint64_t>(p, g, tr, o, d_queues, d_counts, d_stats, nullptr);
                e = mg::launch_comine<uint64_t>(p, o.blocks, st);
            }
            if (e != hipSuccess)
                return fail(MG_EDEVICE, "co-mining launch failed: %s", hipGetErrorString(e));
        }
        uint64_t h[mg::kMaxQueries];
        uint64_t hs[mg::kStats];
        if (nq) HIP_TRY(hipMemcpyAsync(h, d_counts, 8 * nq, hipMemcpyDeviceToHost, st));
        if (d_stats) HIP_TRY(hipMemcpyAsync(hs, d_stats, sizeof hs, hipMemcpyDeviceToHost, st));
        HIP_TRY(hipStreamSynchronize(st));
        map_counts(tr, h, counts);
        if (o.stats) std::copy(hs, hs + mg::kStats, o.stats);
        return MG_OK;
    } catch (...) {
        return fail(MG_EINTERNAL, "unexpected exception");
    }
}

void mg_cursor_init(mg_cursor *c) {
    if (c) std::memset(c, 0, sizeof *c);
}

void mg_count_opts_init(mg_count_opts *o) {
    if (!o) return;
    std::memset(o, 0, sizeof *o);
    o->mode = MG_MODE_COMINE;
}

int mg_count(const mg_graph *g, const mg_tree *tr_c, const mg_count_opts *opts,
             uint64_t *counts) {
    try {
        if (!g || !tr_c || !counts) return fail(MG_EINVAL, "NULL argument");
        if (g->host_only) return fail(MG_EINVAL, "the graph is on the host only (MG_HOST_ONLY)");
        mg_tree *tr = const_cast<mg_tree *>(tr_c);   // device copy is a cache
        mg_count_opts o;
        mg_count_opts_init(&o);
        if (opts) o = *opts;
        if (o.mode == MG_MODE_AUTO) {
            mg_advice a{};
            int rc = mg_comine_advice(g, tr, MG_PLATFORM_GPU, &a);
            if (rc) return rc;
            o.mode = a.co_mine ? MG_MODE_COMINE : MG_MODE_PER_MOTIF;
        }
        if (o.mode != MG_MODE_COMINE && o.mode != MG_MODE_PER_MOTIF)
            return fail(MG_EINVAL, "unknown mode %d", o.mode);
        if (o.chunk < 0 || (o.chunk % 64) != 0 || o.chunk > (1 << 16))
            return fail(MG_EINVAL, "chunk must be a multiple of 64 in [0, 65536]");
        if (o.roots && o.n_roots < 0) return fail(MG_EINVAL, "n_roots < 0");
        if (o.queues < 0 || o.queues > mg::kQueues)
            return fail(MG_EINVAL, "queues must be in [0, %d]", mg::kQueues);
        if (o.stats && o.root_cost)
            return fail(MG_EINVAL, "stats and root_cost are exclusive");
        if (o.wave_clock && (o.mode != MG_MODE_COMINE || o.wave_clock_len < 0))
            return fail(MG_EINVAL, "wave_clock needs co-mining and a length >= 0");
        if (o.sched != MG_SCHED_PLAIN && o.sched != MG_SCHED_LEARNED)
            return fail(MG_EINVAL, "unknown schedule %d", o.sched);
        if (o.max_chunks < 0 || o.max_chunks > 0xffffffffll)
            return fail(MG_EINVAL, "max_chunks must be in [0, 2^32)");
        const bool stoppable = o.stop || o.max_chunks || o.cursor;
        if (stoppable && (o.mode != MG_MODE_COMINE || o.sched != MG_SCHED_PLAIN))
            return fail(MG_EINVAL, "stop, max_chunks and cursor need co-mining with the plain schedule");
        if (o.epoch_idle < 0 || o.epoch_idle > 100 || o.max_epochs < 0)
            return fail(MG_EINVAL, "epoch_idle must be in [0, 100] and max_epochs >= 0");
        if (o.epoch_idle && (o.mode != MG_MODE_COMINE || o.sched != MG_SCHED_PLAIN || stoppable ||
                             o.stats || o.root_cost || o.wave_clock))
            return fail(MG_EINVAL, "epochs need co-mining with the plain schedule, without stop, "
                                   "max_chunks, cursor, stats, root_cost or wave_clock");
        if (o.cursor && o.cursor->started) {
            const int32_t ch = o.chunk > 0 ? o.chunk : 64, nq = o.queues > 0 ? o.queues : mg::kQueues;
            const int64_t nr = o.roots ? o.n_roots : g->E;
            if (o.cursor->n_roots != nr || o.cursor->chunk != ch || o.cursor->queues != nq)
                return fail(MG_EINVAL, "the cursor belongs to a count with other roots, chunk or queues");
            for (int q = 0; q < nq; ++q) {
                const uint32_t len = mg::queue_end((uint32_t)nr, (uint32_t)nq, (uint32_t)q) -
                                     mg::queue_begin((uint32_t)nr, (uint32_t)nq, (uint32_t)q);
                if (o.cursor->head[q] > len) return fail(MG_EINVAL, "cursor head %d past its queue", q);
            }
        }
        if (o.sched == MG_SCHED_LEARNED) {
            if (!o.model) return fail(MG_EINVAL, "the learned schedule needs a model");
            if (o.roots) return fail(MG_EINVAL, "the learned schedule searches every root");
            if (o.sample < 0 || o.sample > mg::kSeg || (o.sample & (o.sample - 1)))
                return fail(MG_EINVAL, "sample must be 0 or a power of two up to %d", mg::kSeg);
            if (o.model->device != g->device) return fail(MG_EINVAL, "model on another device");
        }
        int dev = 0;
        HIP_TRY(hipGetDevice(&dev));
        if (dev != g->device) return fail(MG_EINVAL, "graph lives on device %d, current is %d",
                                          g->device, dev);
        hipStream_t st = (hipStream_t)o.stream;
        if (o.mode == MG_MODE_COMINE && o.sched == MG_SCHED_PLAIN && !stoppable && !o.roots &&
            !o.stats && !o.root_cost && !o.elapsed_ms && !o.wave_clock && !o.epoch_idle) {
            int rc = upload_tree(tr, dev, st);
            if (rc) return rc;
            std::vector<uint64_t> h(n_slots(tr));
            if (g->time_bytes == 4 ? small_count<uint32_t>(g, tr, o, true, h.data(), st, &rc)
                                   : small_count<uint64_t>(g, tr, o, true, h.data(), st, &rc)) {
                if (!rc) map_counts(tr, h.data(), counts);
                return rc;
            }
        }

        // roots
        DevBuf d_roots;
        uint32_t n_roots = (uint32_t)g->E;
        if (o.roots) {
            std::vector<uint32_t> r(o.n_roots);
            for (int64_t i = 0; i < o.n_roots; ++i) {
                if (o.roots[i] < 0 || o.roots[i] >= g->E)
                    return fail(MG_EINVAL, "root %lld outside [0, %lld)", (long long)o.roots[i],
                                (long long)g->E);
                r[i] = (uint32_t)o.roots[i];
            }
            n_roots = (uint32_t)o.n_roots;
            int rc = dev_alloc(d_roots, sizeof(uint32_t) * r.size(), (void *)st);
            if (rc) return rc;
            if (!r.empty())
                HIP_TRY(hipMemcpyAsync(d_roots.ptr, r.data(), sizeof(uint32_t) * r.size(),
                                       hipMemcpyHostToDevice, st));
        }
        struct Guard { DevBuf *b; ~Guard() { dev_free(*b); } } gr{&d_roots};

        // trees to run: the whole group, or one chain per distinct motif
        std::vector<mg_tree *> runs;
        if (o.mode == MG_MODE_COMINE) {
            runs.push_back(tr);
        } else {
            int rc = chain_trees(tr);
            if (rc) return rc;
            for (auto &u : tr->singles) runs.push_back(u.get());
        }
        size_t maxq = 1;
        for (mg_tree *t : runs) maxq = std::max(maxq, n_slots(t));
        static_assert(mg::kStats == MG_NSTATS, "stats layout");
        if (o.mode == MG_MODE_PER_MOTIF && n_roots > 0 && o.sched == MG_SCHED_PLAIN && !stoppable &&
            !o.roots && !o.stats && !o.root_cost && !o.wave_clock && !o.epoch_idle && !o.blocks &&
            (!o.chunk || o.chunk == 64) && (!o.queues || o.queues == mg::kQueues)) {
            // (64-root chunks and every queue: the defaults, spelled out)
            std::vector<uint64_t> qcount(n_slots(tr), 0);
            float ms = 0.f;
            bool taken = false;
            int rc = g->time_bytes == 4
                         ? count_runs<uint32_t>(g, runs, o, qcount.data(), &taken, st, o.elapsed_ms ? &ms : nullptr)
                         : count_runs<uint64_t>(g, runs, o, qcount.data(), &taken, st, o.elapsed_ms ? &ms : nullptr);
            if (rc) return rc;
            if (taken) {
                map_counts(tr, qcount.data(), counts);
                if (o.elapsed_ms) *o.elapsed_ms = ms;
                return MG_OK;
            }
        }
        // One region per run: queue heads, counters, statistics.  One fill kernel
        // clears them all, and they come back in one copy after the last run
        // (per-motif mode waited for the device after each of its searches:
        // 36 x 35 us).
        DevBuf d_work;
        const size_t words = (size_t)mg::kQueueWords + maxq + mg::kStats;
        int rc = dev_alloc(d_work, 8 * words * runs.size(), (void *)st);
        if (rc) return rc;
        struct Guard2 { DevBuf *b; ~Guard2() { dev_free(*b); } } gw{&d_work};
        unsigned long long *work = (unsigned long long *)d_work.ptr;
        HIP_TRY(mg::launch_fill_u64(work, (uint32_t)(words * runs.size()), 0ull, st));
        std::vector<uint64_t> stats_sum(mg::kStats, 0);
        DevBuf d_cost;
        if (o.root_cost) {
            rc = dev_alloc(d_cost, sizeof(uint64_t) * (size_t)g->E, (void *)st);
            if (rc) return rc;
            if (g->E) HIP_TRY(hipMemsetAsync(d_cost.ptr, 0, sizeof(uint64_t) * (size_t)g->E, st));
        }
        struct Guard3 { DevBuf *b; ~Guard3() { dev_free(*b); } } gc{&d_cost};
        DevBuf d_clock;
        if (o.wave_clock && o.wave_clock_len >= 2) {
            rc = dev_alloc(d_clock, 8 * (size_t)o.wave_clock_len, (void *)st);
            if (rc) return rc;
            HIP_TRY(hipMemsetAsync(d_clock.ptr, 0, 8 * (size_t)o.wave_clock_len, st));
        }
        struct Guard4 { DevBuf *b; ~Guard4() { dev_free(*b); } } gk{&d_clock};

        Scratch own;
        mg::EpochCtx *ctx = nullptr;
        bool deep = false;
        for (const mg_tree *t : runs) deep = deep || t->kdepth > 2;
        if (deep && hands_on(o, n_roots)) (void)own.get(&ctx, kHandOnCap, st);

        std::vector<uint64_t> qcount(n_slots(tr), 0);
        float total_ms = 0.f;
        mg_cursor cur{};
        for (size_t ri = 0; ri < runs.size(); ++ri) {
            mg_tree *t = runs[ri];
            rc = upload_tree(t, dev, st);
            if (rc) return rc;
            float ms = 0.f;
            unsigned long long *d_queues = work + ri * words;
            unsigned long long *d_counts = d_queues + mg::kQueueWords;
            unsigned long long *d_stats = o.stats ? d_counts + maxq : nullptr;
            rc = g->time_bytes == 4
                     ? launch_tree<uint32_t>(g, t, (const uint32_t *)d_roots.ptr, n_roots,
                                             d_queues, d_counts, d_stats,
                                             (unsigned long long *)d_cost.ptr,
                                             (unsigned long long *)d_clock.ptr, ctx, o, st,
                                             o.elapsed_ms ? &ms : nullptr)
                     : launch_tree<uint64_t>(g, t, (const uint32_t *)d_roots.ptr, n_roots,
                                             d_queues, d_counts, d_stats,
                                             (unsigned long long *)d_cost.ptr,
                                             (unsigned long long *)d_clock.ptr, ctx, o, st,
                                             o.elapsed_ms ? &ms : nullptr);
            if (rc) return rc;
            total_ms += ms;
            if (o.cursor) {
                std::vector<unsigned long long> q(mg::kQueueWords);
                HIP_TRY(hipMemcpyAsync(q.data(), d_queues, kQueueBytes, hipMemcpyDeviceToHost, st));
                HIP_TRY(hipStreamSynchronize(st));
                const uint32_t nq = o.queues > 0 ? (uint32_t)o.queues : (uint32_t)mg::kQueues;
                cur.n_roots = n_roots;
                cur.chunk = o.chunk > 0 ? o.chunk : 64;
                cur.queues = (int32_t)nq;
                cur.started = 1;
                cur.done = 1;
                for (uint32_t i = 0; i < (uint32_t)mg::kQueues; ++i) {
                    const uint64_t len = i < nq ? mg::queue_end(n_roots, nq, i) -
                                                      mg::queue_begin(n_roots, nq, i)
                                                : 0;
                    cur.head[i] = std::min<uint64_t>(q[(size_t)i * mg::kQueueStride], len);
                    if (cur.head[i] < len) cur.done = 0;
                }
            }
        }
        // (a single run needs its counters and statistics only)
        const size_t skip = runs.size() == 1 ? (size_t)mg::kQueueWords : 0;
        std::vector<uint64_t> h(words * runs.size() - skip);
        HIP_TRY(hipMemcpyAsync(h.data(), work + skip, 8 * h.size(), hipMemcpyDeviceToHost, st));
        HIP_TRY(hipStreamSynchronize(st));
        for (size_t ri = 0, at = 0; ri < runs.size(); ++ri) {
            const uint64_t *c = h.data() + ri * words + mg::kQueueWords - skip;
            const size_t n = n_slots(runs[ri]);
            std::copy(c, c + n, qcount.begin() + at);
            at += n;
            for (int i = 0; i < mg::kStats; ++i) stats_sum[i] += c[maxq + i];
        }
        map_counts(tr, qcount.data(), counts);
        if (o.root_cost && g->E) {
            HIP_TRY(hipMemcpyAsync(o.root_cost, d_cost.ptr, sizeof(uint64_t) * (size_t)g->E,
                                   hipMemcpyDeviceToHost, st));
            HIP_TRY(hipStreamSynchronize(st));
        }
        if (d_clock.ptr) {
            HIP_TRY(hipMemcpyAsync(o.wave_clock, d_clock.ptr, 8 * (size_t)o.wave_clock_len,
                                   hipMemcpyDeviceToHost, st));
            HIP_TRY(hipStreamSynchronize(st));
        }
        if (o.elapsed_ms) *o.elapsed_ms = total_ms;
        if (o.stats) std::copy(stats_sum.begin(), stats_sum.end(), o.stats);
        if (o.cursor) *o.cursor = cur;
        return MG_OK;
    } catch (const std::bad_alloc &) {
        return fail(MG_ENOMEM, "out of host memory");
    } catch (...) {
        return fail(MG_EINTERNAL, "unexpected exception");
    }
}


}  // extern "C"

// ---------------------------------------------------------------- autotuner
namespace {

// Identity of a (graph, tree, device) for the tuning cache: the graph's and
// tree's statistics and the device's name and compute-unit count.
std::string tune_key(const mg_graph *g, const mg_tree *tr) {
    hipDeviceProp_t prop{};
    if (hipGetDeviceProperties(&prop, g->device) != hipSuccess) prop.name[0] = 0;
    uint64_t h = 1469598103934665603ull;   // FNV-1a over the relabelled motifs
    auto mix = [&](uint64_t x) { h = (h ^ x) * 1099511628211ull; };
    for (const Motif &m : tr->distinct) {
        mix(m.size());
        for (auto &e : m) mix((uint64_t)e.first << 8 | (uint64_t)e.second);
    }
    for (int64_t w : tr->deltas) mix((uint64_t)w);
    char buf[512];
    snprintf(buf, sizeof buf, "%s/%d|E=%lld|V=%d|span=%lld|tb=%d|loops=%lld|motifs=%zu|depth=%d|"
             "prefixes=%d|trees=%016llx", prop.name, prop.multiProcessorCount, (long long)g->E,
             g->V, (long long)(g->t_max - g->t_min), g->time_bytes, (long long)g->self_loops,
             tr->distinct.size(), tr->depth, tr->info.n_prefixes, (unsigned long long)h);
    std::string k(buf);
    for (char &c : k)
        if (c == '"' || c == '\\' || c == '\n') c = '_';
    return k;
}

// One cache line: {"key": "...", "blocks": b, "chunk": c, "queues": q, "leaf_scan": l, "ms": t}
bool cache_lookup(const char *path, const std::string &key, mg_tune_result *r) {
    FILE *f = fopen(path, "r");
    if (!f) return false;
    char line[1024];
    bool found = false;
    const std::string want = "{\"key\": \"" + key + "\"";
    while (fgets(line, sizeof line, f)) {
        if (strncmp(line, want.c_str(), want.size()) != 0 || line[want.size()] != ',') continue;
        mg_tune_result t{};
        if (sscanf(line + want.size(),
                   ", \"blocks\": %d, \"chunk\": %d, \"queues\": %d, \"leaf_scan\": %d, "
                   "\"ms\": %f, \"default_ms\": %f",
                   &t.blocks, &t.chunk, &t.queues, &t.leaf_scan, &t.ms, &t.default_ms) == 6) {
            if (t.chunk == 64) t.chunk = 0;   // what the default was called before it depended
                                              // on the number of roots
            *r = t;
            found = true;   // the last entry for a key wins
        }
    }
    fclose(f);
    return found;
}

int cache_store(const char *path, const std::string &key, const mg_tune_result &r) {
    FILE *f = fopen(path, "a");
    if (!f) return fail(MG_EINVAL, "cannot append to the tuning cache %s", path);
    fprintf(f,
            "{\"key\": \"%s\", \"blocks\": %d, \"chunk\": %d, \"queues\": %d, \"leaf_scan\": %d, "
            "\"ms\": %.4f, \"default_ms\": %.4f}\n",
            key.c_str(), r.blocks, r.chunk, r.queues, r.leaf_scan, r.ms, r.default_ms);
    fclose(f);
    return MG_OK;
}

}  // namespace

extern "C" {

int mg_tune(const mg_graph *g, const mg_tree *tr, const char *cache_path, void *stream,
            mg_tune_result *out) {
    try {
        if (!g || !tr || !out) return fail(MG_EINVAL, "NULL argument");
        if (g->host_only) return fail(MG_EINVAL, "the graph is on the host only (MG_HOST_ONLY)");
        const std::string key = tune_key(g, tr);
        mg_tune_result best{};
        if (cache_path && cache_lookup(cache_path, key, &best)) {
            best.from_cache = 1;
            *out = best;
            return MG_OK;
        }
        int dev = 0, ncu = 0;
        HIP_TRY(hipGetDevice(&dev));
        HIP_TRY(hipDeviceGetAttribute(&ncu, hipDeviceAttributeMultiprocessorCount, dev));
        // median of three timed counts after one untimed one
        int32_t trials = 0;
        auto time_of = [&](const mg_tune_result &c, float *ms) -> int {
            mg_count_opts o;
            mg_count_opts_init(&o);
            o.blocks = c.blocks;
            o.chunk = c.chunk;
            o.queues = c.queues;
            o.leaf_scan = c.leaf_scan;
            o.stream = stream;
            std::vector<uint64_t> cnt((size_t)tr->n_motifs * tr->delta_slot.size());
            int rc = mg_count(g, tr, &o, cnt.data());
            if (rc) return rc;
            float t[3];
            o.elapsed_ms = nullptr;
            for (float &x : t) {
                o.elapsed_ms = &x;
                rc = mg_count(g, tr, &o, cnt.data());
                if (rc) return rc;
            }
            std::sort(t, t + 3);
            *ms = t[1];
            ++trials;
            return MG_OK;
        };
        // coordinate descent from the defaults, one setting at a time
        mg_tune_result cur{};
        cur.blocks = 0;
        cur.chunk = 0;   // (the launch chooses: fill_params, launch_ds)
        cur.queues = mg::kQueues;
        cur.leaf_scan = (int32_t)mg::kLeafScanDefault;
        int rc = time_of(cur, &cur.ms);
        if (rc) return rc;
        cur.default_ms = cur.ms;
        const std::vector<int32_t> chunks = {0, 128, 256}, queues = {8, 4, 2, 1},
                                   scans = {64, 128, 256, 512, 1024},
                                   blocks = {0, ncu * 4, ncu * 6};
        for (int sweep = 0; sweep < 2; ++sweep) {
            bool moved = false;
            for (int dim = 0; dim < 4; ++dim) {
                const std::vector<int32_t> &vals =
                    dim == 0 ? scans : dim == 1 ? chunks : dim == 2 ? queues : blocks;
                for (int32_t v : vals) {
                    mg_tune_result c = cur;
                    int32_t &field = dim == 0 ? c.leaf_scan : dim == 1 ? c.chunk
                                     : dim == 2 ? c.queues : c.blocks;
                    if (field == v) continue;
                    field = v;
                    rc = time_of(c, &c.ms);
                    if (rc) return rc;
                    // a new setting must win by more than the noise of one timing
                    if (c.ms < 0.98f * cur.ms) {
                        cur = c;
                        moved = true;
                    }
                }
            }
            if (!moved) break;
        }
        cur.trials = trials;
        if (cache_path) {
            rc = cache_store(cache_path, key, cur);
            if (rc) return rc;
        }
        *out = cur;
        return MG_OK;
    } catch (const std::bad_alloc &) {
        return fail(MG_ENOMEM, "out of host memory");
    } catch (...) {
        return fail(MG_EINTERNAL, "unexpected exception");
    }
}

}  // extern "C"
