// Graph ingest on the device: stable time sort, time-sorted out- and in-lists
// and the per-edge list ranks.  Internal interface between host.cpp and
// ingest.hip.
#pragma once
#include <hip/hip_runtime_api.h>
#include <stdint.h>

#include "comine.h"

namespace mg {

// What the edge arrays hold, found by one pass over them.  Times as biased
// 64-bit values (sign bit flipped), so that unsigned minima are signed ones.
struct EdgeFacts {
    unsigned long long first_bad;   // first edge with a vertex outside [0, V), else ~0
    unsigned long long unsorted;    // 1 when some time is below its predecessor's
    unsigned long long loops;       // self-loops
    unsigned long long t_min, t_max;
};
inline int64_t unbias_time(unsigned long long t) { return (int64_t)(t ^ (1ull << 63)); }
hipError_t launch_edge_facts(const int32_t *src, const int32_t *dst, const int64_t *t, uint32_t n,
                             int32_t n_nodes, EdgeFacts *facts, hipStream_t st);

// Scratch bytes of a stable radix sort of n (key, 32-bit value) pairs.
size_t sort_scratch_bytes(uint32_t n);

// Stable sort of n pairs by the low `bits` bits of the key.  The pairs start
// in k[0] and v[0] (with iota: the values are 0..n-1 and v[0] is not read),
// pass between the two sides and end in k[*where], v[*where].
template <typename K>
hipError_t sort_pairs(K *const k[2], uint32_t *const v[2], bool iota, uint32_t n, int bits,
                      void *scratch, int *where, hipStream_t st);

// keys[i] = t[i] - t_min
template <typename TT>
hipError_t launch_time_keys(const int64_t *t, int64_t t_min, uint32_t n, TT *keys, hipStream_t st);

// The time-ordered edge list from the caller's arrays: edge i is input edge
// order[i] (order NULL: i).  okey / ikey: its source / destination, V for a
// self-loop (sorted past every vertex, so left out of the lists).
template <typename TT>
hipError_t launch_place_edges(const int32_t *src, const int32_t *dst, const int64_t *t,
                              int64_t t_min, const uint32_t *order, uint32_t n, uint32_t n_nodes,
                              int32_t *gsrc, int32_t *gdst, TT *gt, uint32_t *okey, uint32_t *ikey,
                              hipStream_t st);

// One side's lists from its sorted (vertex, edge id) pairs: off[0..V], and for
// the n_adj entries the other endpoint and time, and each edge's entry index.
template <typename TT>
hipError_t launch_lists(const uint32_t *key, const uint32_t *eid, uint32_t n_adj, uint32_t n_nodes,
                        const int32_t *other, const TT *gt, uint32_t *off, Entry<TT> *adj,
                        uint32_t *pos, hipStream_t st);

// gx and gn (DevGraph) of every edge, given where each edge sits in its two
// lists.
template <typename TT>
hipError_t launch_ranks(const DevGraph<TT> &g, const uint32_t *opos, const uint32_t *ipos,
                        uint4 *gx, uint2 *gn, hipStream_t st);

// Pair order (edge ids pe[0..n_adj) by destination, source, time): pair_t, gp
// (with the entries' records where g.gp_out says so), the pair codes of gn and the
// next codes of both lists' entries.  psrc: scratch, n_adj words.
template <typename TT>
hipError_t launch_pairs(const DevGraph<TT> &g, const uint32_t *pe, uint32_t n_adj,
                        const uint32_t *opos, const uint32_t *ipos, int32_t *psrc, TT *pair_t,
                        uint4 *gp, uint2 *gn, Entry<TT> *out_adj,
                        Entry<TT> *in_adj, hipStream_t st);

// keys[j] = key_of[eid[j]] for n entries
hipError_t launch_gather(const uint32_t *eid, const int32_t *key_of, uint32_t n, uint32_t *keys,
                         hipStream_t st);

}  // namespace mg
