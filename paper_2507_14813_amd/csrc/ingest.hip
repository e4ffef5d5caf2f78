// Graph ingest for gfx950: everything between the caller's edge arrays and
// the arrays the search reads runs here, on the device.
//
// The lists are built by stable radix sorts of 32-bit edge ids: by time (only
// when the input is not in time order), then, over the time-ordered edges, by
// source and by destination, which leaves every list ascending in time.  A
// sort is least-significant-digit first, 8 bits per pass and only the bits
// the keys can have; each pass is a digit histogram per tile, one exclusive
// scan over (digit, tile) and a scatter.
//
// The passes stream the pairs (8 B read for the histogram and the scatter
// each, 8 B written) and are bound by memory, the scatter by its 256 write
// streams per tile.  What the host did before in one thread (counting sorts
// with random writes) and per edge (four bisections) took 145 ms for a
// million unsorted edges, uploads included; here the same takes 1.1 ms.
#include <hip/hip_runtime.h>

#include <algorithm>

#include "device_util.h"
#include "ingest.h"

namespace mg {
namespace {

constexpr int kIB = 256;                   // threads per block
constexpr int kDigits = 256;               // 8 bits per pass
constexpr int kRounds = 16;                // keys per thread and tile
constexpr int kTile = kIB * kRounds;
constexpr int kIWaves = kIB / kWave;
constexpr int kScanTile = kIB * 16;        // elements per scan block
static_assert(kDigits == kIB, "one thread per digit");

inline uint32_t grid_for(uint64_t n, uint32_t per_block, uint32_t most = 16384) {
    return (uint32_t)std::max<uint64_t>(1, std::min<uint64_t>((n + per_block - 1) / per_block, most));
}

// ------------------------------------------------------------ edge facts
__global__ void facts_init(EdgeFacts *f) {
    f->first_bad = ~0ull;
    f->unsorted = 0;
    f->loops = 0;
    f->t_min = ~0ull;
    f->t_max = 0;
}

__device__ __forceinline__ unsigned long long wave_min(unsigned long long v) {
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) v = min(v, (unsigned long long)__shfl_xor((unsigned long long)v, o));
    return v;
}
__device__ __forceinline__ unsigned long long wave_max(unsigned long long v) {
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) v = max(v, (unsigned long long)__shfl_xor((unsigned long long)v, o));
    return v;
}

__global__ void __launch_bounds__(kIB)
edge_facts(const int32_t *src, const int32_t *dst, const int64_t *t, uint32_t n, int32_t n_nodes,
           EdgeFacts *f) {
    unsigned long long bad = ~0ull, lo = ~0ull, hi = 0;
    uint32_t loops = 0;
    bool unsorted = false;
    for (uint64_t i = blockIdx.x * (uint64_t)kIB + threadIdx.x; i < n; i += gridDim.x * (uint64_t)kIB) {
        const int32_t s = src[i], d = dst[i];
        if ((s < 0 || s >= n_nodes || d < 0 || d >= n_nodes) && i < bad) bad = i;
        loops += s == d ? 1u : 0u;
        const int64_t x = t[i];
        if (i && x < t[i - 1]) unsorted = true;
        const unsigned long long b = (unsigned long long)x ^ (1ull << 63);
        lo = min(lo, b);
        hi = max(hi, b);
    }
    // one set of atomics per block: on one address they come one after another
    // (one set per wave of a full grid took 140 us)
    __shared__ unsigned long long s_bad[kIWaves], s_lo[kIWaves], s_hi[kIWaves];
    __shared__ uint32_t s_loops[kIWaves], s_uns[kIWaves];
    const int w = threadIdx.x / kWave;
    bad = wave_min(bad);
    lo = wave_min(lo);
    hi = wave_max(hi);
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) loops += __shfl_xor(loops, o);
    const bool any = __ballot(unsorted) != 0;
    if ((threadIdx.x & (kWave - 1)) == 0) {
        s_bad[w] = bad;
        s_lo[w] = lo;
        s_hi[w] = hi;
        s_loops[w] = loops;
        s_uns[w] = any;
    }
    __syncthreads();
    if (threadIdx.x != 0) return;
    unsigned long long nl = 0;
    uint32_t uns = 0;
    for (int k = 0; k < kIWaves; ++k) {
        bad = min(bad, s_bad[k]);
        lo = min(lo, s_lo[k]);
        hi = max(hi, s_hi[k]);
        nl += s_loops[k];
        uns |= s_uns[k];
    }
    if (bad != ~0ull) atomicMin(&f->first_bad, bad);
    if (uns) f->unsorted = 1;
    if (nl) atomicAdd(&f->loops, nl);
    if (lo != ~0ull) atomicMin(&f->t_min, lo);
    if (hi) atomicMax(&f->t_max, hi);
}

// ------------------------------------------------------------ radix sort
// digit counts of every tile, laid out digit-major: hist[d * n_tiles + tile]
template <typename K>
__global__ void __launch_bounds__(kIB)
digit_hist(const K *key, uint32_t n, int shift, uint32_t mask, uint32_t n_tiles, uint32_t *hist) {
    __shared__ uint32_t cnt[kDigits];
    cnt[threadIdx.x] = 0;
    __syncthreads();
    const uint64_t base = (uint64_t)blockIdx.x * kTile;
#pragma unroll
    for (int r = 0; r < kRounds; ++r) {
        const uint64_t i = base + r * kIB + threadIdx.x;
        if (i < n) atomicAdd(&cnt[(uint32_t)(key[i] >> shift) & mask], 1u);
    }
    __syncthreads();
    hist[(uint64_t)threadIdx.x * n_tiles + blockIdx.x] = cnt[threadIdx.x];
}

// inclusive scan of one value per thread over the block (kIB threads)
__device__ __forceinline__ uint32_t block_incl(uint32_t x, uint32_t *sums) {
    const int lane = threadIdx.x & (kWave - 1), w = threadIdx.x / kWave;
    uint32_t s = incl_scan32(x, lane);
    if (lane == kWave - 1) sums[w] = s;
    __syncthreads();
    for (int k = 0; k < w; ++k) s += sums[k];
    __syncthreads();
    return s;
}

__global__ void __launch_bounds__(kIB)
scan_reduce(const uint32_t *x, uint32_t n, uint32_t *sums) {
    __shared__ uint32_t part[kIWaves];
    const uint64_t base = (uint64_t)blockIdx.x * kScanTile;
    uint32_t s = 0;
#pragma unroll
    for (int r = 0; r < 16; ++r) {
        const uint64_t i = base + r * kIB + threadIdx.x;
        if (i < n) s += x[i];
    }
    s = block_incl(s, part);
    if (threadIdx.x == kIB - 1) sums[blockIdx.x] = s;
}

// exclusive scan of the block sums (one block)
__global__ void __launch_bounds__(kIB) scan_sums(uint32_t *sums, uint32_t n) {
    __shared__ uint32_t part[kIWaves];
    __shared__ uint32_t carry;
    if (threadIdx.x == 0) carry = 0;
    __syncthreads();
    for (uint32_t b = 0; b < n; b += kIB) {
        const uint32_t i = b + threadIdx.x;
        const uint32_t x = i < n ? sums[i] : 0u;
        const uint32_t s = block_incl(x, part) + carry;
        if (i < n) sums[i] = s - x;
        __syncthreads();
        if (threadIdx.x == kIB - 1) carry = s;
        __syncthreads();
    }
}

// exclusive scan in place: element i of a scan block gets the block's sum
// plus the elements before it (16 consecutive elements per thread; n is a
// multiple of 4 and x 16-byte aligned)
__global__ void __launch_bounds__(kIB)
scan_apply(uint32_t *x, uint32_t n, const uint32_t *sums) {
    __shared__ uint32_t part[kIWaves];
    const uint64_t base = (uint64_t)blockIdx.x * kScanTile + threadIdx.x * 16ull;
    uint4 v[4];
    uint32_t s = 0;
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        v[k] = make_uint4(0, 0, 0, 0);
        if (base + 4 * k < n) v[k] = reinterpret_cast<const uint4 *>(x)[base / 4 + k];
        s += v[k].x + v[k].y + v[k].z + v[k].w;
    }
    uint32_t run = block_incl(s, part) - s + sums[blockIdx.x];
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        uint4 o;
        o.x = run;
        o.y = o.x + v[k].x;
        o.z = o.y + v[k].y;
        o.w = o.z + v[k].z;
        run = o.w + v[k].w;
        if (base + 4 * k < n) reinterpret_cast<uint4 *>(x)[base / 4 + k] = o;
    }
}

// A key's rank among the wave's keys of its digit d (b bits) in input order, where
// cnt holds how many of each digit the wave has had: the lanes that hold the same
// digit find each other with one ballot per digit bit.  So the sort is stable.
__device__ __forceinline__ uint32_t rank_in_wave(uint32_t d, int b, bool in, uint32_t *cnt) {
    uint64_t same = __ballot(in);
    for (int i = 0; i < b; ++i) {
        const uint64_t one = __ballot((d >> i) & 1u);
        same &= ((d >> i) & 1u) ? one : ~one;
    }
    uint32_t rank = 0;
    if (in) rank = cnt[d] + mbcnt(same);
    wave_sync();
    if (in && mbcnt(same) == 0) cnt[d] += (uint32_t)__popcll(same);
    wave_sync();
    return rank;
}

// Scatter of one tile.  A wave takes 16 rounds of 64 consecutive keys.
template <typename K>
__global__ void __launch_bounds__(kIB)
digit_scatter(const K *key, const uint32_t *val, uint32_t n, int shift, int bits, uint32_t n_tiles,
              const uint32_t *hist, K *key_out, uint32_t *val_out) {
    __shared__ uint32_t cnt[kIWaves][kDigits];
    const int lane = threadIdx.x & (kWave - 1), w = threadIdx.x / kWave;
    const uint32_t mask = (1u << bits) - 1u;
#pragma unroll
    for (int k = 0; k < kIWaves; ++k) cnt[k][threadIdx.x] = 0;
    __syncthreads();
    const uint64_t base = (uint64_t)blockIdx.x * kTile + (uint64_t)w * (kWave * kRounds);
    K k[kRounds];
    uint32_t rank[kRounds];
#pragma unroll
    for (int r = 0; r < kRounds; ++r) {
        const uint64_t i = base + r * kWave + lane;
        k[r] = i < n ? key[i] : (K)0;
    }
#pragma unroll
    for (int r = 0; r < kRounds; ++r) {
        const bool in = base + r * kWave + lane < n;
        rank[r] = rank_in_wave((uint32_t)(k[r] >> shift) & mask, bits, in, cnt[w]);
    }
    __syncthreads();
    // where each wave's keys of digit threadIdx.x start
    {
        const uint32_t d = threadIdx.x;
        uint32_t at = hist[(uint64_t)d * n_tiles + blockIdx.x];
#pragma unroll
        for (int x = 0; x < kIWaves; ++x) {
            const uint32_t c = cnt[x][d];
            cnt[x][d] = at;
            at += c;
        }
    }
    __syncthreads();
#pragma unroll
    for (int r = 0; r < kRounds; ++r) {
        const uint64_t i = base + r * kWave + lane;
        if (i < n) {
            const uint32_t to = cnt[w][(uint32_t)(k[r] >> shift) & mask] + rank[r];
            key_out[to] = k[r];
            val_out[to] = val ? val[i] : (uint32_t)i;
        }
    }
}

// All passes of a sort of at most one tile, by one workgroup: the pairs stay in
// registers and change places through LDS.  A small graph's build is its launches
// and allocations: 1,000 unsorted edges from host memory took 251 us with five
// launches per pass and 22 allocations, now one of each per sort, and three: 135.
template <typename K>
__global__ void __launch_bounds__(kIB)
sort_tile(const K *key, const uint32_t *val, uint32_t n, int bits, int passes, K *key_out,
          uint32_t *val_out) {
    __shared__ uint32_t cnt[kIWaves][kDigits];
    __shared__ uint32_t part[kIWaves];
    __shared__ K ks[kTile];
    __shared__ uint32_t vs[kTile];
    const int lane = threadIdx.x & (kWave - 1), w = threadIdx.x / kWave;
    const uint32_t rounds = (n + kIB - 1) / kIB;   // per wave
    const uint32_t base = (uint32_t)w * rounds * kWave + (uint32_t)lane;
    K k[kRounds];
    uint32_t v[kRounds], rank[kRounds];
#pragma unroll
    for (int r = 0; r < kRounds; ++r) {
        const uint32_t i = base + r * kWave;
        const bool in = (uint32_t)r < rounds && i < n;
        k[r] = in ? key[i] : (K)0;
        v[r] = in && val ? val[i] : i;
    }
    int shift = 0;
    for (int p = 0; p < passes; ++p) {
        const int b = (bits - shift + (passes - p) - 1) / (passes - p);
        const uint32_t mask = (1u << b) - 1u;
#pragma unroll
        for (int x = 0; x < kIWaves; ++x) cnt[x][threadIdx.x] = 0;
        __syncthreads();
#pragma unroll
        for (int r = 0; r < kRounds; ++r) {
            const bool in = base + r * kWave < n;
            if ((uint32_t)r < rounds) rank[r] = rank_in_wave((uint32_t)(k[r] >> shift) & mask, b, in, cnt[w]);
        }
        __syncthreads();
        {
            const uint32_t d = threadIdx.x;
            uint32_t c[kIWaves], sum = 0;
#pragma unroll
            for (int x = 0; x < kIWaves; ++x) sum += c[x] = cnt[x][d];
            uint32_t at = block_incl(sum, part) - sum;
#pragma unroll
            for (int x = 0; x < kIWaves; ++x) {
                cnt[x][d] = at;
                at += c[x];
            }
        }
        __syncthreads();
#pragma unroll
        for (int r = 0; r < kRounds; ++r) {
            if ((uint32_t)r < rounds && base + r * kWave < n) {
                const uint32_t to = cnt[w][(uint32_t)(k[r] >> shift) & mask] + rank[r];
                ks[to] = k[r];
                vs[to] = v[r];
            }
        }
        __syncthreads();
#pragma unroll
        for (int r = 0; r < kRounds; ++r) {
            const uint32_t i = base + r * kWave;
            if ((uint32_t)r < rounds && i < n) {
                k[r] = ks[i];
                v[r] = vs[i];
            }
        }
        shift += b;
    }
#pragma unroll
    for (int r = 0; r < kRounds; ++r) {
        const uint32_t i = base + r * kWave;
        if ((uint32_t)r < rounds && i < n) {
            key_out[i] = k[r];
            val_out[i] = v[r];
        }
    }
}

__global__ void iota_u32(uint32_t *p, uint32_t n) {
    for (uint64_t i = blockIdx.x * (uint64_t)kIB + threadIdx.x; i < n; i += gridDim.x * (uint64_t)kIB)
        p[i] = (uint32_t)i;
}

// ------------------------------------------------------------ edges and lists
template <typename TT>
__global__ void __launch_bounds__(kIB)
time_keys(const int64_t *t, int64_t t_min, uint32_t n, TT *key) {
    for (uint64_t i = blockIdx.x * (uint64_t)kIB + threadIdx.x; i < n; i += gridDim.x * (uint64_t)kIB)
        key[i] = (TT)((uint64_t)t[i] - (uint64_t)t_min);
}

template <typename TT>
__global__ void __launch_bounds__(kIB)
place_edges(const int32_t *src, const int32_t *dst, const int64_t *t, int64_t t_min,
            const uint32_t *order, uint32_t n, uint32_t n_nodes, int32_t *gsrc, int32_t *gdst,
            TT *gt, uint32_t *okey, uint32_t *ikey) {
    for (uint64_t i = blockIdx.x * (uint64_t)kIB + threadIdx.x; i < n; i += gridDim.x * (uint64_t)kIB) {
        const uint32_t j = order ? order[i] : (uint32_t)i;
        const int32_t s = src[j], d = dst[j];
        gsrc[i] = s;
        gdst[i] = d;
        gt[i] = (TT)((uint64_t)t[j] - (uint64_t)t_min);
        okey[i] = s == d ? n_nodes : (uint32_t)s;
        ikey[i] = s == d ? n_nodes : (uint32_t)d;
    }
}

// off[v] = the first entry whose vertex is v or later
__global__ void __launch_bounds__(kIB)
list_offsets(const uint32_t *key, uint32_t n_adj, uint32_t n_nodes, uint32_t *off) {
    for (uint64_t v = blockIdx.x * (uint64_t)kIB + threadIdx.x; v <= n_nodes;
         v += gridDim.x * (uint64_t)kIB) {
        uint32_t lo = 0, n = n_adj;
        while (n > 0) {
            const uint32_t h = n >> 1;
            if (key[lo + h] < (uint32_t)v) { lo += h + 1; n -= h + 1; }
            else n = h;
        }
        off[v] = lo;
    }
}

template <typename TT>
__global__ void __launch_bounds__(kIB)
list_entries(const uint32_t *eid, uint32_t n_adj, const int32_t *other, const TT *gt,
             Entry<TT> *adj, uint32_t *pos) {
    for (uint64_t j = blockIdx.x * (uint64_t)kIB + threadIdx.x; j < n_adj;
         j += gridDim.x * (uint64_t)kIB) {
        const uint32_t e = eid[j];
        Entry<TT> x{};
        x.v = other[e];
        x.t = gt[e];
        if constexpr (sizeof(TT) == 4) x.eid = e;
        adj[j] = x;
        pos[e] = (uint32_t)j;
    }
}

// An edge u -> v at t: the first entries after t in out(u) and in(v) lie just
// past its own entries (past those with its time); the ones in in(u) and
// out(v) by bisection.
template <typename TT>
__global__ void __launch_bounds__(kIB)
list_ranks(const DevGraph<TT> g, const uint32_t *opos, const uint32_t *ipos, uint4 *gx,
           uint2 *gn) {
    const TT *ot = times_of(g.out_adj), *it = times_of(g.in_adj);
    for (uint64_t e = blockIdx.x * (uint64_t)kIB + threadIdx.x; e < g.n_edges;
         e += gridDim.x * (uint64_t)kIB) {
        const int32_t u = g.gsrc[e], v = g.gdst[e];
        uint4 x = make_uint4(0, 0, 0, 0);
        uint2 n = make_uint2(~0u, ~0u);
        if (u != v) {
            const TT t = g.gt[e];
            const uint32_t eu = g.out_off[u + 1], iu = g.in_off[u + 1];
            const uint32_t ev = g.out_off[v + 1], iv = g.in_off[v + 1];
            auto code = [&](const TT *a, uint32_t i, uint32_t end, int k) {
                if (i >= end) return;
                const uint32_t c = next_code((TT)(a[(size_t)i << kAdjShift<TT>] - t));
                n.y = (n.y & ~(255u << (8 * k))) | (c << (8 * k));
            };
            x.x = gallop_greater(ot, kAdjShift<TT>, opos[e] + 1, eu, t);
            x.y = first_greater(it, kAdjShift<TT>, g.in_off[u], iu, t);
            x.z = first_greater(ot, kAdjShift<TT>, g.out_off[v], ev, t);
            x.w = gallop_greater(it, kAdjShift<TT>, ipos[e] + 1, iv, t);
            code(ot, x.x, eu, 0);
            code(it, x.y, iu, 1);
            code(ot, x.z, ev, 2);
            code(it, x.w, iv, 3);
        }
        gx[e] = x;
        gn[e] = n;
    }
}

__global__ void __launch_bounds__(kIB)
gather_keys(const uint32_t *eid, const int32_t *key_of, uint32_t n, uint32_t *keys) {
    for (uint64_t j = blockIdx.x * (uint64_t)kIB + threadIdx.x; j < n; j += gridDim.x * (uint64_t)kIB)
        keys[j] = (uint32_t)key_of[eid[j]];
}

template <typename TT>
__global__ void __launch_bounds__(kIB)
pair_entries(const DevGraph<TT> g, const uint32_t *pe, uint32_t n_adj, int32_t *psrc, TT *pair_t) {
    for (uint64_t j = blockIdx.x * (uint64_t)kIB + threadIdx.x; j < n_adj;
         j += gridDim.x * (uint64_t)kIB) {
        const uint32_t e = pe[j];
        psrc[j] = g.gsrc[e];
        pair_t[j] = g.gt[e];
    }
}

// Entry j of the pair order is edge u -> v at t.  The edges into v are the
// entries [in_off[v], in_off[v + 1]) and ascend in source, so the pair's end
// is found by galloping from j, and the pair v -> u by bisection among the
// edges into u.
template <typename TT>
__global__ void __launch_bounds__(kIB)
pair_links(const DevGraph<TT> g, const uint32_t *pe, uint32_t n_adj, const uint32_t *opos,
           const uint32_t *ipos, const int32_t *psrc, const TT *pair_t, uint4 *gp, uint2 *gn, Entry<TT> *out_adj, Entry<TT> *in_adj) {
    for (uint64_t j = blockIdx.x * (uint64_t)kIB + threadIdx.x; j < n_adj;
         j += gridDim.x * (uint64_t)kIB) {
        const uint32_t e = pe[j];
        const int32_t u = psrc[j], v = g.gdst[e];
        const TT t = pair_t[j];
        uint4 p = make_uint4(0, 0, 0, 0);
        p.y = gallop_greater(psrc, 0, (uint32_t)j + 1, g.in_off[v + 1], u);
        p.x = gallop_greater(pair_t, 0, (uint32_t)j + 1, p.y, t);
        const uint32_t e0 = g.in_off[u], e1 = g.in_off[u + 1];
        const uint32_t r0 = first_greater(psrc, 0, e0, e1, v - 1);
        const uint32_t r1 = gallop_greater(psrc, 0, r0, e1, v);
        if (r0 < r1) {
            p.z = first_greater(pair_t, 0, r0, r1, t);
            p.w = r1;
        }
        const uint32_t op = opos[e], ip = ipos[e];
        gp[e] = p;
        if (g.gp_out) {
            gp[g.gp_out + op] = p;
            gp[g.gp_in + ip] = p;
        }
        const uint32_t fwd = p.x < p.y ? next_code((TT)(pair_t[p.x] - t)) : 255u;
        const uint32_t rev = p.z < p.w ? next_code((TT)(pair_t[p.z] - t)) : 255u;
        const uint32_t pairs = fwd | (rev << 8), lists = gn[e].y;
        gn[e].x = pairs;
        out_adj[op].nx = pairs | (lists & 0xffff0000u);
        in_adj[ip].nx = pairs | (lists << 16);
    }
}

inline uint64_t tiles_of(uint32_t n) { return ((uint64_t)n + kTile - 1) / kTile; }
inline uint64_t scan_blocks(uint64_t n) { return (n + kScanTile - 1) / kScanTile; }

}  // namespace

hipError_t launch_edge_facts(const int32_t *src, const int32_t *dst, const int64_t *t, uint32_t n,
                             int32_t n_nodes, EdgeFacts *facts, hipStream_t st) {
    hipLaunchKernelGGL(facts_init, dim3(1), dim3(1), 0, st, facts);
    hipLaunchKernelGGL(edge_facts, dim3(grid_for(n, kIB * 8, 512)), dim3(kIB), 0, st, src, dst, t,
                       n, n_nodes, facts);
    return hipGetLastError();
}

size_t sort_scratch_bytes(uint32_t n) {
    const uint64_t h = tiles_of(n) * kDigits;
    return (size_t)(4 * (h + scan_blocks(h)) + 64);
}

template <typename K>
hipError_t sort_pairs(K *const k[2], uint32_t *const v[2], bool iota, uint32_t n, int bits,
                      void *scratch, int *where, hipStream_t st) {
    *where = 0;
    const uint32_t tiles = (uint32_t)tiles_of(n);
    uint32_t *hist = (uint32_t *)scratch;
    const uint32_t nh = tiles * kDigits;
    uint32_t *sums = hist + nh;
    const int passes = (bits + 7) / 8;
    if (n == 0) return hipSuccess;
    if (passes == 0) {
        if (iota) hipLaunchKernelGGL(iota_u32, dim3(grid_for(n, kIB)), dim3(kIB), 0, st, v[0], n);
        return hipGetLastError();
    }
    if (tiles == 1) {
        hipLaunchKernelGGL(sort_tile<K>, dim3(1), dim3(kIB), 0, st, k[0], iota ? nullptr : v[0], n,
                           bits, passes, k[1], v[1]);
        *where = 1;
        return hipGetLastError();
    }
    int shift = 0;
    for (int p = 0; p < passes; ++p) {
        // the bits spread evenly over the passes: fewer write streams per tile
        const int b = (bits - shift + (passes - p) - 1) / (passes - p);
        const int a = p & 1;
        hipLaunchKernelGGL(digit_hist<K>, dim3(tiles), dim3(kIB), 0, st, k[a], n, shift,
                           (1u << b) - 1u, tiles, hist);
        const uint32_t sb = (uint32_t)scan_blocks(nh);
        hipLaunchKernelGGL(scan_reduce, dim3(sb), dim3(kIB), 0, st, hist, nh, sums);
        hipLaunchKernelGGL(scan_sums, dim3(1), dim3(kIB), 0, st, sums, sb);
        hipLaunchKernelGGL(scan_apply, dim3(sb), dim3(kIB), 0, st, hist, nh, sums);
        const uint32_t *vin = (p == 0 && iota) ? nullptr : v[a];
        hipLaunchKernelGGL(digit_scatter<K>, dim3(tiles), dim3(kIB), 0, st, k[a], vin, n, shift, b,
                           tiles, hist, k[a ^ 1], v[a ^ 1]);
        shift += b;
    }
    *where = passes & 1;
    return hipGetLastError();
}

template <typename TT>
hipError_t launch_time_keys(const int64_t *t, int64_t t_min, uint32_t n, TT *keys, hipStream_t st) {
    hipLaunchKernelGGL(time_keys<TT>, dim3(grid_for(n, kIB)), dim3(kIB), 0, st, t, t_min, n, keys);
    return hipGetLastError();
}

template <typename TT>
hipError_t launch_place_edges(const int32_t *src, const int32_t *dst, const int64_t *t,
                              int64_t t_min, const uint32_t *order, uint32_t n, uint32_t n_nodes,
                              int32_t *gsrc, int32_t *gdst, TT *gt, uint32_t *okey, uint32_t *ikey,
                              hipStream_t st) {
    hipLaunchKernelGGL(place_edges<TT>, dim3(grid_for(n, kIB)), dim3(kIB), 0, st, src, dst, t,
                       t_min, order, n, n_nodes, gsrc, gdst, gt, okey, ikey);
    return hipGetLastError();
}

template <typename TT>
hipError_t launch_lists(const uint32_t *key, const uint32_t *eid, uint32_t n_adj, uint32_t n_nodes,
                        const int32_t *other, const TT *gt, uint32_t *off, Entry<TT> *adj,
                        uint32_t *pos, hipStream_t st) {
    hipLaunchKernelGGL(list_offsets, dim3(grid_for((uint64_t)n_nodes + 1, kIB)), dim3(kIB), 0, st,
                       key, n_adj, n_nodes, off);
    if (n_adj)
        hipLaunchKernelGGL(list_entries<TT>, dim3(grid_for(n_adj, kIB)), dim3(kIB), 0, st, eid,
                           n_adj, other, gt, adj, pos);
    return hipGetLastError();
}

template <typename TT>
hipError_t launch_ranks(const DevGraph<TT> &g, const uint32_t *opos, const uint32_t *ipos,
                        uint4 *gx, uint2 *gn, hipStream_t st) {
    if (g.n_edges == 0) return hipSuccess;
    hipLaunchKernelGGL(list_ranks<TT>, dim3(grid_for(g.n_edges, kIB)), dim3(kIB), 0, st, g, opos,
                       ipos, gx, gn);
    return hipGetLastError();
}

hipError_t launch_gather(const uint32_t *eid, const int32_t *key_of, uint32_t n, uint32_t *keys,
                         hipStream_t st) {
    if (n == 0) return hipSuccess;
    hipLaunchKernelGGL(gather_keys, dim3(grid_for(n, kIB)), dim3(kIB), 0, st, eid, key_of, n, keys);
    return hipGetLastError();
}

template <typename TT>
hipError_t launch_pairs(const DevGraph<TT> &g, const uint32_t *pe, uint32_t n_adj,
                        const uint32_t *opos, const uint32_t *ipos, int32_t *psrc, TT *pair_t,
                        uint4 *gp, uint2 *gn, Entry<TT> *out_adj,
                        Entry<TT> *in_adj, hipStream_t st) {
    if (n_adj == 0) return hipSuccess;
    const dim3 grid(grid_for(n_adj, kIB));
    hipLaunchKernelGGL(pair_entries<TT>, grid, dim3(kIB), 0, st, g, pe, n_adj, psrc, pair_t);
    hipLaunchKernelGGL(pair_links<TT>, grid, dim3(kIB), 0, st, g, pe, n_adj, opos, ipos, psrc,
                       pair_t, gp, gn, out_adj, in_adj);
    return hipGetLastError();
}

template hipError_t sort_pairs<uint32_t>(uint32_t *const[2], uint32_t *const[2], bool, uint32_t,
                                         int, void *, int *, hipStream_t);
template hipError_t sort_pairs<uint64_t>(uint64_t *const[2], uint32_t *const[2], bool, uint32_t,
                                         int, void *, int *, hipStream_t);
#define MG_INGEST(TT)                                                                             \
    template hipError_t launch_time_keys<TT>(const int64_t *, int64_t, uint32_t, TT *,            \
                                             hipStream_t);                                        \
    template hipError_t launch_place_edges<TT>(const int32_t *, const int32_t *, const int64_t *, \
                                               int64_t, const uint32_t *, uint32_t, uint32_t,     \
                                               int32_t *, int32_t *, TT *, uint32_t *,            \
                                               uint32_t *, hipStream_t);                          \
    template hipError_t launch_lists<TT>(const uint32_t *, const uint32_t *, uint32_t, uint32_t,  \
                                         const int32_t *, const TT *, uint32_t *, Entry<TT> *,    \
                                         uint32_t *, hipStream_t);                                \
    template hipError_t launch_ranks<TT>(const DevGraph<TT> &, const uint32_t *,                  \
                                         const uint32_t *, uint4 *, uint2 *, hipStream_t);        \
    template hipError_t launch_pairs<TT>(const DevGraph<TT> &, const uint32_t *, uint32_t,        \
                                         const uint32_t *, const uint32_t *, int32_t *, TT *,     \
                                         uint4 *, uint2 *, Entry<TT> *,         \
                                         Entry<TT> *, hipStream_t);
MG_INGEST(uint32_t)
MG_INGEST(uint64_t)
#undef MG_INGEST

}  // namespace mg
