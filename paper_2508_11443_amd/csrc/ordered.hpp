// Ordered lookups: many needles against a table far larger than the caches.
//
// A lookup in the needles' own order fetches a 128-byte line from HBM for every 16 bytes it reads
// and runs at the device's rate of such lines (about 54 G/s), so the same line is fetched for each
// of the needles that need it.  Here the needles are first grouped by the part of the table that
// answers them, tile by tile (k_ord_group: a counting sort in LDS, written to the tile's own
// place), then every part is answered by the workgroups of one XCD, through whose L2 its lines
// pass once (the structure's own kernel over OrdRuns), and the answers go back to the needles'
// order, tile by tile (k_ord_return).  The two extra passes move about 30 bytes per needle,
// all of it in streams.
//
// 10^7 needles over as many keys: 347 us in their own order, 234 us so (grouping 44, answers 156,
// return 22); 2^26 over 2^26: 2.10 and 1.38 ms.  Runs are kept long (large tiles, few parts): with 512
// parts a run is 30 needles, and its partial lines cost more than the smaller parts gain
// (264 us, 1.60 ms).  Part w mod 8 on each XCD rather than a stretch of neighbours: parts differ
// in needles where keys are clustered, and neighbours alike (a sorted map 632 us instead of 516).
// Reading the next part's lines ahead of their use changed nothing (253 us) or lost (1.74 ms).
//
// Needles that crowd few parts (a key asked again and again, one map of a batch) would leave the
// work to the few workgroups of those parts, on one XCD each, though their lines stay in every L2.  So a
// part's workgroup leaves out runs of more than a kOrdCrowd-th of a tile (twenty times a part's share of
// evenly spread needles), and workgroups of the tile's own answer them, on any XCD.  A tile with more than
// half of its needles in such runs is not grouped at all: its workgroups answer it in the caller's order.
// 10^7 needles over as many keys, one key asked by all of them 701 us and so 95 (41 without grouping), by a
// tenth 253 and 235 (317); a sorted map's 3157 and 272 (137), 426 and 325 (1880); 2^24 needles of a batch
// of 64 maps that all ask one map 2018 and 292 (371), four maps evenly 732 and 366 (434).  The tiles'
// workgroups, idle for evenly spread needles, cost those up to 1 %.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "fks_internal.hpp"
#include "prof.hpp"

namespace fks {

constexpr uint32_t kOrdThreads = 1024;
constexpr uint32_t kOrdBins = 512;          // most parts of a table
constexpr uint32_t kOrdItems = 15;          // needles per thread of a tile: 8 bytes each in LDS ...
constexpr uint32_t kOrdItemsIds = 12;       // ... or 12 with a map id
constexpr uint32_t kOrdRunTiles = 32;        // tiles whose runs of one part a workgroup answers
constexpr uint32_t kOrdBlock = 1024;        // its threads
constexpr uint32_t kOrdCrowd = 12;
constexpr uint32_t kOrdTileBlocks = 2;      // workgroups for a tile's crowded runs ...
constexpr uint32_t kOrdTileShare = 2048;    // ... where they are longer than this
// what a tile leaves to them
enum OrdState : uint16_t { kOrdEven, kOrdCrowded, kOrdDirect };

// Device arrays of one call (m needles in `tiles` tiles of `tile`, the last one short).
struct OrdArgs {
    uint64_t m;
    uint32_t tile, tiles, bins;   // bins: parts of the table, at most kOrdBins
    uint64_t* x;        // needles, every tile grouped by part
    uint32_t* id;       // their map ids (batches)
    uint16_t* slot;     // the place in its tile of every needle of the caller's order
    uint16_t* start;    // tiles x (bins + 2): where a part's run starts in its tile; its end; OrdState
    void* val;          // answers at the needles' places
    uint8_t* found;
    // the caller's arrays
    const uint64_t* q;
    const uint32_t* ids;
    void* vals_out;
    uint8_t* found_out;
};

__host__ __device__ inline uint32_t ord_crowd(const OrdArgs& o) { return o.tile / kOrdCrowd; }   // longest run of an even tile
// (the same for all lanes, and kept so: what depends on it stays in scalar registers)
__device__ __forceinline__ uint32_t ord_state(const OrdArgs& o, uint32_t tile) {
    return (uint32_t)__builtin_amdgcn_readfirstlane((int)o.start[(uint64_t)tile * (o.bins + 2) + o.bins + 1]);
}
__device__ __forceinline__ uint16_t* ord_row(const OrdArgs& o, uint32_t tile) {
    return o.start + (uint64_t)tile * (o.bins + 2);
}

// exclusive scan of one value per thread over the block's first kOrdBins threads
__device__ __forceinline__ uint32_t ord_exscan(uint32_t v, uint32_t* wsum) {
    const uint32_t lane = threadIdx.x & 63u, w = threadIdx.x >> 6;
    uint32_t inc = v;
#pragma unroll
    for (int d = 1; d < 64; d <<= 1) {
        const uint32_t u = __shfl_up(inc, d, 64);
        if (lane >= (uint32_t)d) inc += u;
    }
    if (lane == 63 && w < kOrdBins / 64) wsum[w] = inc;
    __syncthreads();
    uint32_t pre = 0;
#pragma unroll
    for (uint32_t q = 0; q < kOrdBins / 64; ++q) pre += q < w ? wsum[q] : 0u;
    return pre + inc - v;
}

// One tile of needles grouped by part.  Part: setup(lds) once (512 words of LDS), then of(lds, x, id).
template <typename Part, bool IDS>
__global__ __launch_bounds__(kOrdThreads) void k_ord_group(Part part, OrdArgs o) {
    constexpr uint32_t ITEMS = IDS ? kOrdItemsIds : kOrdItems, TILE = kOrdThreads * ITEMS;
    __shared__ uint64_t sx[TILE];
    __shared__ uint32_t sid[IDS ? TILE : 1];
    __shared__ uint32_t cnt[kOrdBins], at[kOrdBins], wsum[kOrdBins / 64], crowded;   // crowded: needles in long runs
    __shared__ uint64_t own[Part::kLds ? Part::kLds : 1];
    const uint64_t* const __restrict__ q = o.q;
    const uint32_t* const __restrict__ ids = o.ids;
    const uint32_t tid = threadIdx.x;
    const uint64_t base = (uint64_t)blockIdx.x * o.tile;
    const uint32_t count = (uint32_t)min((uint64_t)o.tile, o.m - base);   // at most TILE
    uint64_t x[ITEMS];
    uint32_t id[IDS ? ITEMS : 1];
#pragma unroll
    for (uint32_t k = 0; k < ITEMS; ++k) {
        const uint32_t i = tid + k * kOrdThreads;
        x[k] = i < count ? __builtin_nontemporal_load(q + base + i) : 0;
        if (IDS) id[IDS ? k : 0] = i < count ? __builtin_nontemporal_load(ids + base + i) : 0;
    }
    part.setup(own);
    if (tid < kOrdBins) cnt[tid] = 0;
    if (tid == 0) crowded = 0;
    __syncthreads();
    uint32_t bin[ITEMS], rank[ITEMS];
#pragma unroll
    for (uint32_t k = 0; k < ITEMS; ++k) bin[k] = part.of(own, x[k], IDS ? id[IDS ? k : 0] : 0u);
#pragma unroll
    for (uint32_t k = 0; k < ITEMS; ++k) {
        if (tid + k * kOrdThreads < count) {
            // a wave whose needles all fall into one part counts them at once: atomics of 64 lanes
            // on one word would be served one after the other
            const uint32_t first = (uint32_t)__builtin_amdgcn_readfirstlane((int)bin[k]);
            const uint64_t here = __ballot(true);
            if (__all(bin[k] == first)) {
                uint32_t r = 0;
                const uint32_t lane = tid & 63u;
                if (lane == 0) r = atomicAdd(&cnt[first], (uint32_t)__popcll(here));
                rank[k] = (uint32_t)__builtin_amdgcn_readfirstlane((int)r) + lane;
            } else {
                rank[k] = atomicAdd(&cnt[bin[k]], 1u);
            }
        }
    }
    __syncthreads();
    bool direct;
    {
        const uint32_t c = tid < kOrdBins ? cnt[tid] : 0u;
        if (c > ord_crowd(o)) atomicAdd(&crowded, c);
        const uint32_t e = ord_exscan(c, wsum);   // with a barrier
        if (tid < kOrdBins) at[tid] = e;
        direct = 2 * crowded > count;
        uint16_t* const row = ord_row(o, blockIdx.x);
        if (tid <= o.bins) row[tid] = (uint16_t)(direct ? 0u : tid < o.bins ? e : count);
        if (tid == 0) row[o.bins + 1] = direct ? kOrdDirect : crowded ? kOrdCrowded : kOrdEven;
    }
    if (direct) return;   // the whole block
    __syncthreads();
#pragma unroll
    for (uint32_t k = 0; k < ITEMS; ++k) {
        const uint32_t i = tid + k * kOrdThreads;
        if (i < count) {
            const uint32_t e = at[bin[k]] + rank[k];
            sx[e] = x[k];
            if (IDS) sid[IDS ? e : 0] = id[IDS ? k : 0];
            o.slot[base + i] = (uint16_t)e;
        }
    }
    __syncthreads();
#pragma unroll
    for (uint32_t k = 0; k < ITEMS; ++k) {
        const uint32_t i = tid + k * kOrdThreads;
        if (i < count) {
            o.x[base + i] = sx[i];
            if (IDS) o.id[base + i] = sid[IDS ? i : 0];
        }
    }
}

// What a workgroup answers, as one sequence: the runs of one part in kOrdRunTiles consecutive tiles, or
// the crowded runs of one tile, or all of a tile in the caller's order.
struct OrdRuns {
    uint32_t pre[kOrdRunTiles + 1];
    uint64_t src[kOrdRunTiles];
};
static_assert(kOrdCrowd <= kOrdRunTiles, "the crowded runs of a tile are such a sequence");
// where the needles of the sequence are, and their answers go
struct OrdSide {
    const uint64_t* x;
    const uint32_t* id;
    void* val;
    uint8_t* found;
    uint32_t begin;   // where in the sequence the workgroup starts
    bool all_parts;   // the sequence may belong to any part
};
__host__ __device__ inline uint32_t ord_chunks(uint32_t tiles) { return (tiles + kOrdRunTiles - 1) / kOrdRunTiles; }
__host__ __device__ inline uint32_t ord_grouped(const OrdArgs& o) { return ((o.bins + 7) / 8) * 8 * ord_chunks(o.tiles); }
// workgroups of the answering kernel
inline unsigned ord_grid(const OrdArgs& o) { return ord_grouped(o) + o.tiles * kOrdTileBlocks; }
// a tile's workgroup with nothing to do (asked before anything else, as most of them are)
__device__ __forceinline__ bool ord_idle(const OrdArgs& o) {
    const uint32_t grouped = ord_grouped(o);
    return blockIdx.x >= grouped && ord_state(o, (blockIdx.x - grouped) % o.tiles) == kOrdEven;
}
// this workgroup's sequence in R (and its part), from side.begin up to the end that is returned (after a
// barrier); not of an idle one
__device__ __forceinline__ uint32_t ord_runs(const OrdArgs& o, OrdRuns& R, OrdSide& side, uint32_t& part) {
    const uint32_t grouped = ord_grouped(o), crowd = ord_crowd(o), t = threadIdx.x;
    uint32_t len = 0;
    uint64_t at = 0;
    const bool own = blockIdx.x >= grouped;   // a tile's
    const uint32_t tile_of = own ? (blockIdx.x - grouped) % o.tiles : 0;
    const bool direct = own && ord_state(o, tile_of) == kOrdDirect;
    side = OrdSide{direct ? o.q : o.x, direct ? o.ids : o.id, direct ? o.vals_out : o.val,
                   direct ? o.found_out : o.found, 0, own};
    if (!own) {
        // workgroups are dealt to the eight XCDs in turn: all of a part on one of them, the parts of eight
        // in an order that changes, so that parts a constant distance apart do not meet on one
        const uint32_t chunks = ord_chunks(o.tiles), g = blockIdx.x >> 3, eight = g / chunks;
        part = eight * 8 + ((blockIdx.x + eight + (eight >> 3)) & 7u);
        const uint32_t tile = (g % chunks) * kOrdRunTiles + t;
        if (t < kOrdRunTiles && tile < o.tiles && part < o.bins) {
            const uint16_t* const row = ord_row(o, tile);
            at = (uint64_t)tile * o.tile + row[part];
            len = (uint32_t)row[part + 1] - row[part];
            if (len > crowd) len = 0;
        }
    } else {
        const uint16_t* const row = ord_row(o, tile_of);
        const uint64_t base = (uint64_t)tile_of * o.tile;
        part = 0;
        if (direct) {
            at = base;
            len = t == 0 ? (uint32_t)min((uint64_t)o.tile, o.m - base) : 0u;
        } else if (t < 64) {
            uint32_t k = 0;
            for (uint32_t p0 = 0; p0 < o.bins; p0 += 64) {
                const uint32_t p = p0 + t, s = p < o.bins ? row[p] : 0u, l = p < o.bins ? row[p + 1] - s : 0u;
                const uint64_t long_runs = __ballot(l > crowd);
                if (l > crowd) {
                    const uint32_t e = k + (uint32_t)__popcll(long_runs & ((1ull << t) - 1));
                    R.pre[e] = l;
                    R.src[e] = base + s;
                }
                k += (uint32_t)__popcll(long_runs);
            }
            __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
            __builtin_amdgcn_wave_barrier();
            if (t < k) {
                len = R.pre[t];
                at = R.src[t];
            }
            __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
            __builtin_amdgcn_wave_barrier();
        }
    }
    if (t < 64) {
        uint32_t inc = len;
#pragma unroll
        for (int d = 1; d < (int)kOrdRunTiles; d <<= 1) {
            const uint32_t u = __shfl_up(inc, d, 64);
            if (t >= (uint32_t)d) inc += u;
        }
        if (t < kOrdRunTiles) {
            R.pre[t + 1] = inc;
            R.src[t] = at - (inc - len);
        }
        if (t == 0) R.pre[0] = 0;
    }
    __syncthreads();
    const uint32_t all = (uint32_t)__builtin_amdgcn_readfirstlane((int)R.pre[kOrdRunTiles]);
    if (!own) return all;
    const uint32_t share = max(kOrdTileShare, (all + kOrdTileBlocks - 1) / kOrdTileBlocks);
    side.begin = min(all, (blockIdx.x - grouped) / o.tiles * share);
    return min(all, side.begin + share);
}
// the place of needle i of the sequence
__device__ __forceinline__ uint64_t ord_place(const OrdRuns& R, uint32_t i) {
    uint32_t r = 0;
#pragma unroll
    for (uint32_t st = kOrdRunTiles >> 1; st; st >>= 1) r += R.pre[r + st] <= i ? st : 0u;
    return R.src[r] + i;
}

// One tile of answers back in the caller's order.  Four neighbours per thread and access, all
// loads in flight before the first is used: 2^26 answers 129 us, 215 with one access of 1, 2 or 4
// bytes per needle; 10^7 22 and 35.  Bound by its streams, 12 bytes per needle.  The caller's arrays may start
// anywhere their type allows: whole vectors are stored where they are aligned.
template <typename T>
using OrdVec4 = T __attribute__((ext_vector_type(4)));

template <typename V, uint32_t TILE>
__global__ __launch_bounds__(kOrdThreads) void k_ord_return(OrdArgs o) {
    if (ord_state(o, blockIdx.x) == kOrdDirect) return;   // the whole block
    V* const __restrict__ vals = (V*)o.vals_out;
    uint8_t* const __restrict__ found = o.found_out;
    constexpr uint32_t ITEMS = (TILE / 4 + kOrdThreads - 1) / kOrdThreads;
    __shared__ __attribute__((aligned(16))) V sv[TILE];
    __shared__ __attribute__((aligned(16))) uint8_t sf[TILE];
    const uint64_t base = (uint64_t)blockIdx.x * o.tile;   // a multiple of 64
    const uint32_t count = (uint32_t)min((uint64_t)o.tile, o.m - base), tid = threadIdx.x;   // at most TILE
    const uint32_t fours = count / 4;
    const V* val = (const V*)o.val + base;
    const OrdVec4<uint16_t>* slot4 = (const OrdVec4<uint16_t>*)(o.slot + base);
    const OrdVec4<V>* val4 = (const OrdVec4<V>*)val;
    const uint32_t* found4 = (const uint32_t*)(o.found + base);
    OrdVec4<uint16_t> slot[ITEMS];
    OrdVec4<V> v[ITEMS];
    uint32_t f[ITEMS];
    if (fours) {
#pragma unroll
        for (uint32_t k = 0; k < ITEMS; ++k) {
            const uint32_t i = min(tid + k * kOrdThreads, fours - 1);
            slot[k] = __builtin_nontemporal_load(slot4 + i);
            if (vals) v[k] = __builtin_nontemporal_load(val4 + i);
            if (found) f[k] = __builtin_nontemporal_load(found4 + i);
        }
#pragma unroll
        for (uint32_t k = 0; k < ITEMS; ++k) {
            const uint32_t i = tid + k * kOrdThreads;
            if (i < fours) {
                if (vals) ((OrdVec4<V>*)sv)[i] = v[k];
                if (found) ((uint32_t*)sf)[i] = f[k];
            }
        }
    }
    const uint32_t rest = fours * 4 + tid;   // fewer than four, by as many threads
    if (rest < count) {
        if (vals) sv[rest] = val[rest];
        if (found) sf[rest] = o.found[base + rest];
    }
    __syncthreads();
    V* const vout = vals ? vals + base : nullptr;
    uint8_t* const fout = found ? found + base : nullptr;
    const bool whole_v = ((uintptr_t)vout & (sizeof(OrdVec4<V>) - 1)) == 0, whole_f = ((uintptr_t)fout & 3u) == 0;
#pragma unroll
    for (uint32_t k = 0; k < ITEMS; ++k) {
        const uint32_t i = tid + k * kOrdThreads;
        if (i >= fours) break;
        const OrdVec4<uint16_t> e = slot[k];
        if (vals) {
            const OrdVec4<V> r = {sv[e.x], sv[e.y], sv[e.z], sv[e.w]};
            if (whole_v) {
                __builtin_nontemporal_store(r, (OrdVec4<V>*)vout + i);
            } else {
#pragma unroll
                for (uint32_t c = 0; c < 4; ++c) __builtin_nontemporal_store(r[c], vout + 4 * i + c);
            }
        }
        if (found) {
            const uint32_t r = sf[e.x] | (uint32_t)sf[e.y] << 8 | (uint32_t)sf[e.z] << 16 | (uint32_t)sf[e.w] << 24;
            if (whole_f) {
                __builtin_nontemporal_store(r, (uint32_t*)fout + i);
            } else {
#pragma unroll
                for (uint32_t c = 0; c < 4; ++c) __builtin_nontemporal_store((uint8_t)(r >> (8 * c)), fout + 4 * i + c);
            }
        }
    }
    if (rest < count) {
        const uint32_t e = o.slot[base + rest];
        if (vals) vout[rest] = sv[e];
        if (found) fout[rest] = sf[e];
    }
}

// ---- host side ---------------------------------------------------------------------------

constexpr uint64_t kOrdSlice = 1ull << 27;   // needles at a time: 2 GB of scratch
constexpr uint32_t ord_tile_max(bool ids) { return kOrdThreads * (ids ? kOrdItemsIds : kOrdItems); }
// Tiles of a size that gives all 256 CUs equally many (a CU holds one workgroup of the grouping
// pass): 2^22 needles 84 us (88 with tiles of 15360), 10^7 239 (243), 2^24 358 (368).  With map ids the
// tiles are smaller to begin with, and shorter runs cost what even rounds gain.
inline uint32_t ord_tile(uint64_t m, bool ids) {
    if (ids) return ord_tile_max(ids);
    const uint64_t round = 256ull * ord_tile_max(ids), rounds = (m + round - 1) / round;
    const uint64_t tile = (m + 256 * rounds - 1) / (256 * rounds);
    return (uint32_t)((tile + 63) & ~63ull);
}

// Scratch of one call on stream s, given back in stream order when it goes out of scope.
class OrdScratch {
  public:
    // false: no memory, or the stream is being captured (a graph would keep the scratch)
    OrdScratch(uint64_t m, uint32_t bins, bool ids, uint32_t val_bytes, bool found, hipStream_t s, size_t more = 0);
    void* more() const { return more_; }   // as many bytes for the caller
    ~OrdScratch();
    OrdScratch(const OrdScratch&) = delete;
    OrdScratch& operator=(const OrdScratch&) = delete;
    explicit operator bool() const { return base_ != nullptr; }
    // for a slice of m needles; vals, found may be null
    template <typename V>
    OrdArgs part(uint64_t m, const uint64_t* q, const uint32_t* ids, V* vals, uint8_t* found) const {
        OrdArgs a = a_;
        a.m = m;
        a.tiles = (uint32_t)((m + a.tile - 1) / a.tile);
        a.q = q;
        a.ids = ids;
        a.vals_out = vals;
        a.found_out = found;
        return a;
    }

  private:
    OrdArgs a_{};
    void *base_ = nullptr, *more_ = nullptr;
    hipStream_t st_;
};

// parts for a table of that many bytes; 0: the lookup stays in the caller's order
uint32_t ord_parts(uint64_t m, uint64_t table_bytes);

template <typename Part, bool IDS>
void ord_group(const Part& part, const OrdArgs& a, hipStream_t st) {
    FKS_TIMED("fks_order_group", st,
              hipLaunchKernelGGL((k_ord_group<Part, IDS>), a.tiles, kOrdThreads, 0, st, part, a));
}
template <typename V, bool IDS>
void ord_return(const OrdArgs& a, hipStream_t st) {
    FKS_TIMED("fks_order_return", st,
              hipLaunchKernelGGL((k_ord_return<V, ord_tile_max(IDS)>), a.tiles, kOrdThreads, 0, st, a));
}

}  // namespace fks
