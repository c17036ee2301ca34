// Partitioned construction: the level-one attempt as a few streaming passes.
//
// Buckets are cut into partitions of 1024 consecutive buckets (q = j >> 10).  Keys are
// moved into partition order by one to three coalescing radix passes over q (at most 8
// bits, 256 bins, per pass, so every 12288-record tile writes runs of about 48 records per
// bin); each worker's runs go to offsets from a scanned count matrix, or are reserved with
// one atomic add per (tile, bin) on a cursor into a fixed-capacity region.  Then every
// partition is finished by one workgroup that holds its ~1024 keys in LDS: ranks from an
// LDS histogram, scan of the 128 group statistics, grouping, the per-bucket level-two
// search of make_2, and the coalesced write of the partition's contiguous cells and group
// headers.  Only the partition totals of squared sizes (the offsets of Section 2.2, at
// partition granularity) cross partitions: either a size pass and a scan turn them into
// cell bases and the table size S, or the final pass publishes each total and finds its
// own base by a look-back over its predecessors'.  Device-scope atomics serve only the
// cursors, the final pass's look-back words, and an attempt's outcome flags;
// every per-key access is a coalesced stream or LDS.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <type_traits>

#include "fks_internal.hpp"
#include "partition.hpp"
#include "prof.hpp"

namespace fks {

constexpr uint32_t kPB = 256;                 // threads per block, partition passes
constexpr uint32_t kPItems = 16;              // keys per thread per tile
constexpr uint32_t kPTile = kPB * kPItems;    // 4096 keys per tile
// scatter tiles of the single-map passes: 1024 threads x 12 records (12288 records, runs of ~48
// per bin, 149 KB of LDS: one workgroup and four waves per SIMD on a CU), or x 8 when an aux
// word travels (16-byte records, 8192-record tiles, 133 KB)
constexpr uint32_t kPScatterThreads = 1024, kPScatterItems = 12, kPScatterItemsAux = 8;
constexpr uint32_t kBins = 256;               // bins per scatter pass
// Keys from which every XCD has regions of its own in the first pass's bins (with an aux word in
// every record, and without): where the records outgrow the 256 MiB Infinity Cache, which merges
// what the L2s write in pieces.  Build, one lookup and release with one region per bin and with
// eight: 1.6 * 10^7 keys with 64-bit values 581 and 566 us, 3.3 * 10^7 1171 and 1091, 2^26 2336 and 2120; without
// aux words 2.4 * 10^7 613 and 628, 3.3 * 10^7 848 and 846, 2^26 1671 and 1604.
constexpr uint64_t kSubRegionKeysAux = 1ull << 24, kSubRegionKeys = 1ull << 25;
constexpr uint32_t kFinalKeyCap = 1248;       // keys of one partition held in LDS (mean 1024, sd 32)
constexpr uint32_t kLdsTrials = 16;          // level-two triples held in the final pass's LDS (larger trials are rare)
constexpr uint32_t kFinalCellCap = 3072;      // cells of one partition staged in LDS (mean <= 2048, sd ~106)
constexpr uint32_t kGroupsPerPart = kPartBuckets / 8;

__global__ void k_zero_words(uint32_t* __restrict__ p, uint64_t count) {
    for (uint64_t i = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; i < count;
         i += (uint64_t)gridDim.x * blockDim.x)
        p[i] = 0;
}

__device__ __forceinline__ uint32_t bucket_of(const Triple& A, uint64_t magic, uint32_t n, uint64_t x) {
    return fastmod(mshash(A, x), magic, n);
}

// Worker bx of W in segment by: segment = the whole input
// (ranges == nullptr) or [ranges[s], ranges[s+1]); the worker owns one
// contiguous chunk of it and walks the chunk in tiles, so that counting and
// scattering see the keys in the same order.
__device__ __forceinline__ void worker_range(uint32_t bx, uint32_t by, const uint64_t* ranges, uint64_t n, uint32_t W, uint64_t& a,
                                             uint64_t& b, const uint64_t* ranges_hi = nullptr,
                                             uint64_t hi_cap = 0) {
    uint64_t lo = 0, hi = n;
    if (ranges) {
        lo = ranges[by];
        // a cursor that ran past its region's end (overflow raised) stops at the end
        hi = ranges_hi ? min(ranges_hi[by], lo + hi_cap) : ranges[by + 1];
    }
    const uint64_t chunk = (hi - lo + W - 1) / W;
    a = min(hi, lo + (uint64_t)bx * chunk);
    b = min(hi, a + chunk);
}

// counts of one worker per bin: cnt[(segment * 256 + bin) * W + worker]
__global__ __launch_bounds__(kPB) void k_dcount(const uint64_t* __restrict__ keys, uint64_t n, Triple A,
                                                  uint64_t magic, const uint64_t* __restrict__ ranges, uint32_t W,
                                                  uint32_t shift, uint32_t mask, uint32_t* __restrict__ cnt) {
    __shared__ uint32_t bins[kBins];
    uint64_t a, b;
    worker_range(blockIdx.x, blockIdx.y, ranges, n, W, a, b);
    for (uint32_t k = threadIdx.x; k < kBins; k += kPB) bins[k] = 0;
    __syncthreads();
    for (uint64_t ts = a; ts < b; ts += kPTile) {
        uint64_t x[kPItems];
#pragma unroll
        for (uint32_t k = 0; k < kPItems; ++k) {
            const uint64_t i = ts + threadIdx.x + (uint64_t)k * kPB;
            x[k] = i < b ? keys[i] : 0;
        }
#pragma unroll
        for (uint32_t k = 0; k < kPItems; ++k) {
            const uint64_t i = ts + threadIdx.x + (uint64_t)k * kPB;
            if (i < b) {
                const uint32_t q = bucket_of(A, magic, (uint32_t)n, x[k]) >> kPartBits;
                atomicAdd(&bins[(q >> shift) & mask], 1u);
            }
        }
    }
    __syncthreads();
    for (uint32_t k = threadIdx.x; k < kBins; k += kPB)
        cnt[((uint64_t)blockIdx.y * kBins + k) * W + blockIdx.x] = bins[k];
}

// exclusive scan of 256 per-thread values across the block (one value per thread)
__device__ __forceinline__ uint32_t block_exscan256(uint32_t v, uint32_t* wsum) {
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    uint32_t inc = v;
#pragma unroll
    for (int d = 1; d < 64; d <<= 1) {
        const uint32_t u = __shfl_up(inc, d, 64);
        if (lane >= d) inc += u;
    }
    if (lane == 63) wsum[w] = inc;
    __syncthreads();
    uint32_t pre = 0;
    for (int q = 0; q < w; ++q) pre += wsum[q];
    __syncthreads();
    return pre + inc - v;
}

// Scatter of one worker's chunk: every tile is sorted by bin in LDS, then each
// bin's run is written to consecutive addresses from the worker's scanned
// offset (no device atomics; the output order is a function of the input).
// BT threads per block (at least one per bin), ITEMS records per thread per tile
// CURSOR: instead of offsets from a count matrix, every tile reserves each bin's run with
// one atomic add on the bin's cursor (bins are fixed-capacity regions: bin i of segment s
// owns [(s * (mask + 1) + i) * cap, ... + cap)); records that would land beyond their
// region are dropped and *overflow is raised, so the attempt can be redone with counts.
// Segment s reads [ranges[s], ranges_hi[s]).  The order of records inside a bin then
// depends on timing, which the final pass does not see: its table depends only on which
// records each partition holds.
// segs (a batch): workgroup x takes tile x of the list, records of one wide map with its own
// hash, to the map's partitions; an overflow rejects the map alone (overflow: four words per map).
template <bool AUX, uint32_t ITEMS, uint32_t BT = kPB, bool CURSOR = false>
__global__ __launch_bounds__(BT) void k_dscatter(const uint64_t* __restrict__ keys,
                                                    const uint32_t* __restrict__ vals,
                                                    const uint32_t* __restrict__ aux, uint64_t n, Triple A,
                                                    uint64_t magic, const uint64_t* __restrict__ ranges, uint32_t W,
                                                    uint32_t shift, uint32_t mask, const uint32_t* __restrict__ off,
                                                    uint64_t* __restrict__ keys_out, uint32_t* __restrict__ vals_out,
                                                    uint32_t* __restrict__ aux_out,
                                                    const WideSeg* __restrict__ segs = nullptr,
                                                    const uint2* __restrict__ tiles = nullptr,
                                                    unsigned long long* __restrict__ cursor = nullptr,
                                                    const uint64_t* __restrict__ ranges_hi = nullptr,
                                                    uint64_t cap = 0, uint32_t* __restrict__ overflow = nullptr,
                                                    uint64_t in_cap = 0, uint32_t subs = 0, uint32_t in_subs = 0,
                                                    const uint64_t* __restrict__ pairs = nullptr) {
    __shared__ uint64_t skey[(BT * ITEMS)];
    __shared__ uint32_t sval[(BT * ITEMS)];
    __shared__ uint32_t saux[AUX ? (BT * ITEMS) : 1];
    __shared__ uint32_t run[kBins], tcnt[kBins], toff[kBins];
    __shared__ uint32_t wsum[BT / 64];
    static_assert(BT >= kBins && BT % 64 == 0, "one bin per thread");
    __shared__ uint64_t lim[CURSOR ? kBins : 1];
    // Workgroups are dealt to the XCDs in turn, and a line that several runs share is written to memory
    // whole only if they meet in one XCD's L2.  So all workers of a bin of the first pass go to one
    // XCD, and with subs > 0 (the first pass itself) every XCD has regions of its own in each bin.
    // 2^26 records of 12 bytes: second pass 461 and 375 us, first pass 425 and 364.
    uint32_t bx = blockIdx.x, by = blockIdx.y;
    if (CURSOR && gridDim.y > 1) {
        const uint32_t per = gridDim.x << in_subs, bins = gridDim.y >> in_subs;   // workgroups of a bin, bins
        const uint32_t l = by * gridDim.x + bx, turn = l >> 3;
        if (l < (bins & ~7u) * per) {
            by = (((turn / per) * 8 + (l & 7u)) << in_subs) + turn % per / gridDim.x;
            bx = turn % gridDim.x;
        }
    }
    // the regions and cursors of the bins: bin0, bin0 + step, ...
    uint64_t a, b, bin0 = (uint64_t)(by >> in_subs) * (mask + 1);
    uint32_t step = 1;
    if (CURSOR && subs) {
        bin0 = bx & 7u;
        step = 8;
    }
    if (CURSOR && segs) {
        // neighbours in the list, a map's tiles among them, on one XCD
        const uint32_t each = gridDim.x >> 3, l = blockIdx.x;
        const uint2 t = tiles[l < 8 * each ? (l & 7u) * each + (l >> 3) : l];
        const WideSeg& sg = segs[t.x];
        A = sg.A;
        magic = sg.magic;
        n = sg.n;
        a = sg.in_lo + t.y;
        b = min(a + (sg.n + sg.tiles - 1) / sg.tiles, sg.in_hi);
        bin0 = sg.part0;
        overflow += 4 * t.x;
    } else {
        worker_range(bx, by, ranges, n, W, a, b, ranges_hi, in_cap);
    }
    const uint32_t tid = threadIdx.x;
    if (!CURSOR && tid < kBins) run[tid] = off[((uint64_t)by * kBins + tid) * W + bx];
    if (CURSOR && tid < kBins) lim[tid] = (bin0 + tid * step + 1) * cap;
    // a tile's records are loaded into registers one tile ahead: the loads of
    // tile i+1 are in flight while tile i is written out
    uint64_t x[ITEMS];
    uint32_t v[ITEMS], u[AUX ? ITEMS : 1];
    auto load = [&](uint64_t ts) {
        if (AUX && pairs) {   // 64-bit values: low halves as values, high as aux words
#pragma unroll
            for (uint32_t k = 0; k < ITEMS; ++k) {
                const uint64_t i = ts + tid + (uint64_t)k * BT;
                x[k] = i < b ? keys[i] : 0;
                const uint64_t p = i < b ? pairs[i] : 0;
                v[k] = (uint32_t)p;
                u[AUX ? k : 0] = (uint32_t)(p >> 32);
            }
            return;
        }
#pragma unroll
        for (uint32_t k = 0; k < ITEMS; ++k) {
            const uint64_t i = ts + tid + (uint64_t)k * BT;
            x[k] = i < b ? keys[i] : 0;
            v[k] = i < b ? vals[i] : 0;
            if (AUX) u[AUX ? k : 0] = i < b ? (aux ? aux[i] : (uint32_t)i) : 0;
        }
    };
    if (a < b) load(a);
    for (uint64_t ts = a; ts < b; ts += (BT * ITEMS)) {
        if (tid < kBins) tcnt[tid] = 0;
        __syncthreads();
        uint32_t bin[ITEMS], rank[ITEMS];
#pragma unroll
        for (uint32_t k = 0; k < ITEMS; ++k) {
            const uint64_t i = ts + tid + (uint64_t)k * BT;
            if (i < b) {
                const uint32_t q = bucket_of(A, magic, (uint32_t)n, x[k]) >> kPartBits;
                bin[k] = (q >> shift) & mask;
                rank[k] = atomicAdd(&tcnt[bin[k]], 1u);
            }
        }
        __syncthreads();
        if (CURSOR && tid <= mask && tcnt[tid]) {
            // this tile's run of bin tid: reserved now, written after the tile is sorted
            const unsigned long long at =
                atomicAdd(&cursor[bin0 + tid * step], (unsigned long long)tcnt[tid]);
            run[tid] = (uint32_t)at;
            if (at + tcnt[tid] > lim[tid]) atomicOr(overflow, 1u);
        }
        {
            const uint32_t e = block_exscan256(tid < kBins ? tcnt[tid] : 0u, wsum);
            if (tid < kBins) toff[tid] = e;
        }
        __syncthreads();
#pragma unroll
        for (uint32_t k = 0; k < ITEMS; ++k) {
            const uint64_t i = ts + tid + (uint64_t)k * BT;
            if (i < b) {
                const uint32_t e = toff[bin[k]] + rank[k];
                skey[e] = x[k];
                sval[e] = v[k];
                if (AUX) saux[e] = u[AUX ? k : 0];
            }
        }
        if (ts + (BT * ITEMS) < b) load(ts + (BT * ITEMS));
        __syncthreads();
        const uint32_t cnt = (uint32_t)min((uint64_t)(BT * ITEMS), b - ts);
        for (uint32_t e = tid; e < cnt; e += BT) {
            // the bin is hashed again rather than staged in LDS: the pass waits on memory,
            // and a staged byte per record measured the same
            const uint32_t bb = ((bucket_of(A, magic, (uint32_t)n, skey[e]) >> kPartBits) >> shift) & mask;
            const uint64_t dest = (uint64_t)run[bb] + (e - toff[bb]);
            if (CURSOR && dest >= lim[bb]) continue;   // beyond the bin's region: dropped, overflow raised
            keys_out[dest] = skey[e];
            vals_out[dest] = sval[e];
            if (AUX) aux_out[dest] = saux[e];
        }
        __syncthreads();
        if (!CURSOR && tid < kBins) run[tid] += tcnt[tid];
    }
}

// The set-up of an attempt in one launch: the outcome words cleared and the level-two triples
// written (start), the cursor of fixed-capacity region i of either pass at i * cap (begin[i] keeps
// that start), the one partition of an input without passes, and the fused final pass's look-back
// words (nzw words) at zero.  A launch costs a small build more than its work does: these
// were one to four of its four to seven.
__global__ void k_attempt_init(AttemptStart start, unsigned long long* __restrict__ cur1, uint64_t* __restrict__ beg1,
                               uint64_t count1, uint64_t cap1, unsigned long long* __restrict__ cur2,
                               uint64_t* __restrict__ beg2, uint64_t count2, uint64_t cap2,
                               uint64_t* __restrict__ one, uint64_t n, uint32_t* __restrict__ zw, uint64_t nzw) {
    const uint64_t stride = (uint64_t)gridDim.x * blockDim.x;
    for (uint64_t i = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; i < count1 + count2 + nzw; i += stride) {
        if (i < count1) {
            cur1[i] = i * cap1;
            beg1[i] = i * cap1;
        } else if (i < count1 + count2) {
            const uint64_t j = i - count1;
            cur2[j] = j * cap2;
            beg2[j] = j * cap2;
        } else {
            zw[i - count1 - count2] = 0;
        }
    }
    if (blockIdx.x != 0) return;
    if (threadIdx.x < start.words) start.clear[threadIdx.x] = 0;
    for (uint32_t t = threadIdx.x; t < start.T; t += blockDim.x) start.C[t] = level2_triple(start.seed, start.r, t);
    if (threadIdx.x == 0 && one) {
        one[0] = 0;
        one[1] = n;
    }
}

// ---- exclusive scan of a u32 array across blocks (values sum below 2^32) --------------------

constexpr uint32_t kXItems = 8;
constexpr uint32_t kXTile = kPB * kXItems;

__global__ __launch_bounds__(kPB) void k_xscan_reduce(const uint32_t* __restrict__ in, uint64_t N,
                                                        uint32_t* __restrict__ tsum) {
    __shared__ uint32_t wsum[kPB / 64];
    const uint64_t base = (uint64_t)blockIdx.x * kXTile + (uint64_t)threadIdx.x * kXItems;
    uint32_t s = 0;
#pragma unroll
    for (uint32_t k = 0; k < kXItems; ++k)
        if (base + k < N) s += in[base + k];
    for (int d = 32; d >= 1; d >>= 1) s += __shfl_xor(s, d, 64);
    if ((threadIdx.x & 63) == 0) wsum[threadIdx.x >> 6] = s;
    __syncthreads();
    if (threadIdx.x == 0) {
        uint32_t t = 0;
        for (uint32_t w = 0; w < kPB / 64; ++w) t += wsum[w];
        tsum[blockIdx.x] = t;
    }
}

__global__ __launch_bounds__(kPB) void k_xscan_down(const uint32_t* __restrict__ in, uint64_t N,
                                                      const uint64_t* __restrict__ tpre, uint32_t* __restrict__ out) {
    __shared__ uint32_t wsum[kPB / 64];
    const uint64_t base = (uint64_t)blockIdx.x * kXTile + (uint64_t)threadIdx.x * kXItems;
    uint32_t v[kXItems];
    uint32_t s = 0;
#pragma unroll
    for (uint32_t k = 0; k < kXItems; ++k) {
        v[k] = base + k < N ? in[base + k] : 0u;
        s += v[k];
    }
    uint32_t run = (uint32_t)tpre[blockIdx.x] + block_exscan256(s, wsum);
#pragma unroll
    for (uint32_t k = 0; k < kXItems; ++k) {
        if (base + k < N) out[base + k] = run;
        run += v[k];
    }
}

// the same downsweep with 64-bit outputs; out[N] = the total (tpre[tiles])
__global__ __launch_bounds__(kPB) void k_xscan_down64(const uint32_t* __restrict__ in, uint64_t N,
                                                        const uint64_t* __restrict__ tpre,
                                                        uint64_t* __restrict__ out) {
    __shared__ uint32_t wsum[kPB / 64];
    const uint64_t base = (uint64_t)blockIdx.x * kXTile + (uint64_t)threadIdx.x * kXItems;
    uint32_t v[kXItems];
    uint32_t s = 0;
#pragma unroll
    for (uint32_t k = 0; k < kXItems; ++k) {
        v[k] = base + k < N ? in[base + k] : 0u;
        s += v[k];
    }
    uint64_t run = tpre[blockIdx.x] + block_exscan256(s, wsum);
#pragma unroll
    for (uint32_t k = 0; k < kXItems; ++k) {
        if (base + k < N) out[base + k] = run;
        run += v[k];
    }
    if (blockIdx.x == gridDim.x - 1 && threadIdx.x == 0) out[N] = tpre[gridDim.x];
}

// offsets of bins from a scanned count matrix: out[i] = off[((i >> bits) * 256 + (i & mask)) * W]
// for i < count, out[count] = total
__global__ void k_extract_offsets(const uint32_t* __restrict__ off, uint32_t W, uint32_t bits, uint32_t count,
                                  uint64_t total, uint64_t* __restrict__ out) {
    const uint32_t mask = (1u << bits) - 1;
    for (uint32_t i = blockIdx.x * blockDim.x + threadIdx.x; i <= count; i += gridDim.x * blockDim.x)
        out[i] = i < count ? (uint64_t)off[((uint64_t)(i >> bits) * kBins + (i & mask)) * W] : total;
}

// single block: exclusive prefix of cnt[0..N) into off (u64), copy into cursor,
// off[N] = total; the total also into *total when given
__global__ __launch_bounds__(1024) void k_scan_counts(const uint32_t* __restrict__ cnt, uint32_t N,
                                                        uint64_t* __restrict__ off, uint64_t* __restrict__ cursor,
                                                        uint64_t* __restrict__ total) {
    __shared__ uint64_t part[1024];
    const uint32_t per = (N + 1023) / 1024;
    const uint32_t a = threadIdx.x * per, b = min(N, a + per);
    uint64_t s = 0;
    for (uint32_t i = a; i < b; ++i) s += cnt[i];
    part[threadIdx.x] = s;
    __syncthreads();
    for (uint32_t d = 1; d < 1024; d <<= 1) {
        const uint64_t v = threadIdx.x >= d ? part[threadIdx.x - d] : 0;
        __syncthreads();
        part[threadIdx.x] += v;
        __syncthreads();
    }
    uint64_t run = part[threadIdx.x] - s;
    for (uint32_t i = a; i < b; ++i) {
        off[i] = run;
        if (cursor) cursor[i] = run;
        run += cnt[i];
    }
    if (threadIdx.x == 1023) {
        off[N] = part[1023];
        if (total) *total = part[1023];
    }
}

// per partition: 4-bit bucket sizes (written to the global size words) and the
// partition's sum of squared sizes
__global__ __launch_bounds__(kPB) void k_psizes(const uint64_t* __restrict__ keys, uint64_t n, Triple A,
                                                  uint64_t magic, const uint64_t* __restrict__ offQ,
                                                  uint32_t* __restrict__ sizes, uint64_t G,
                                                  uint32_t* __restrict__ sq_out, uint32_t* __restrict__ oversize) {
    __shared__ uint32_t words[kGroupsPerPart];
    __shared__ uint32_t red[kPB / 64];
    const uint32_t q = blockIdx.x;
    for (uint32_t g = threadIdx.x; g < kGroupsPerPart; g += kPB) words[g] = 0;
    __syncthreads();
    const uint64_t lo = offQ[q], hi = offQ[q + 1];
    bool over = false;
    auto count = [&](uint64_t x) {
        const uint32_t lb = bucket_of(A, magic, (uint32_t)n, x) & (kPartBuckets - 1);
        const uint32_t sh = 4 * (lb & 7u);
        const uint32_t old = atomicAdd(&words[lb >> 3], 1u << sh);
        over |= ((old >> sh) & 15u) == 15u;
    };
    // a typical partition's keys are all loaded before the first is hashed
    constexpr uint32_t KPT = 5;
    uint64_t x[KPT];
#pragma unroll
    for (uint32_t k = 0; k < KPT; ++k) {
        const uint64_t i = lo + threadIdx.x + (uint64_t)k * kPB;
        x[k] = i < hi ? keys[i] : 0;
    }
#pragma unroll
    for (uint32_t k = 0; k < KPT; ++k)
        if (lo + threadIdx.x + (uint64_t)k * kPB < hi) count(x[k]);
    for (uint64_t i = lo + threadIdx.x + (uint64_t)KPT * kPB; i < hi; i += kPB) count(keys[i]);
    if (over) atomicOr(oversize, 1u);
    __syncthreads();
    uint32_t sq = 0;
    for (uint32_t g = threadIdx.x; g < kGroupsPerPart; g += kPB) {
        const uint32_t w = words[g];
        if ((uint64_t)q * kGroupsPerPart + g < G) sizes[(uint64_t)q * kGroupsPerPart + g] = w;
#pragma unroll
        for (int k = 0; k < 8; ++k) {
            const uint32_t s = nib(w, k);
            sq += s * s;
        }
    }
    for (int d = 32; d >= 1; d >>= 1) sq += __shfl_xor(sq, d, 64);
    if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = sq;
    __syncthreads();
    if (threadIdx.x == 0) {
        uint32_t t = 0;
        for (uint32_t w = 0; w < kPB / 64; ++w) t += red[w];
        sq_out[q] = t;
    }
}

__device__ __forceinline__ bool test_set4(uint64_t& m0, uint64_t& m1, uint64_t& m2, uint64_t& m3, uint32_t h) {
    const uint64_t bit = 1ull << (h & 63u);
    const uint32_t w = h >> 6;
    const uint64_t cur = w == 0 ? m0 : w == 1 ? m1 : w == 2 ? m2 : m3;
    if (cur & bit) return true;
    if (w == 0) m0 |= bit;
    else if (w == 1) m1 |= bit;
    else if (w == 2) m2 |= bit;
    else m3 |= bit;
    return false;
}

template <typename KeyAt>
__device__ __forceinline__ uint32_t min_trial(const Triple* C, uint32_t T, uint32_t s, KeyAt key_at,
                                              uint32_t t0 = 0) {
    const uint32_t s2 = s * s;
    for (uint32_t t = t0; t < T; ++t) {
        const Triple c = C[t];
        uint64_t m0 = 0, m1 = 0, m2 = 0, m3 = 0;
        bool collide = false;
        for (uint32_t i = 0; i < s && !collide; ++i) collide = test_set4(m0, m1, m2, m3, mshash(c, key_at(i)) % s2);
        if (!collide) return t;
    }
    return T;
}

__device__ __forceinline__ bool same_string(const int64_t* off, const uint8_t* bytes, uint32_t a, uint32_t b) {
    const int64_t la = off[a + 1] - off[a], lb = off[b + 1] - off[b];
    if (la != lb) return false;
    const uint8_t* pa = bytes + off[a];
    const uint8_t* pb = bytes + off[b];
    for (int64_t i = 0; i < la; ++i)
        if (pa[i] != pb[i]) return false;
    return true;
}

// Keys (14 bits: at most 15 * 1024) and cells (18 bits: at most 225 * 1024) of a partition up to some
// point, in one word, so that one scan and one LDS read serve both.
__device__ __forceinline__ uint32_t pos_of(uint32_t keys, uint32_t cells) { return cells << 14 | keys; }
__device__ __forceinline__ uint32_t pos_keys(uint32_t pos) { return pos & 0x3FFFu; }
__device__ __forceinline__ uint32_t pos_cells(uint32_t pos) { return pos >> 14; }
// of the buckets in a size word: byte-wise dot products over its even and its odd nibbles
__device__ __forceinline__ uint32_t word_pos(uint32_t w) {
    const uint32_t e = w & 0x0F0F0F0Fu, o = (w >> 4) & 0x0F0F0F0Fu;
    return pos_of(__builtin_amdgcn_udot4(e, 0x01010101u, __builtin_amdgcn_udot4(o, 0x01010101u, 0u, false), false),
                  __builtin_amdgcn_udot4(e, e, __builtin_amdgcn_udot4(o, o, 0u, false), false));
}
// where bucket kk of a group starts: its group's start and the buckets before it
__device__ __forceinline__ uint32_t bucket_pos(uint64_t gpos, uint32_t kk) {
    return (uint32_t)(gpos >> 32) + word_pos((uint32_t)gpos & ~(~0u << (4 * kk)));
}

// inclusive prefix sums over the wave's lanes (all active)
__device__ __forceinline__ uint32_t wave_scan(uint32_t v) {
    v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x111, 0xF, 0xF, false);   // from 1 lane to the left, by rows of 16
    v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x112, 0xF, 0xF, false);
    v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x114, 0xF, 0xF, false);
    v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x118, 0xF, 0xF, false);
    v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x142, 0xA, 0xF, false);   // lane 15 of a row to rows 1 and 3
    v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x143, 0xC, 0xF, false);   // lane 31 to the upper half
    return v;
}

// remainder magic of s^2 for s = 1..15 (fastmod_magic, whose 64-bit division is a chain of a
// hundred instructions)
struct SquareMagics {
    uint64_t m[16];
    constexpr SquareMagics() : m() {
        for (uint32_t s = 1; s < 16; ++s) m[s] = 0xFFFFFFFFFFFFFFFFull / (s * s) + 1;
    }
};
__constant__ const SquareMagics kSquareMagics{};

template <bool AUX>
struct FinalLds {
    uint64_t key[kFinalKeyCap];
    uint32_t val[kFinalKeyCap];
    uint32_t aux[AUX ? kFinalKeyCap : 1];
    uint16_t smap[kFinalCellCap];
    uint32_t cnt2[kGroupsPerPart];      // bucket sizes counted while ranking, 4 bits each
    uint64_t gpos[kGroupsPerPart];      // a group's size word, and above it where its keys and cells start (pos_of)
    alignas(4) uint8_t tb[kPartBuckets];
    uint32_t occ[kFinalCellCap / 32];   // cells taken by trial 0
    uint32_t fl[kPartBuckets / 32];     // buckets where trial 0 collides
    uint16_t hard[kFinalKeyCap / 2];   // buckets of two or more keys that trial 0 does not place
    uint64_t mag[16];             // remainder magic of s^2, s = 0..15
    Triple tri[kLdsTrials];       // the first level-two triples (larger trials are rare)
    uint32_t nhard;
    uint32_t wsum;       // the first wave's groups
    uint32_t flags[3];   // exhausted, dup, max_t
    uint64_t c0;         // fused form: the partition's first cell, from the look-back
    uint32_t sqtot;      // the partition's sum of squared sizes
    uint32_t over;       // fused form: a bucket above 15 keys
};

// Polls of a predecessor's look-back word (about 0.1 ms) before its sum is taken from its records
// instead (of the calling thread's builds).
static thread_local uint32_t tl_patience = 128;
void part_patience(uint32_t polls) { tl_patience = polls; }

// The fused final pass (single map, level-two search in partition order): each partition
// sizes its buckets itself, publishes its sum of squared sizes, and finds
// its first cell by a look-back over its predecessors' published sums (a decoupled
// look-back scan: the nearest predecessor that already published its inclusive prefix
// ends it).  state holds one word per partition: value << 2 | 1 (the partition's own sum)
// or value << 2 | 2 (the inclusive prefix); zero means not yet published.
//
// A partition is its workgroup's number.  Workgroups are dispatched in the order of their numbers, so
// with one such grid on the device the sums before a running workgroup's are there or on their way.
// Two grids on two streams can keep each other's earlier workgroups off the CUs, each waiting for a
// sum that cannot come; so a look-back that has polled a word long enough takes the sum from that
// partition's records (which are all in place), and ends whether or not its workgroup ever runs.
// Partitions from a ticket counter need no such order either, but are atomics on one word, at
// 11.4 ns each: final pass of 10^7 keys 166 us with tickets, 141 without; 2^26 keys 939 and 874.
struct FuseArgs {
    uint64_t* state;      // Q words, zero before the launch
    uint64_t* S_out;      // the table's S, written by the last partition
    uint32_t* oversize;   // set when some bucket holds more than 15 keys
    uint32_t Q;
    uint32_t patience;    // polls of a word before its sum is taken from the records (0: always so)
    const uint64_t* qend; // partition q's records are [offQ[q], min(qend[q], offQ[q] + qcap))
    uint64_t qcap;        // 0: no cap
    const uint32_t* parts;   // a batch: segment * kSegParts + partition within the map
    // the outcome, for the host (null: another launch brings it): outcome_words words from
    // outcome_dev, once `done` has counted all workgroups
    uint32_t* outcome;
    const uint32_t* outcome_dev;
    uint32_t outcome_words;
    uint32_t* done;
};

// largest of a small value (below 16) over the wave's active lanes
__device__ __forceinline__ uint32_t wave_max16(uint32_t v) {
    uint32_t m = 0;
#pragma unroll
    for (int b = 3; b >= 0; --b) {
        const uint32_t c = m | (1u << b);
        if (__any(v >= c)) m = c;
    }
    return m;
}

// smallest trial from t0 on for a bucket of 2..8 keys held in registers: one 64-bit
// occupancy mask, remainders by multiplication.  smax: the largest bucket among the
// wave's active lanes; key slots beyond it are skipped by the whole wave
// (tri(t): triple t)
template <typename TriAt>
__device__ __forceinline__ uint32_t min_trial_small(TriAt tri, uint32_t T, uint32_t s, const uint64_t (&kx)[8],
                                                    uint64_t M, uint32_t t0 = 0, uint32_t smax = 8) {
    const uint32_t s2 = s * s;
    for (uint32_t t = t0; t < T; ++t) {
        const Triple c = tri(t);
        uint64_t m = 0;
        bool collide = false;
#pragma unroll
        for (uint32_t i = 0; i < 8; ++i) {
            if (i >= smax) break;
            if (i < s && !collide) {
                const uint64_t bit = 1ull << fastmod(mshash(c, kx[i]), M, s2);
                collide = (m & bit) != 0;
                m |= bit;
            }
        }
        if (!collide) return t;
    }
    return T;
}

// waves per SIMD the final pass is compiled for (registers within 80, or 96 with an aux
// word): the LDS of six workgroups (25.4 KB each), or five with an aux word (30.3 KB),
// fits a CU
template <bool AUX>
constexpr unsigned kFinalWaves = AUX ? 5u : 6u;

// AUX: an aux word travels with every key (a string key's index, or the high
// half of a 64-bit value); STR: keys are string fingerprints, so equal keys
// are told apart by their bytes
// MULTI: workgroup q's partition is entry q of a list over the wide maps of a batch (segs); the
// map's hash, triples (Cg + map*T), header and cells (pool offsets) come from its descriptor, the
// partition's records lie in region q, the look-back ends at the map's first partition, and
// ctrl_flags points to four outcome words per map
// FUSED: the final pass sizes its own partition and finds its first cell by the look-back above
// (no separate size pass and scan; grid = Q)
// BT: threads of the workgroup
template <bool AUX, bool STR, bool MULTI = false, bool FUSED = false, uint32_t BT = kPB>
__global__ __launch_bounds__(BT) __attribute__((amdgpu_waves_per_eu(BT == kPB ? kFinalWaves<AUX> : BT / 256))) void k_pfinal(const uint64_t* __restrict__ keys, const uint32_t* __restrict__ vals,
                                                  const uint32_t* __restrict__ aux, int aux_is_pos, uint64_t n,
                                                  Triple A, uint64_t magic, const uint64_t* __restrict__ offQ,
                                                  const uint64_t* __restrict__ cbase, const uint32_t* __restrict__ sizes,
                                                  uint64_t G, const Triple* __restrict__ Cg, uint32_t T,
                                                  Group* __restrict__ header, Cell* __restrict__ slots,
                                                  uint32_t* __restrict__ ctrl_flags, const int64_t* __restrict__ ctx_off,
                                                  const uint8_t* __restrict__ ctx_bytes,
                                                  const uint8_t* __restrict__ given_t,
                                                  const WideSeg* __restrict__ segs = nullptr,
                                                  const uint32_t* __restrict__ reject = nullptr,
                                                  uint64_t cap = ~0ull, FuseArgs fa = FuseArgs{}) {
    static_assert(!MULTI || FUSED, "the maps of a batch are sized by the final pass");
    __shared__ FinalLds<AUX> L;
    const uint32_t tid = threadIdx.x;
    // few partitions: the last workgroup to end writes the attempt's outcome to the host (a launch
    // less; with many, one more atomic on one word for each would cost more)
    constexpr bool REPORT = FUSED && !MULTI && BT != kPB;
    auto ended = [&]() {
        if (!REPORT || !fa.outcome) return;
        __syncthreads();
        if (tid == 0) {
            asm volatile("s_waitcnt vmcnt(0)" ::: "memory");   // this thread's outcome words are written
            if (atomicAdd(fa.done, 1u) == gridDim.x - 1)
                for (uint32_t k = 0; k < fa.outcome_words; ++k)
                    fa.outcome[k] =
                        __hip_atomic_load(fa.outcome_dev + k, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        }
    };
    // an attempt already rejected by the size pass (a bucket above 15 keys) or by bad
    // string offsets is skipped (both flags are set before this kernel starts; the fused form sets
    // the first itself, and every workgroup that others may look back to goes on)
    if (reject && ((FUSED ? 0u : reject[0]) | reject[1])) {   // the whole block
        ended();
        return;
    }
    const uint32_t q = blockIdx.x;
    uint32_t qh = q;       // the partition's place among its map's partitions
    uint32_t q0 = 0;       // the map's first partition
    uint32_t seg = 0;
    if (MULTI) {
        const uint32_t entry = fa.parts[q];
        seg = entry / kSegParts;
        qh = entry % kSegParts;
        const WideSeg& sg = segs[seg];
        q0 = sg.part0;
        A = sg.A;
        magic = sg.magic;
        n = sg.n;
        G = sg.G;
        Cg += (uint64_t)sg.map * T;
        header += sg.hdr_off;
        slots += sg.slot_off;
        cap = (uint64_t)sg.c * sg.n;
        fa.oversize = ctrl_flags + 4 * seg;
        ctrl_flags += 4 * seg + 1;
    }
    auto begin_of = [&](uint32_t p) { return MULTI ? p * fa.qcap : offQ[p]; };
    auto end_of = [&](uint32_t p, uint64_t from) {
        return !FUSED ? offQ[p + 1] : fa.qcap ? min(fa.qend[p], from + fa.qcap) : fa.qend[p];
    };
    const uint64_t k0 = begin_of(q), k1 = end_of(q, k0);
    const uint32_t nq = (uint32_t)(k1 - k0);
    const bool keys_fit = nq <= kFinalKeyCap;
    // a partition whose cells would end beyond the cells allocated is skipped (the attempt
    // then runs this pass again into an exact allocation); the fused form learns its cells
    // below
    uint64_t c0 = 0;
    uint32_t Sq = 0;
    if (!FUSED) {
        c0 = cbase[q];
        Sq = (uint32_t)(cbase[q + 1] - c0);
        if (c0 + Sq > cap) return;   // the whole block
    }
    bool fast = FUSED ? keys_fit : keys_fit && Sq <= kFinalCellCap;
    // the partition's records go in flight first; the set-up below overlaps their latency
    constexpr uint32_t KPT = (kFinalKeyCap + BT - 1) / BT;   // record slots per thread
    uint64_t xk[KPT];
    uint32_t vk[KPT], ak[KPT];
    if (fast) {
#pragma unroll
        for (uint32_t k = 0; k < KPT; ++k) {
            const uint32_t i = tid + k * BT;
            if (i < nq) {
                // streaming loads: each record is read once here (and each cell and group
                // record below written once), so none of them displaces the caches' other data
                xk[k] = __builtin_nontemporal_load(keys + k0 + i);
                vk[k] = __builtin_nontemporal_load(vals + k0 + i);
                if (AUX) ak[k] = aux_is_pos ? (uint32_t)(k0 + i) : aux[k0 + i];
            }
        }
    }
    // the first kLdsTrials level-two triples are staged in LDS; larger trials read theirs
    // from global memory
    const Triple* const LC = Cg;
    for (uint32_t t = tid; t < kLdsTrials && t < T; t += BT) L.tri[t] = Cg[t];
    auto tri = [&](uint32_t t) { return t < kLdsTrials ? L.tri[t] : Cg[t]; };
    // the size words of the separate size pass (the fused form takes the counts of the ranking)
    uint32_t word = 0;
    if (!FUSED && tid < kGroupsPerPart && (uint64_t)qh * kGroupsPerPart + tid < G)
        word = sizes[(uint64_t)q * kGroupsPerPart + tid];
    static_assert(BT >= kGroupsPerPart, "a thread per group");
    if (tid < 3) L.flags[tid] = 0;
    if (FUSED && tid == 0) L.over = 0;
    if (FUSED || fast) {
        if (tid < kGroupsPerPart) L.cnt2[tid] = 0;
        if (tid < kPartBuckets / 4) reinterpret_cast<uint32_t*>(L.tb)[tid] = 0;
        static_assert(BT >= kPartBuckets / 4, "a thread per word of trial bytes");
        for (uint32_t w = tid; w < kFinalCellCap / 32; w += BT) L.occ[w] = 0;
        if (tid < kPartBuckets / 32) L.fl[tid] = 0;
        if (tid < 16) L.mag[tid] = kSquareMagics.m[tid];
        if (tid == 0) L.nhard = 0;
    }
    __syncthreads();
    uint32_t lbk[KPT], rk[KPT], c0k[KPT];   // c0k: bucket size, first cell and trial-0 cell
    static_assert(kFinalCellCap <= 4096, "12 bits for a cell of the partition");
    // rank the partition's records (when they fit) in their buckets: ranks come from an LDS
    // histogram of the 4-bit bucket sizes, which the fused form also takes as the
    // partition's sizes.  The records stay in registers until they are grouped.
    auto stage = [&]() {
        bool over = false;
#pragma unroll
        for (uint32_t k = 0; k < KPT; ++k) {
            const uint32_t i = tid + k * BT;
            if (i < nq) {
                const uint32_t lb = bucket_of(A, magic, (uint32_t)n, xk[k]) & (kPartBuckets - 1);
                lbk[k] = lb;
                const uint32_t sh = 4 * (lb & 7u);
                rk[k] = (atomicAdd(&L.cnt2[lb >> 3], 1u << sh) >> sh) & 15u;
                over |= rk[k] == 15u;   // this key is the bucket's sixteenth
            }
        }
        return over;
    };
    if (FUSED) {
        bool over = false;
        if (keys_fit) {
            over = stage();
        } else {
            // too many keys to stage: their sizes from one pass over them
            for (uint32_t i = tid; i < nq; i += BT) {
                const uint32_t lb = bucket_of(A, magic, (uint32_t)n, keys[k0 + i]) & (kPartBuckets - 1);
                const uint32_t sh = 4 * (lb & 7u);
                over |= ((atomicAdd(&L.cnt2[lb >> 3], 1u << sh) >> sh) & 15u) == 15u;
            }
        }
        if (over) atomicOr(&L.over, 1u);
        __syncthreads();
        if (tid < kGroupsPerPart) word = L.cnt2[tid];
    }
    // where each group's keys and cells start inside the partition
    {
        const uint32_t own = word_pos(word), inc = wave_scan(own);
        static_assert(kGroupsPerPart == 128, "two waves hold the groups");
        if (tid == 63) L.wsum = inc;
        __syncthreads();
        const uint32_t all = inc + (tid >= 64 ? L.wsum : 0u);
        if (tid < kGroupsPerPart) L.gpos[tid] = (uint64_t)(all - own) << 32 | word;
        if (tid == kGroupsPerPart - 1) L.sqtot = pos_cells(all);
    }
    // fused form: the partition's first cell, from the predecessors' published sums back to
    // the nearest published inclusive prefix (64 per round: lane l reads partition
    // end - 1 - l); then this partition's inclusive prefix is published.  Called by the
    // whole workgroup as late as can be, when its cells are known and only their addresses are
    // not: the predecessors' sums, which each publishes as soon as it has sized its buckets, are there
    // to read, and the nearer an inclusive prefix is, the fewer rounds.  Final pass of 10^7 keys 139 us; before the cells'
    // indices are read 158, and 196 by a wave of its own while the others group the records.
    // partition p's sum of squared sizes, as its own workgroup publishes it, counted by the first wave
    // alone (the others wait for the look-back); cnt2 has been read by then
    auto squares_of = [&](uint32_t p) {
        for (uint32_t g = tid; g < kGroupsPerPart; g += 64) L.cnt2[g] = 0;
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        __builtin_amdgcn_wave_barrier();
        const uint64_t from = begin_of(p), to = end_of(p, from);
        for (uint64_t i = from + tid; i < to; i += 64) {
            const uint32_t lb = bucket_of(A, magic, (uint32_t)n, keys[i]) & (kPartBuckets - 1);
            atomicAdd(&L.cnt2[lb >> 3], 1u << (4 * (lb & 7u)));
        }
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        __builtin_amdgcn_wave_barrier();
        uint32_t sq = 0;
        for (uint32_t g = tid; g < kGroupsPerPart; g += 64) sq += pos_cells(word_pos(L.cnt2[g]));
        for (int d = 32; d >= 1; d >>= 1) sq += __shfl_xor(sq, d, 64);
        __builtin_amdgcn_wave_barrier();
        return sq;
    };
    auto lookback = [&]() {
        if (tid < 64) {
            const uint32_t lane = tid;
            uint64_t excl = 0;
            int64_t end = (int64_t)q;
            for (;;) {
                const int64_t idx = end - 1 - (int64_t)lane;
                uint64_t v = 2;   // before the map's first partition: an inclusive prefix of 0
                if (idx >= (int64_t)q0) {
                    v = 0;
                    for (uint32_t polls = 0; polls < fa.patience; ++polls) {
                        v = __hip_atomic_load(&fa.state[idx], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                        if (v & 3u) break;
                        __builtin_amdgcn_s_sleep(1);
                    }
                }
                const uint64_t incl = __ballot((v & 3u) == 2u);
                // sums that did not come, nearer than the nearest inclusive prefix
                for (uint64_t miss = __ballot((v & 3u) == 0u) & ((incl & (0 - incl)) - 1); miss; miss &= miss - 1) {
                    const uint32_t l = (uint32_t)__ffsll((long long)miss) - 1;
                    const uint32_t sq = squares_of((uint32_t)(end - 1 - l));
                    if (lane == l) {
                        v = (uint64_t)sq << 2 | 1u;
                        // for the other look-backs, unless the partition itself has published by now
                        atomicCAS(reinterpret_cast<unsigned long long*>(&fa.state[idx]), 0ull, (unsigned long long)v);
                    }
                }
                uint64_t take = v >> 2;
                const bool last = incl != 0;
                if (last && lane > (uint32_t)(__ffsll((long long)incl) - 1)) take = 0;
                for (int d = 32; d >= 1; d >>= 1) take += __shfl_xor(take, d, 64);
                excl += take;
                if (last) break;
                end -= 64;
            }
            if (lane == 0) {
                L.c0 = excl;
                __hip_atomic_store(&fa.state[q], ((excl + Sq) << 2) | 2u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                if (MULTI) {
                    if ((uint64_t)(qh + 1) * kPartBuckets >= n) {   // the map's last partition
                        fa.S_out[seg] = excl + Sq;
                        if (excl + Sq > cap) atomicOr(fa.oversize, 2u);
                    }
                } else if (q + 1 == fa.Q) {
                    __hip_atomic_store(fa.S_out, excl + Sq, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                }
            }
        }
        __syncthreads();
        c0 = L.c0;
    };
    if (FUSED) {
        __syncthreads();
        Sq = L.sqtot;
        // publish this partition's sum at once: the look-backs of later partitions read it
        if (tid == 0)
            __hip_atomic_store(&fa.state[q], ((uint64_t)Sq << 2) | 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        if (L.over) {
            lookback();
            if (tid == 0) atomicOr(fa.oversize, 1u);
            ended();
            return;   // the whole block: the attempt is rejected
        }
        fast = keys_fit && Sq <= kFinalCellCap;
        if (MULTI && !fast) {
            // keys too uneven for the LDS staging (consecutive integers, say): the map goes to the kernel
            // that builds a map by one workgroup, which they do not slow down.  1000 maps of 4096 consecutive
            // keys 2513 us by the gathering below and 144 so, 500 of 65536 5126 and 1560.
            if (tid == 0) atomicOr(fa.oversize, 1u);
            return;   // the whole block; its sum is published
        }
    }
    if (fast) {
        if (!FUSED) (void)stage();
        __syncthreads();
        // group by bucket: each record goes to the LDS slot of its rank in its bucket, so a
        // bucket's keys lie together (from here on a record is named by its slot).  A lone
        // key owns its bucket's single cell.  Every key of a larger bucket tries trial 0 at
        // once: the second key to claim a cell marks its bucket as colliding, and only those
        // buckets are searched below.
        const Triple c0t = L.tri[0];
#pragma unroll
        for (uint32_t k = 0; k < KPT; ++k) {
            const uint32_t i = tid + k * BT;
            if (i < nq) {
                const uint32_t lb = lbk[k], kk = lb & 7u;
                const uint64_t gp = L.gpos[lb >> 3];
                const uint32_t s = nib((uint32_t)gp, kk), pos = bucket_pos(gp, kk);
                const uint32_t off = pos_cells(pos), slot = pos_keys(pos) + rk[k];
                if (s >= 2) {
                    // the key of rank r marks cells [r*s, r*s + s) of its bucket with the
                    // bucket's first cell; placement below overwrites the cells keys take, and
                    // the write-out resolves a cell still marked to the bucket's lowest
                    // occupied cell (the fill rule)
                    const uint32_t from = off + rk[k] * s;
                    for (uint32_t u = 0; u < s; ++u) L.smap[from + u] = (uint16_t)(0x8000u | off);
                }
                rk[k] = slot;
                L.key[slot] = xk[k];
                L.val[slot] = vk[k];
                if (AUX) L.aux[slot] = ak[k];
                c0k[k] = s << 24 | off << 12 | off;
                const uint32_t h0 = mshash(c0t, xk[k]);   // trial 0
                if (s == 1) {
                    L.smap[off] = (uint16_t)slot;
                    L.tb[lb] = (uint8_t)tag_of(h0);   // trial 0; the byte holds the key's tag
                } else {
                    if (!given_t) {
                        const uint32_t cell = off + fastmod(h0, L.mag[s], s * s);
                        c0k[k] = s << 24 | off << 12 | cell;
                        const uint32_t bit = 1u << (cell & 31u), bb = 1u << (lb & 31u);
                        if ((atomicOr(&L.occ[cell >> 5], bit) & bit) && !(atomicOr(&L.fl[lb >> 5], bb) & bb))
                            L.hard[atomicAdd(&L.nhard, 1u)] = (uint16_t)lb;
                    }
                }
            }
        }
        __syncthreads();
        // Trials: a bucket that trial 0 places keeps t = 0 (tb is zero); given trials (the
        // rounds schedule) are taken as they are
        if (given_t) {
            for (uint32_t b = tid; b < kPartBuckets; b += BT) {
                if (nib((uint32_t)L.gpos[b >> 3], b & 7u) < 2) continue;
                const uint32_t t = given_t[(uint64_t)q * kPartBuckets + b];
                L.tb[b] = (uint8_t)t;
                if (t) atomicMax(&L.flags[2], t);
            }
        }
        // the colliding buckets, one lane each, trials from 1 on with the keys in registers;
        // bucket j goes to lane j / 4 of wave j % 4, so that all four SIMDs search (a packed
        // list of ~80 buckets would otherwise occupy one and a half waves)
        const uint32_t nh = given_t ? 0u : L.nhard;
        for (uint32_t j = (tid & 63u) * (BT / 64) + (tid >> 6); j < nh; j += BT) {
            const uint32_t b = L.hard[j];
            const uint64_t gp = L.gpos[b >> 3];
            const uint32_t sb = nib((uint32_t)gp, b & 7u);
            const uint32_t kst = pos_keys(bucket_pos(gp, b & 7u));
            uint32_t t;
            if (sb <= 8) {
                const uint32_t smax = wave_max16(sb);
                uint64_t kx[8];
#pragma unroll
                for (uint32_t i = 0; i < 8; ++i) kx[i] = i < sb ? L.key[kst + i] : 0;
                t = min_trial_small(tri, T, sb, kx, L.mag[sb], 1, smax);
            } else {
                t = min_trial(LC, T, sb, [&](uint32_t i) { return L.key[kst + i]; }, 1);
            }
            if (t < T) {
                L.tb[b] = (uint8_t)t;
                atomicMax(&L.flags[2], t);
            } else {
                // no trial separates the bucket: the attempt fails, or the build when
                // two keys are equal; the cells get any in-range content
                bool dup = false;
                for (uint32_t a2 = 0; a2 < sb; ++a2)
                    for (uint32_t b2 = a2 + 1; b2 < sb; ++b2) {
                        const uint32_t ia = kst + a2, ib = kst + b2;
                        if (STR) dup |= same_string(ctx_off, ctx_bytes, L.aux[ia], L.aux[ib]);
                        else dup |= L.key[ia] == L.key[ib];
                    }
                atomicOr(&L.flags[0], 1u);
                if (dup) atomicOr(&L.flags[1], 1u);
            }
        }
        __syncthreads();
        // every key of a larger bucket writes its own cell
#pragma unroll
        for (uint32_t k = 0; k < KPT; ++k) {
            const uint32_t i = tid + k * BT;
            if (i < nq) {
                const uint32_t sb = c0k[k] >> 24;
                if (sb >= 2) {
                    const uint32_t t = L.tb[lbk[k]];
                    uint32_t cell = c0k[k] & 0xFFFu;
                    if (t || given_t)
                        cell = (c0k[k] >> 12 & 0xFFFu) + fastmod(mshash(tri(t), L.key[rk[k]]), L.mag[sb], sb * sb);
                    L.smap[cell] = (uint16_t)rk[k];
                }
            }
        }
        __syncthreads();
        // write-out: indices first (a marked cell resolves to the bucket's lowest
        // occupied cell; every bucket holds a key), then the records
        constexpr uint32_t CPT = kFinalCellCap / BT;
        static_assert(kFinalCellCap % BT == 0, "whole cells per thread");
        uint32_t idx[CPT];
#pragma unroll
        for (uint32_t k = 0; k < CPT; ++k) {
            const uint32_t p = tid + k * BT;
            idx[k] = p < Sq ? L.smap[p] : 0u;
        }
#pragma unroll
        for (uint32_t k = 0; k < CPT; ++k) {
            if (idx[k] & 0x8000u) {
                uint32_t i;
                for (uint32_t p2 = idx[k] & 0x7FFFu; (i = L.smap[p2]) & 0x8000u; ++p2) {}
                idx[k] = i;
            }
        }
        if (FUSED) {
            lookback();
            if (c0 + Sq > cap) {   // the whole block
                ended();
                return;
            }
        }
#pragma unroll
        for (uint32_t k = 0; k < CPT; ++k) {
            const uint32_t p = tid + k * BT;
            if (p < Sq) {
                const uint32_t i = idx[k];
                Cell c;
                c.key = L.key[i];
                c.val = L.val[i];
                c.aux = AUX ? L.aux[i] : 0u;
                store_cell_once(slots + c0 + p, c);
            }
        }
    } else {
        // rare: the partition does not fit the LDS staging; every bucket gathers its
        // own keys from HBM (a scan of the partition), searches and writes its cells
        __syncthreads();
        if (FUSED) {
            lookback();
            if (c0 + Sq > cap) {   // the whole block
                ended();
                return;
            }
        }
        for (uint32_t b = tid; b < kPartBuckets; b += BT) {
            const uint64_t gp = L.gpos[b >> 3];
            const uint32_t s = nib((uint32_t)gp, b & 7u);
            const uint32_t off = pos_cells(bucket_pos(gp, b & 7u));
            uint64_t mine[kSMax];
            uint32_t pos[kSMax];
            uint32_t got = 0;
            if (s) {
                for (uint32_t i = 0; i < nq && got < s; ++i) {
                    const uint64_t x = keys[k0 + i];
                    if ((bucket_of(A, magic, (uint32_t)n, x) & (kPartBuckets - 1)) == b) {
                        mine[got] = x;
                        pos[got] = i;
                        ++got;
                    }
                }
            }
            uint32_t t = 0;
            bool exhausted = false;
            if (s >= 2) {
                t = given_t ? given_t[(uint64_t)q * kPartBuckets + b]
                            : min_trial(LC, T, s, [&](uint32_t i) { return mine[i]; });
                exhausted = t == T;
            }
            const uint32_t s2 = s * s;
            if (s >= 1 && !exhausted) {
                const Triple c = LC[t];
                uint32_t first_p = s2, first_i = 0;
                for (uint32_t i = 0; i < s; ++i) {
                    const uint32_t h = mshash(c, mine[i]) % s2;
                    if (h < first_p) {
                        first_p = h;
                        first_i = i;
                    }
                }
                for (uint32_t p = 0; p < s2; ++p) {
                    uint32_t who = first_i;
                    for (uint32_t i = 0; i < s; ++i)
                        if (mshash(c, mine[i]) % s2 == p) who = i;
                    Cell cl;
                    cl.key = mine[who];
                    cl.val = vals[k0 + pos[who]];
                    cl.aux = AUX ? (aux_is_pos ? (uint32_t)(k0 + pos[who]) : aux[k0 + pos[who]]) : 0u;
                    slots[c0 + off + p] = cl;
                }
            }
            if (exhausted) {
                bool dup = false;
                for (uint32_t a = 0; a < s; ++a)
                    for (uint32_t b2 = a + 1; b2 < s; ++b2) {
                        if (STR) {
                            const uint32_t xa = aux_is_pos ? (uint32_t)(k0 + pos[a]) : aux[k0 + pos[a]];
                            const uint32_t xb = aux_is_pos ? (uint32_t)(k0 + pos[b2]) : aux[k0 + pos[b2]];
                            dup |= same_string(ctx_off, ctx_bytes, xa, xb);
                        } else {
                            dup |= mine[a] == mine[b2];
                        }
                    }
                atomicOr(&L.flags[0], 1u);
                if (dup) atomicOr(&L.flags[1], 1u);
                t = 0;
            }
            if (t) atomicMax(&L.flags[2], t);
            L.tb[b] = (uint8_t)(s == 1 ? key_tag(LC[0], mine[0]) : t);
        }
        __syncthreads();
    }
    for (uint32_t g = tid; g < kGroupsPerPart; g += BT) {
        const uint64_t gg = (uint64_t)qh * kGroupsPerPart + g;
        if (gg < G) {
            Group h;
            h.base = (uint32_t)(c0 + pos_cells((uint32_t)(L.gpos[g] >> 32)));
            h.sizes = (uint32_t)L.gpos[g];
            h.t_lo = (uint32_t)L.tb[8 * g] | ((uint32_t)L.tb[8 * g + 1] << 8) | ((uint32_t)L.tb[8 * g + 2] << 16) |
                     ((uint32_t)L.tb[8 * g + 3] << 24);
            h.t_hi = (uint32_t)L.tb[8 * g + 4] | ((uint32_t)L.tb[8 * g + 5] << 8) |
                     ((uint32_t)L.tb[8 * g + 6] << 16) | ((uint32_t)L.tb[8 * g + 7] << 24);
            const u32x4 hw = {h.base, h.sizes, h.t_lo, h.t_hi};
            __builtin_nontemporal_store(hw, reinterpret_cast<u32x4*>(header) + gg);
        }
    }
    if (tid == 0) {
        if (L.flags[0]) atomicOr(&ctrl_flags[0], 1u);
        if (L.flags[1]) atomicOr(&ctrl_flags[1], 1u);
        if (L.flags[2]) atomicMax(&ctrl_flags[2], L.flags[2]);
    }
    ended();
}

// ---- host planning and launches ------------------------------------------------------

// Regions of the cursor form: a first-level bin covers 2^shiftA partitions of 1024
// buckets and a partition 1024 buckets; with n keys in n buckets the keys of B buckets
// number B on average with a standard deviation of about sqrt(B), and the regions hold
// 12 deviations more (an overflow only sends the attempt back to the counted passes).
static uint64_t part_region(uint64_t B) {
    const uint64_t sd = (uint64_t)std::ceil(std::sqrt((double)B));
    return (B + 12 * sd + 64 + 255) & ~(uint64_t)255;
}

PartPlan part_plan(uint64_t n, bool carry) {
    PartPlan P{};
    P.Q = (uint32_t)((n + kPartBuckets - 1) / kPartBuckets);
    uint32_t bits = 0;
    while ((1ull << bits) < P.Q) ++bits;
    P.bits_q = bits;
    auto clampu = [](uint64_t v, uint64_t lo, uint64_t hi) { return (uint32_t)(v < lo ? lo : v > hi ? hi : v); };
    // Tiles of the cursor form and keys per worker, so that a small input is not left to a few
    // CUs.  Build, one lookup and release with tiles of 12288 keys, two per worker, and here: 2^16 keys
    // (three workers) 69 and 56 us with tiles of 2048 (57 of 4096), 2^18 75 and 62, 2^20 107
    // and 98 with tiles of 4096 (104 of 2048); 3 * 10^6 156, 157 and 172 with tiles of 12288, 4096
    // and 2048.
    uint64_t worker = 2ull * kPScatterThreads * kPScatterItems;
    if (n <= 256ull * kPartBuckets) {
        P.items = 2;
        worker = (uint64_t)kPScatterThreads * P.items;
    } else if (n < (1ull << 21)) {
        P.items = 4;
        worker = (uint64_t)kPScatterThreads * P.items;
    }
    P.W1 = clampu((n + worker - 1) / worker, 1, 4096);
    // the large tiles leave a CU to one worker: as many workers as fill all 256 CUs the same number of
    // times.  First pass of 2^23 records with an aux word 76 us with 342 workers and 63 with 512, of
    // 2^22 39 with 171 and 32 with 256, of 10^7 without 65 with 407 and 62 with 512.
    if (P.items == 0) P.W1 = (P.W1 + 255) & ~255u;
    if (P.Q <= 1) {
        P.passes = 0;
    } else if (bits <= 8) {
        P.passes = 1;
        P.binsA = P.Q;
        P.capQ = part_region(kPartBuckets);
    } else if (bits <= 16) {
        P.passes = 2;
        P.shiftA = bits - 8;
        P.binsA = (uint32_t)((P.Q + (1u << P.shiftA) - 1) >> P.shiftA);
        P.bitsB = P.shiftA;
        P.W2 = clampu((n / P.binsA + worker - 1) / worker, 1, 64);
        P.cap1 = part_region((uint64_t)kPartBuckets << P.shiftA);
        P.capQ = part_region(kPartBuckets);
        P.regions1 = P.binsA;
        P.W2c = P.W2;
        if (n >= (carry ? kSubRegionKeysAux : kSubRegionKeys)) {
            // an eighth of a bin for every XCD: at most this many of the first pass's records, two tiles
            // at a time
            const uint64_t chunk = (n + P.W1 - 1) / P.W1, most = (P.W1 + 7) / 8 * chunk;
            P.subs = 3;
            P.cap1 = part_region((((uint64_t)kPartBuckets << P.shiftA) * most + n - 1) / n);
            P.regions1 = P.binsA << P.subs;
            P.W2c = clampu((most / P.binsA + worker / 2 - 1) / (worker / 2), 1, 64);
        }
    } else {
        P.passes = 3;
        P.shiftA = bits - 8;
        P.binsA = (uint32_t)((P.Q + (1u << P.shiftA) - 1) >> P.shiftA);
        P.bitsC = bits - 16;
        P.bitsB = 8;
        P.binsAB = (uint32_t)((P.Q + (1u << P.bitsC) - 1) >> P.bitsC);
        P.W2 = clampu((n / P.binsA + worker - 1) / worker, 1, 64);
        P.W3 = clampu((n / P.binsAB + worker - 1) / worker, 1, 64);
    }
    uint64_t m1 = (uint64_t)kBins * P.W1;
    uint64_t m2 = P.passes >= 2 ? (uint64_t)P.binsA * kBins * P.W2 : 0;
    uint64_t m3 = P.passes == 3 ? (uint64_t)P.binsAB * kBins * P.W3 : 0;
    P.matrix = std::max(m1, std::max(m2, m3));
    return P;
}

size_t part_scratch(const PartPlan& plan, uint64_t n, bool carry, bool cursor, bool sizes, char* base, PartArgs* a) {
    size_t total = 0;
    auto carve = [&](auto PartArgs::*field, size_t bytes) {
        if (base) a->*field = reinterpret_cast<std::remove_reference_t<decltype(a->*field)>>(base + total);
        total += (bytes + 255) & ~(size_t)255;
    };
    const uint64_t Q = plan.Q;
    // the cursor form keeps its records in fixed-capacity regions (binsA of them after a first
    // of two passes, Q after the last)
    const uint64_t r1 = cursor ? std::max<uint64_t>(n, plan.cap1 * plan.regions1) : n;
    const uint64_t r2 = cursor ? std::max<uint64_t>(n, plan.capQ * Q) : n;
    if (plan.passes >= 2) {
        carve(&PartArgs::k1, 8 * r1);
        carve(&PartArgs::v1, 4 * r1);
        if (carry) carve(&PartArgs::a1, 4 * r1);
    }
    if (plan.passes >= 1) {
        carve(&PartArgs::k2, 8 * r2);
        carve(&PartArgs::v2, 4 * r2);
        if (carry) carve(&PartArgs::a2, 4 * r2);
    }
    if (cursor) {
        carve(&PartArgs::cur1, 8 * (size_t)plan.regions1);
        carve(&PartArgs::cur2, 8 * Q);
        carve(&PartArgs::begA, 8 * (size_t)plan.regions1);
        carve(&PartArgs::begQ, 8 * Q);
    }
    carve(&PartArgs::cnt, 4 * plan.matrix);
    carve(&PartArgs::off, 4 * plan.matrix);
    carve(&PartArgs::tsum, 4 * part_scan_tiles(plan));
    carve(&PartArgs::tpre, 8 * (part_scan_tiles(plan) + 1));
    carve(&PartArgs::offA, 8 * 257);
    carve(&PartArgs::offQ, 8 * (Q + 1));
    carve(&PartArgs::sqQ, 4 * Q);
    if (plan.passes == 3) carve(&PartArgs::offAB, 8 * ((size_t)plan.binsAB + 1));
    carve(&PartArgs::cbase, 8 * (Q + 1));
    if (sizes) carve(&PartArgs::sizes, 4 * Q * kGroupsPerPart);
    return total;
}

uint64_t exscan_tiles(uint64_t N) { return (N + kXTile - 1) / kXTile; }
uint64_t part_scan_tiles(const PartPlan& P) { return exscan_tiles(std::max<uint64_t>(P.matrix, P.Q)); }

void exscan_u32(const uint32_t* in, uint64_t N, uint32_t* tsum, uint64_t* tpre, uint32_t* out, hipStream_t st) {
    const uint32_t nt = (uint32_t)exscan_tiles(N);
    hipLaunchKernelGGL(k_xscan_reduce, nt, kPB, 0, st, in, N, tsum);
    hipLaunchKernelGGL(k_scan_counts, 1, 1024, 0, st, tsum, nt, tpre, nullptr, nullptr);
    hipLaunchKernelGGL(k_xscan_down, nt, kPB, 0, st, in, N, tpre, out);
}

static void scan_matrix(const PartArgs& a, uint64_t N, hipStream_t st) { exscan_u32(a.cnt, N, a.tsum, a.tpre, a.off, st); }

template <bool AUX>
static void scatter(const PartArgs& a, const uint64_t* kin, const uint32_t* vin, const uint32_t* ain,
                    const uint64_t* ranges, dim3 grid, uint32_t W, uint32_t shift, uint32_t mask, uint64_t* kout,
                    uint32_t* vout, uint32_t* aout, hipStream_t st) {
    FKS_TIMED("fks_part_scatter", st,
              hipLaunchKernelGGL((k_dscatter<AUX, AUX ? kPScatterItemsAux : kPScatterItems, kPScatterThreads>), grid,
                                 kPScatterThreads, 0, st, kin, vin, ain, a.n, a.A, a.magic, ranges, W,
                                 shift, mask, a.off, kout, vout, aout));
}

template <bool AUX>
static void scatter_cursor(const PartArgs& a, const PartPlan& P, const uint64_t* kin, const uint32_t* vin,
                           const uint32_t* ain, const uint64_t* ranges, const uint64_t* ranges_hi, uint64_t in_cap,
                           dim3 grid, uint32_t W, uint32_t shift, uint32_t mask, uint64_t* kout, uint32_t* vout,
                           uint32_t* aout, unsigned long long* cursor, uint64_t cap, uint32_t subs, uint32_t in_subs,
                           hipStream_t st) {
    auto launch = [&](auto kernel) {
        FKS_TIMED("fks_part_scatter", st,
                  hipLaunchKernelGGL(kernel, grid, kPScatterThreads, 0, st, kin, vin, ain, a.n, a.A, a.magic, ranges, W,
                                     shift, mask, nullptr, kout, vout, aout, nullptr, nullptr, cursor, ranges_hi,
                                     cap, a.overflow, in_cap, subs, in_subs,
                                     kin == a.keys ? a.pairs : nullptr));
    };
    if (P.items == 2) launch(k_dscatter<AUX, 2, kPScatterThreads, true>);
    else if (P.items == 4) launch(k_dscatter<AUX, 4, kPScatterThreads, true>);
    else launch(k_dscatter<AUX, AUX ? kPScatterItemsAux : kPScatterItems, kPScatterThreads, true>);
}

static unsigned grid_for_count(uint64_t count) { return (unsigned)std::min<uint64_t>((count + 255) / 256, 4096); }

// Runs the partition passes of one attempt; stream-ordered outputs: offQ, the
// records in partition order (o.keys/vals/aux), the size words, the partition
// sums of squares, their scan (cbase) and the total S (*S_dev).
int part_prepare(const PartArgs& a, hipStream_t st, PartOut& o) {
    const PartPlan P = part_plan(a.n, a.aux);
    const uint64_t n = a.n;
    const bool aux = a.aux;
    o.plan = P;
    o.keys = a.keys;
    o.vals = a.vals;
    o.aux = a.aux_in;
    o.aux_is_pos = a.aux_in ? 0 : 1;
    o.qbeg = a.offQ;
    o.qend = a.offQ + 1;
    o.qcap = 0;   // no cap: the counted passes fill their ranges exactly
    o.prezeroed = o.reported = false;
    auto count = [&](const uint64_t* kin, const uint64_t* ranges, dim3 grid, uint32_t W, uint32_t shift,
                     uint32_t mask) {
        FKS_TIMED("fks_part_count", st,
                  hipLaunchKernelGGL(k_dcount, grid, kPB, 0, st, kin, n, a.A, a.magic, ranges, W, shift, mask,
                                     a.cnt));
    };
    auto init = [&](uint64_t bins1, uint64_t parts, bool one) {
        const uint64_t nzw = a.fused ? 2 * (uint64_t)P.Q : 0;
        hipLaunchKernelGGL(k_attempt_init, grid_for_count(std::max<uint64_t>(1, bins1 + parts + nzw)), 256, 0, st, a.start,
                           a.cur1, a.begA, bins1, P.cap1, a.cur2, a.begQ, parts, P.capQ, one ? a.offQ : nullptr, n,
                           reinterpret_cast<uint32_t*>(a.cbase), nzw);
        o.prezeroed = a.fused;
    };
    if (P.passes == 0) {
        init(0, 0, true);
    } else if (P.passes == 1 && a.cursor) {
        // one pass straight into the partitions' regions, each run reserved on its partition's
        // cursor
        init(0, P.Q, false);
        if (aux)
            scatter_cursor<true>(a, P, a.keys, a.vals, a.aux_in, nullptr, nullptr, 0, dim3(P.W1, 1), P.W1, 0, 255, a.k2,
                                 a.v2, a.a2, a.cur2, P.capQ, 0, 0, st);
        else
            scatter_cursor<false>(a, P, a.keys, a.vals, nullptr, nullptr, nullptr, 0, dim3(P.W1, 1), P.W1, 0, 255,
                                  a.k2, a.v2, a.a2, a.cur2, P.capQ, 0, 0, st);
        o.keys = a.k2;
        o.vals = a.v2;
        o.aux = a.a2;
        o.aux_is_pos = aux ? 0 : 1;
        o.qbeg = a.begQ;
        o.qend = reinterpret_cast<const uint64_t*>(a.cur2);
        o.qcap = P.capQ;
    } else if (P.passes == 1) {
        count(a.keys, nullptr, dim3(P.W1, 1), P.W1, 0, 255);
        scan_matrix(a, (uint64_t)kBins * P.W1, st);
        if (aux)
            scatter<true>(a, a.keys, a.vals, a.aux_in, nullptr, dim3(P.W1, 1), P.W1, 0, 255, a.k2, a.v2, a.a2, st);
        else
            scatter<false>(a, a.keys, a.vals, nullptr, nullptr, dim3(P.W1, 1), P.W1, 0, 255, a.k2, a.v2, a.a2, st);
        hipLaunchKernelGGL(k_extract_offsets, (P.Q + 256) / 256, 256, 0, st, a.off, P.W1, 8u, P.Q, n, a.offQ);
        o.keys = a.k2;
        o.vals = a.v2;
        o.aux = a.a2;
        o.aux_is_pos = aux ? 0 : 1;
    } else if (P.passes == 2 && a.cursor) {
        // first-level bins, then partitions, each reserved run by run on the bin's cursor
        init(P.regions1, P.Q, false);
        if (aux)
            scatter_cursor<true>(a, P, a.keys, a.vals, a.aux_in, nullptr, nullptr, 0, dim3(P.W1, 1), P.W1, P.shiftA,
                                 255, a.k1, a.v1, a.a1, a.cur1, P.cap1, P.subs, 0, st);
        else
            scatter_cursor<false>(a, P, a.keys, a.vals, nullptr, nullptr, nullptr, 0, dim3(P.W1, 1), P.W1, P.shiftA,
                                  255, a.k1, a.v1, a.a1, a.cur1, P.cap1, P.subs, 0, st);
        const uint32_t maskB = (1u << P.bitsB) - 1;
        const uint64_t* hi1 = reinterpret_cast<const uint64_t*>(a.cur1);
        if (aux)
            scatter_cursor<true>(a, P, a.k1, a.v1, a.a1, a.begA, hi1, P.cap1, dim3(P.W2c, P.regions1), P.W2c, 0, maskB, a.k2,
                                 a.v2, a.a2, a.cur2, P.capQ, 0, P.subs, st);
        else
            scatter_cursor<false>(a, P, a.k1, a.v1, nullptr, a.begA, hi1, P.cap1, dim3(P.W2c, P.regions1), P.W2c, 0, maskB,
                                  a.k2, a.v2, a.a2, a.cur2, P.capQ, 0, P.subs, st);
        o.keys = a.k2;
        o.vals = a.v2;
        o.aux = a.a2;
        o.aux_is_pos = aux ? 0 : 1;
        o.qbeg = a.begQ;
        o.qend = reinterpret_cast<const uint64_t*>(a.cur2);
        o.qcap = P.capQ;
    } else if (P.passes == 2) {
        count(a.keys, nullptr, dim3(P.W1, 1), P.W1, P.shiftA, 255);
        scan_matrix(a, (uint64_t)kBins * P.W1, st);
        if (aux)
            scatter<true>(a, a.keys, a.vals, a.aux_in, nullptr, dim3(P.W1, 1), P.W1, P.shiftA, 255, a.k1, a.v1,
                          a.a1, st);
        else
            scatter<false>(a, a.keys, a.vals, nullptr, nullptr, dim3(P.W1, 1), P.W1, P.shiftA, 255, a.k1, a.v1,
                           a.a1, st);
        hipLaunchKernelGGL(k_extract_offsets, (P.binsA + 256) / 256, 256, 0, st, a.off, P.W1, 8u, P.binsA, n, a.offA);
        const uint32_t maskB = (1u << P.bitsB) - 1;
        count(a.k1, a.offA, dim3(P.W2, P.binsA), P.W2, 0, maskB);
        scan_matrix(a, (uint64_t)P.binsA * kBins * P.W2, st);
        if (aux)
            scatter<true>(a, a.k1, a.v1, a.a1, a.offA, dim3(P.W2, P.binsA), P.W2, 0, maskB, a.k2, a.v2, a.a2, st);
        else
            scatter<false>(a, a.k1, a.v1, nullptr, a.offA, dim3(P.W2, P.binsA), P.W2, 0, maskB, a.k2, a.v2, a.a2, st);
        hipLaunchKernelGGL(k_extract_offsets, (P.Q + 256) / 256, 256, 0, st, a.off, P.W2, P.bitsB, P.Q, n, a.offQ);
        o.keys = a.k2;
        o.vals = a.v2;
        o.aux = a.a2;
        o.aux_is_pos = aux ? 0 : 1;
    } else {
        // top 8 bits into k1, the middle 8 bits within each first-level bin into k2, the
        // low bits within each second-level bin back into k1
        count(a.keys, nullptr, dim3(P.W1, 1), P.W1, P.shiftA, 255);
        scan_matrix(a, (uint64_t)kBins * P.W1, st);
        if (aux)
            scatter<true>(a, a.keys, a.vals, a.aux_in, nullptr, dim3(P.W1, 1), P.W1, P.shiftA, 255, a.k1, a.v1,
                          a.a1, st);
        else
            scatter<false>(a, a.keys, a.vals, nullptr, nullptr, dim3(P.W1, 1), P.W1, P.shiftA, 255, a.k1, a.v1,
                           a.a1, st);
        hipLaunchKernelGGL(k_extract_offsets, (P.binsA + 256) / 256, 256, 0, st, a.off, P.W1, 8u, P.binsA, n, a.offA);
        count(a.k1, a.offA, dim3(P.W2, P.binsA), P.W2, P.bitsC, 255);
        scan_matrix(a, (uint64_t)P.binsA * kBins * P.W2, st);
        if (aux)
            scatter<true>(a, a.k1, a.v1, a.a1, a.offA, dim3(P.W2, P.binsA), P.W2, P.bitsC, 255, a.k2, a.v2, a.a2, st);
        else
            scatter<false>(a, a.k1, a.v1, nullptr, a.offA, dim3(P.W2, P.binsA), P.W2, P.bitsC, 255, a.k2, a.v2,
                           a.a2, st);
        hipLaunchKernelGGL(k_extract_offsets, (P.binsAB + 256) / 256, 256, 0, st, a.off, P.W2, 8u, P.binsAB, n,
                           a.offAB);
        const uint32_t maskC = (1u << P.bitsC) - 1;
        count(a.k2, a.offAB, dim3(P.W3, P.binsAB), P.W3, 0, maskC);
        scan_matrix(a, (uint64_t)P.binsAB * kBins * P.W3, st);
        if (aux)
            scatter<true>(a, a.k2, a.v2, a.a2, a.offAB, dim3(P.W3, P.binsAB), P.W3, 0, maskC, a.k1, a.v1, a.a1, st);
        else
            scatter<false>(a, a.k2, a.v2, nullptr, a.offAB, dim3(P.W3, P.binsAB), P.W3, 0, maskC, a.k1, a.v1,
                           nullptr, st);
        hipLaunchKernelGGL(k_extract_offsets, (P.Q + 256) / 256, 256, 0, st, a.off, P.W3, P.bitsC, P.Q, n, a.offQ);
        o.keys = a.k1;
        o.vals = a.v1;
        o.aux = a.a1;
        o.aux_is_pos = aux ? 0 : 1;
    }
    if (a.fused) {
        // the fused final pass sizes the partitions and finds their cell bases itself
        hipError_t e = hipGetLastError();
        return e == hipSuccess ? FKS_OK : hip_fail(e);
    }
    FKS_TIMED("fks_part_sizes", st,
              hipLaunchKernelGGL(k_psizes, P.Q, kPB, 0, st, o.keys, n, a.A, a.magic, a.offQ, a.sizes, a.G, a.sqQ,
                                 a.oversize));
    {
        // cell bases of the partitions (exclusive scan of their sums of squares) and S
        const uint32_t nt = (uint32_t)exscan_tiles(P.Q);
        hipLaunchKernelGGL(k_xscan_reduce, nt, kPB, 0, st, a.sqQ, (uint64_t)P.Q, a.tsum);
        hipLaunchKernelGGL(k_scan_counts, 1, 1024, 0, st, a.tsum, nt, a.tpre, nullptr, a.S_dev);
        hipLaunchKernelGGL(k_xscan_down64, nt, kPB, 0, st, a.sqQ, (uint64_t)P.Q, a.tpre, a.cbase);
    }
    hipError_t e = hipGetLastError();
    return e == hipSuccess ? FKS_OK : hip_fail(e);
}

// Threads per partition.  With few partitions the pass is one workgroup's chain of about 34000
// cycles (16 us), most of it instructions, and 512 threads shorten it; with many it is bound by
// the instructions all waves issue, and wider workgroups add barriers.  Build, one lookup and release
// with 256, 512 and 1024 threads: 2^16 keys 54.7, 51.4 and 50.0 us, 2^19 72.4, 70.5 and 76.7,
// 2^20 87.0, 90.8 and 102.4, 10^7 285, 373 and 512.
constexpr uint32_t kWideFinalThreads = 512, kWideFinalParts = 512;
// Partitions up to which the pass itself writes the outcome to the host: 1000 keys 43.3 and 40.6 us,
// 2^16 51.4 and 49.0, 2^18 (256 partitions) 56.3 and 56.2, 2^19 70.5 and 74.0.
constexpr uint32_t kReportParts = 128;

template <bool AUX, bool STR>
static void launch_fused(const PartArgs& a, PartOut& o, const Triple* C, uint32_t T, Group* header, Cell* slots,
                         uint32_t* flags, const int64_t* ctx_off, const uint8_t* ctx_bytes, const uint32_t* reject,
                         uint64_t cap, hipStream_t st) {
    const uint32_t Q = o.plan.Q;
    // the look-back words (in the cell-base scratch) start at zero (the cursor passes' set-up has
    // cleared them already)
    if (!o.prezeroed)
        hipLaunchKernelGGL(k_zero_words, (2 * Q + 255) / 256, 256, 0, st, reinterpret_cast<uint32_t*>(a.cbase),
                           (uint64_t)2 * Q);
    const FuseArgs fa{a.cbase, a.S_dev, a.oversize, Q, tl_patience, o.qend, o.qcap, nullptr,
                      Q <= kReportParts ? a.outcome : nullptr, a.start.clear, a.start.words, a.done};
    auto launch = [&](auto kernel, uint32_t threads) {
        FKS_TIMED("fks_part_final", st,
                  hipLaunchKernelGGL(kernel, Q, threads, 0, st, o.keys, o.vals, AUX ? o.aux : nullptr,
                                     AUX ? o.aux_is_pos : 1, a.n, a.A, a.magic, o.qbeg, a.cbase, a.sizes, a.G, C, T,
                                     header, slots, flags, ctx_off, ctx_bytes, nullptr, nullptr, reject, cap, fa));
    };
    o.reported = fa.outcome != nullptr;
    if (Q <= kWideFinalParts) launch(k_pfinal<AUX, STR, false, true, kWideFinalThreads>, kWideFinalThreads);
    else launch(k_pfinal<AUX, STR, false, true>, kPB);
}

int part_finish(const PartArgs& a, PartOut& o, const Triple* C, uint32_t T, Group* header, Cell* slots,
                uint32_t* flags, const int64_t* ctx_off, const uint8_t* ctx_bytes, const uint8_t* given_t,
                const uint32_t* reject, uint64_t cap, hipStream_t st) {
    if (a.fused && !given_t) {
        if (a.aux && a.str)
            launch_fused<true, true>(a, o, C, T, header, slots, flags, ctx_off, ctx_bytes, reject, cap, st);
        else if (a.aux)
            launch_fused<true, false>(a, o, C, T, header, slots, flags, nullptr, nullptr, reject, cap, st);
        else
            launch_fused<false, false>(a, o, C, T, header, slots, flags, nullptr, nullptr, reject, cap, st);
        o.prezeroed = false;   // the look-back words are used up: a second run clears them again
        hipError_t e = hipGetLastError();
        return e == hipSuccess ? FKS_OK : hip_fail(e);
    }
    if (a.aux && a.str)
        FKS_TIMED("fks_part_final", st,
                  hipLaunchKernelGGL((k_pfinal<true, true>), o.plan.Q, kPB, 0, st, o.keys, o.vals,
                                     o.aux, o.aux_is_pos, a.n, a.A, a.magic, a.offQ, a.cbase, a.sizes, a.G, C, T,
                                     header, slots, flags, ctx_off, ctx_bytes, given_t, nullptr, reject, cap));
    else if (a.aux)
        FKS_TIMED("fks_part_final", st,
                  hipLaunchKernelGGL((k_pfinal<true, false>), o.plan.Q, kPB, 0, st, o.keys, o.vals,
                                     o.aux, o.aux_is_pos, a.n, a.A, a.magic, a.offQ, a.cbase, a.sizes, a.G, C, T,
                                     header, slots, flags, nullptr, nullptr, given_t, nullptr, reject, cap));
    else
        FKS_TIMED("fks_part_final", st,
                  hipLaunchKernelGGL((k_pfinal<false, false>), o.plan.Q, kPB, 0, st, o.keys, o.vals,
                                     nullptr, 1, a.n, a.A, a.magic, a.offQ, a.cbase, a.sizes, a.G, C, T, header,
                                     slots, flags, nullptr, nullptr, given_t, nullptr, reject, cap));
    hipError_t e = hipGetLastError();
    return e == hipSuccess ? FKS_OK : hip_fail(e);
}

}  // namespace fks

namespace fks {

constexpr uint32_t kWideItems = 4;   // records per thread of a wide map's tile

// What the scatter and the final pass of a batch start from: triples of attempt 0, the lists of
// tiles and partitions, cursors, look-back words and outcome words.
__global__ void k_wide_setup(const WideSeg* __restrict__ segs, uint32_t nseg, uint32_t T, Triple* __restrict__ Cpool,
                             WideLists w, uint64_t cap, uint32_t* __restrict__ flags) {
    const uint64_t at = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x, stride = (uint64_t)gridDim.x * blockDim.x;
    for (uint64_t i = at; i < (uint64_t)nseg * T; i += stride) {
        const WideSeg& sg = segs[i / T];
        Cpool[(uint64_t)sg.map * T + i % T] = level2_triple(sg.seed, 0, (uint32_t)(i % T));
    }
    for (uint64_t i = at; i < (uint64_t)nseg * kSegParts; i += stride) {
        const uint32_t seg = (uint32_t)(i / kSegParts), j = (uint32_t)(i % kSegParts);
        const WideSeg& sg = segs[seg];
        if (j < (sg.n + kPartBuckets - 1) / kPartBuckets) {
            const uint64_t p = sg.part0 + j;
            w.parts[p] = seg * kSegParts + j;
            w.cursor[p] = p * cap;
            w.state[p] = 0;
        }
        if (j < sg.tiles) w.tiles[sg.tile0 + j] = make_uint2(seg, j * ((sg.n + sg.tiles - 1) / sg.tiles));
        if (j < 4) flags[4 * (uint64_t)seg + j] = 0;
    }
}

static size_t wide_carve(uint32_t nseg, uint64_t parts, uint64_t tiles, char* base, WideLists& w) {
    size_t total = 0;
    auto carve = [&](auto*& field, size_t bytes) {
        if (base) field = reinterpret_cast<std::remove_reference_t<decltype(field)>>(base + total);
        total += (bytes + 255) & ~(size_t)255;
    };
    const uint64_t cap = part_region(kPartBuckets);
    carve(w.keys, 8 * parts * cap);
    carve(w.vals, 4 * parts * cap);
    carve(w.cursor, 8 * parts);
    carve(w.state, 8 * parts);
    carve(w.S, 8 * (size_t)nseg);
    carve(w.tiles, sizeof(uint2) * tiles);
    carve(w.parts, 4 * parts);
    return total;
}

uint32_t wide_tiles(uint32_t n) { return (n + kWideItems * kPScatterThreads - 1) / (kWideItems * kPScatterThreads); }

// runs are placed by 32 bits, which a cursor stays within also when all records of a map land past its
// region's end
uint64_t wide_parts_max() { return ((1ull << 32) - (uint64_t)kSegParts * kPartBuckets) / part_region(kPartBuckets) - 1; }

size_t wide_scratch_bytes(uint32_t nseg, uint64_t parts, uint64_t tiles) {
    WideLists none{};
    return wide_carve(nseg, parts, tiles, nullptr, none);
}

// Built like a single map by the cursor passes, all maps at once, over lists of tiles and partitions
// without empty entries: 2.9 * 10^7 keys in 1023 maps 480 us (scatter 141, final pass 332).  With
// a count pass, a size pass and 64 partitions for every map it was 790 us (count 55,
// scatter 162, sizes 80, final pass 467).
int wide_build(const uint64_t* d_keys, const uint32_t* d_vals, const WideSeg* segs, uint32_t nseg, uint64_t parts,
               uint64_t tiles, Triple* Cpool, uint32_t T, Group* hdr_pool, Cell* slot_pool, uint32_t* flags,
               uint64_t** S, void* scratch, hipStream_t st) {
    if (nseg == 0) return FKS_OK;
    WideLists w{};
    wide_carve(nseg, parts, tiles, (char*)scratch, w);
    *S = w.S;
    const uint64_t cap = part_region(kPartBuckets);
    const Triple A0{0, 0, 0};
    hipLaunchKernelGGL(k_wide_setup, (unsigned)std::min<uint64_t>(4096, ((uint64_t)nseg * kSegParts + 255) / 256), 256, 0,
                       st, segs, nseg, T, Cpool, w, cap, flags);
    FKS_TIMED("fks_wide_scatter", st,
              hipLaunchKernelGGL((k_dscatter<false, kWideItems, kPScatterThreads, true>), dim3((unsigned)tiles),
                                 kPScatterThreads, 0, st, d_keys, d_vals, nullptr, 0ull, A0, 0ull, nullptr, 1u, 0u,
                                 kSegParts - 1, nullptr, w.keys, w.vals, nullptr, segs, w.tiles, w.cursor, nullptr, cap,
                                 flags, 0ull));
    const FuseArgs fa{w.state, w.S, nullptr, (uint32_t)parts, tl_patience, (const uint64_t*)w.cursor, cap, w.parts,
                      nullptr, nullptr, 0, nullptr};
    FKS_TIMED("fks_wide_final", st,
              hipLaunchKernelGGL((k_pfinal<false, false, true, true>), (unsigned)parts, kPB, 0, st, w.keys, w.vals,
                                 nullptr, 1, 0ull, A0, 0ull, nullptr, nullptr, nullptr, 0ull, Cpool, T, hdr_pool,
                                 slot_pool, flags, nullptr, nullptr, nullptr, segs, nullptr, ~0ull, fa));
    const hipError_t e = hipGetLastError();
    return e == hipSuccess ? FKS_OK : hip_fail(e);
}

}  // namespace fks
