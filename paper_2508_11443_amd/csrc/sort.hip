// Sample sort: the pairs of a sorted or Eytzinger map.
//
// Splitters from a sorted sample cut the keys into at most 256 buckets, splitters from a sample
// of each bucket cut that into leaves of about 1344 keys, and a workgroup per leaf sorts it in
// LDS and writes it to its place.  Every pair is read and written three times whatever the
// keys' distribution (eight digit passes of a radix sort read the keys twice and write the pairs
// once each).  Buckets and leaves are regions of fixed capacity that the scatter passes fill
// through cursors; a region that overflows is reported and the caller sorts another way.
//
// Splitters rather than key bits because a map's keys need not be spread over the 64-bit range:
// half of them may be one run of consecutive integers.
//
// 2^24 pairs, half of them one dense run: 1.37 ms in eight digit passes, 0.45 ms here (scatter
// passes 135 and 109 us, leaves with their separators 151 us, splitters 57 us, of which 30 us
// for the one bucket that holds the run's end); 10^7 even keys 0.97 and 0.27 ms.  The bytes are
// 1.2 GB: the passes run at 3.0, 3.7 and 2.7 TB/s.
#include <hip/hip_runtime.h>

#include <algorithm>

#include "fks_internal.hpp"
#include "prof.hpp"
#include "sort.hpp"

namespace fks {

constexpr uint32_t kSsBins = 256;          // most buckets, and most leaves of a bucket
constexpr uint32_t kSsSample = 8192;       // most sampled keys (of all keys, and of a bucket)
constexpr uint32_t kSsOver = 64;           // sampled keys per part, as long as they fit the sample
// A leaf has 1344 keys on average and holds 3584: a bucket of 256 parts from 32 sampled keys each
// is above 1.6 times its share about once in 10^3 sorts, and its leaves, from 64 sampled keys
// each (32 beyond 128 leaves), above a further 1.67 times about 3 in 10^6.
// 3584 pairs and the counters are 51 KB of LDS: three workgroups per CU.
constexpr uint32_t kLeafMean = 1344, kLeafCap = 3584, kLeafThreads = 512, kLeafBins = 2048;
constexpr uint32_t kSsThreads = 1024;
static_assert(kSampleSortMax == (uint64_t)kSsBins * kSsBins * kLeafMean, "the limit stated in the header");

struct SortPlan {
    uint32_t levels;            // scatter passes: 0, 1 or 2
    uint32_t bins1, bins2;      // buckets; leaves of a bucket (two passes)
    uint32_t leaves;
    uint32_t sample1, sample2;  // sampled keys
    uint64_t cap1;              // capacity of a bucket's region (two passes)
};

static SortPlan sort_plan(uint64_t n) {
    SortPlan p{};
    p.leaves = 1;
    if (n <= kLeafCap) return p;
    const uint64_t want = (n + kLeafMean - 1) / kLeafMean;
    p.levels = want <= kSsBins ? 1 : 2;
    p.bins1 = p.levels == 1 ? (uint32_t)want : kSsBins;
    p.bins2 = p.levels == 1 ? 1 : (uint32_t)((want + kSsBins - 1) / kSsBins);
    p.leaves = p.bins1 * p.bins2;
    p.sample1 = std::min<uint32_t>(kSsSample, kSsOver * p.bins1);
    p.sample2 = std::min<uint32_t>(kSsSample, kSsOver * p.bins2);
    p.cap1 = (5 * (n / p.bins1) / 2 + 1023) & ~1023ull;
    return p;
}

// ---- sorting in LDS --------------------------------------------------------------------

template <uint32_t CAP, uint32_t BINS, uint32_t THREADS, bool VALS>
struct LdsSort {
    uint64_t key[CAP];
    uint32_t val[VALS ? CAP : 1];
    uint32_t start[BINS + 1];
    uint64_t lo[THREADS / 64], hi[THREADS / 64];
    uint32_t wsum[THREADS / 64];
    uint32_t crowded;
};

// Sorts n <= CAP pairs: load(i, key, val) gives pair i, emit(r, key, val) takes the pair of rank
// r (equal keys take different ranks); while_loading runs once the loads are on their way and
// before the first barrier, before_emit after the last.  Returns whether the calling thread saw two equal keys.
//
// The range of the keys is cut into up to BINS equal bins, pairs are grouped by bin (one
// LDS atomic each), and a pair's rank in its bin comes from comparing it with the others there:
// about one other when the keys are spread evenly, as they nearly are inside a leaf.  A crowded
// bin (keys clustered within their leaf) sends the whole leaf to a bitonic network instead.
template <uint32_t CAP, uint32_t BINS, uint32_t THREADS, bool VALS, typename Load, typename Wait, typename Ready, typename Emit>
__device__ __forceinline__ bool lds_sort(LdsSort<CAP, BINS, THREADS, VALS>& L, uint32_t n, Load load, Wait while_loading,
                                         Ready before_emit, Emit emit) {
    constexpr uint32_t ITEMS = CAP / THREADS, PER = BINS / THREADS, kCrowd = 24;
    static_assert(CAP % THREADS == 0 && BINS % THREADS == 0, "whole rounds");
    const uint32_t tid = threadIdx.x, lane = tid & 63u, wv = tid >> 6;
    uint64_t x[ITEMS];
    uint32_t v[VALS ? ITEMS : 1];
    uint64_t lo = ~0ull, hi = 0;
#pragma unroll
    for (uint32_t k = 0; k < ITEMS; ++k) {
        const uint32_t i = tid + k * THREADS;
        uint32_t val = 0;
        if (i < n) load(i, x[k], val);
        if (VALS) v[k] = val;
    }
    while_loading();
#pragma unroll
    for (uint32_t k = 0; k < ITEMS; ++k) {
        if (tid + k * THREADS < n) {
            lo = min(lo, x[k]);
            hi = max(hi, x[k]);
        }
    }
    for (uint32_t b = tid; b <= BINS; b += THREADS) L.start[b] = 0;
    for (int d = 32; d >= 1; d >>= 1) {
        lo = min(lo, (uint64_t)__shfl_xor((unsigned long long)lo, d, 64));
        hi = max(hi, (uint64_t)__shfl_xor((unsigned long long)hi, d, 64));
    }
    if (lane == 0) {
        L.lo[wv] = lo;
        L.hi[wv] = hi;
    }
    if (tid == 0) L.crowded = 0;
    __syncthreads();
#pragma unroll
    for (uint32_t w = 0; w < THREADS / 64; ++w) {
        lo = min(lo, L.lo[w]);
        hi = max(hi, L.hi[w]);
    }
    const uint32_t bits = hi > lo ? 64u - (uint32_t)__clzll((long long)(hi - lo)) : 0u;
    constexpr uint32_t kBinBits = 31 - __builtin_clz(BINS);
    const uint32_t shift = bits > kBinBits ? bits - kBinBits : 0;
    auto bin_of = [&](uint64_t key) { return (uint32_t)((key - lo) >> shift); };
    uint32_t arrived[ITEMS];
    bool crowded = false;
#pragma unroll
    for (uint32_t k = 0; k < ITEMS; ++k) {
        if (tid + k * THREADS < n) {
            arrived[k] = atomicAdd(&L.start[bin_of(x[k])], 1u);
            crowded |= arrived[k] >= kCrowd;
        }
    }
    if (crowded) L.crowded = 1;
    __syncthreads();
    const bool network = L.crowded != 0;
    if (!network) {
        // counts to starts, PER consecutive bins a thread
        uint32_t c[PER], sum = 0;
#pragma unroll
        for (uint32_t b = 0; b < PER; ++b) {
            c[b] = L.start[tid * PER + b];
            sum += c[b];
        }
        uint32_t inc = sum;
#pragma unroll
        for (int d = 1; d < 64; d <<= 1) {
            const uint32_t u = __shfl_up(inc, d, 64);
            if (lane >= (uint32_t)d) inc += u;
        }
        if (lane == 63) L.wsum[wv] = inc;
        __syncthreads();
        uint32_t at = inc - sum;
        for (uint32_t w = 0; w < wv; ++w) at += L.wsum[w];
#pragma unroll
        for (uint32_t b = 0; b < PER; ++b) {
            L.start[tid * PER + b] = at;
            at += c[b];
        }
        if (tid == 0) L.start[BINS] = n;
        __syncthreads();
#pragma unroll
        for (uint32_t k = 0; k < ITEMS; ++k) {
            if (tid + k * THREADS < n) {
                const uint32_t e = L.start[bin_of(x[k])] + arrived[k];
                L.key[e] = x[k];
                if (VALS) L.val[VALS ? e : 0] = v[VALS ? k : 0];
            }
        }
    } else {
#pragma unroll
        for (uint32_t k = 0; k < ITEMS; ++k) {
            const uint32_t i = tid + k * THREADS;
            if (i < n) {
                L.key[i] = x[k];
                if (VALS) L.val[VALS ? i : 0] = v[VALS ? k : 0];
            }
        }
        // all comparators put the smaller key at the lower place, so places from n on (which
        // would hold the largest keys) need not exist
        uint32_t size = 2;
        while (size < n) size <<= 1;
        auto step = [&](uint32_t t, uint32_t k, uint32_t j) {
            const uint32_t half = j >> 1;
            const uint32_t i = (t & ~(half - 1)) * 2 + (t & (half - 1));
            const uint32_t p = j == k ? i ^ (k - 1) : i + half;   // the first step of a merge is mirrored
            if (p < n) {
                const uint64_t a = L.key[i], b = L.key[p];
                if (b < a) {
                    L.key[i] = b;
                    L.key[p] = a;
                    if (VALS) {
                        const uint32_t va = L.val[VALS ? i : 0];
                        L.val[VALS ? i : 0] = L.val[VALS ? p : 0];
                        L.val[VALS ? p : 0] = va;
                    }
                }
            }
        };
        // 64 consecutive comparators of a step of at most 128 places touch the same 128 places in
        // every such step: one wave runs these steps without the others
        for (uint32_t k = 2; k <= size; k <<= 1) {
            uint32_t j = k;
            for (; j > 128; j >>= 1) {
                __syncthreads();
                for (uint32_t t = tid; t < size / 2; t += THREADS) step(t, k, j);
            }
            if (k >= 128 || k == 2) __syncthreads();
            for (uint32_t t = tid; t < size / 2; t += THREADS)
                for (uint32_t i = j; i >= 2; i >>= 1) {
                    step(t, k, i);
                    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
                    __builtin_amdgcn_wave_barrier();
                }
        }
    }
    __syncthreads();
    before_emit();
    bool dup = false;
#pragma unroll
    for (uint32_t k = 0; k < ITEMS; ++k) {
        const uint32_t i = tid + k * THREADS;
        if (i >= n) break;
        const uint64_t key = L.key[i];
        uint32_t r = i;
        if (network) {
            dup |= i > 0 && L.key[i - 1] == key;
        } else {
            const uint32_t b = bin_of(key), s = L.start[b], e = L.start[b + 1];
            r = s;
            for (uint32_t j = s; j < e; ++j) {
                const uint64_t other = L.key[j];
                r += other < key || (other == key && j < i) ? 1u : 0u;
                dup |= other == key && j != i;
            }
        }
        emit(r, key, VALS ? L.val[VALS ? i : 0] : 0u);
    }
    return dup;
}

// ---- splitters -------------------------------------------------------------------------

// A sample of s out of count positions (s <= 8192, count < 2^32): one in each of s stretches whose
// lengths differ by at most one, so that no position comes twice.
struct Sampled {
    uint32_t s, len, more;   // stretch k starts at k * len + k * more / s
    __device__ Sampled(uint32_t s_, uint32_t count) : s(s_), len(s_ ? count / s_ : 0), more(s_ ? count % s_ : 0) {}
    __device__ uint32_t at(uint32_t k) const {
        const uint32_t a = k * len + k * more / s, b = (k + 1) * len + (k + 1) * more / s;
        return a + (uint32_t)(((uint64_t)(b - a) * (uint32_t)(sm_fin(k + 1) >> 32)) >> 32);
    }
};

// Splitters: spl[b] parts bins b and b + 1 (bin of a key = number of splitters below it); unused
// ones are all ones.
//
// Of all n keys, from the sample that the set-up gathered: every block reads the whole sample into registers and finds the
// ranks of kRankKeys of its keys by comparing them with all (a compare and a bit count per 64
// keys): 10 us.  Sorting the sample in one workgroup took 33 us, and 104 us where half the keys
// were one dense run; with every block gathering the sample itself 20 us.
constexpr uint32_t kRankKeys = 32;
__global__ __launch_bounds__(kSsThreads) void k_ss_splitters(const uint64_t* __restrict__ sampled, uint32_t sample,
                                                            uint32_t bins, uint64_t* __restrict__ spl) {
    constexpr uint32_t ITEMS = kSsSample / kSsThreads;
    __shared__ uint64_t mine[kRankKeys];
    __shared__ uint32_t rank[kRankKeys];
    const uint32_t tid = threadIdx.x;
    uint64_t x[ITEMS];
#pragma unroll
    for (uint32_t k = 0; k < ITEMS; ++k) {
        const uint32_t i = tid + k * kSsThreads;
        x[k] = i < sample ? sampled[i] : ~0ull;   // never below a key
    }
    if (tid < kRankKeys) {
        const uint32_t i = blockIdx.x * kRankKeys + tid;
        mine[tid] = i < sample ? sampled[i] : ~0ull;
        rank[tid] = 0;
    }
    __syncthreads();
    for (uint32_t j = 0; j < kRankKeys; ++j) {
        const uint64_t y = mine[j];
        uint32_t c = 0;
#pragma unroll
        for (uint32_t k = 0; k < ITEMS; ++k) c += (uint32_t)__popcll(__ballot(x[k] < y));
        if ((tid & 63u) == 0) atomicAdd(&rank[j], c);
    }
    __syncthreads();
    if (tid < kRankKeys && blockIdx.x * kRankKeys + tid < sample) {
        const uint32_t r = rank[tid];
        // splitter c - 1 is the key of rank c * sample / bins
        for (uint32_t c = max(1u, (r * bins + sample - 1) / sample); c < bins && c * sample / bins == r; ++c)
            spl[c - 1] = mine[tid];
    }
}

// Of every bucket (its region [blockIdx.x * cap, end[blockIdx.x])), from a sample of its own.
__global__ __launch_bounds__(kSsThreads) void k_ss_bucket_splitters(const uint64_t* __restrict__ keys,
                                                                   const unsigned long long* __restrict__ end,
                                                                   uint64_t cap, uint32_t sample, uint32_t bins,
                                                                   uint64_t* __restrict__ spl) {
    __shared__ LdsSort<kSsSample, kSsSample, kSsThreads, false> L;
    const uint64_t at = blockIdx.x * cap, count = min((uint64_t)end[blockIdx.x] - at, cap);
    keys += at;
    spl += (uint64_t)blockIdx.x * kSsBins;
    const uint32_t s = (uint32_t)min((uint64_t)sample, count);
    if (s == 0) return;   // the whole block
    const Sampled of(s, (uint32_t)count);
    (void)lds_sort(L, s, [&](uint32_t i, uint64_t& x, uint32_t&) { x = keys[of.at(i)]; }, [] {}, [] {},
                   [&](uint32_t r, uint64_t x, uint32_t) {
                       for (uint32_t c = max(1u, (r * bins + s - 1) / s); c < bins && c * s / bins == r; ++c)
                           spl[c - 1] = x;
                   });
}

// cursors at the starts of their regions, splitters and the ends of the separators' levels all
// ones, the sample gathered
__global__ void k_ss_setup(const uint64_t* __restrict__ keys, uint64_t n, uint32_t sample,
                           uint64_t* __restrict__ sampled, unsigned long long* __restrict__ cur1, uint32_t bins1, uint64_t cap1,
                           unsigned long long* __restrict__ cur2, uint32_t leaves, uint64_t* __restrict__ spl,
                           uint32_t splitters, SepIndex sep, uint64_t* __restrict__ index,
                           SortFlags* __restrict__ flags) {
    const uint32_t at = blockIdx.x * blockDim.x + threadIdx.x, stride = gridDim.x * blockDim.x;
    const Sampled of(sample, (uint32_t)n);
    for (uint32_t i = at; i < sample; i += stride) sampled[i] = keys[of.at(i)];
    for (uint32_t i = at; i < bins1; i += stride) cur1[i] = i * cap1;
    for (uint32_t i = at; i < leaves; i += stride) cur2[i] = (unsigned long long)i * kLeafCap;
    for (uint32_t i = at; i < splitters; i += stride) spl[i] = ~0ull;
    for (uint32_t l = 1; l <= sep.levels; ++l) {
        const uint64_t end = l < sep.levels ? sep.at[l + 1] : sep.total;
        for (uint64_t e = sep.at[l] + sep.count[l] + at; e < end; e += stride) index[e] = ~0ull;
    }
    if (at == 0) *flags = SortFlags{0, 0};
}

// ---- scatter -----------------------------------------------------------------------------

// Pairs into the regions of their bins: each tile is grouped by bin in LDS, reserves a run per bin
// on the bin's cursor and writes the runs.  Bound by memory and by the exposed phases of the one
// workgroup that a CU's LDS holds at the large tile; the small tile is for inputs that would
// leave most CUs without one.
template <uint32_t ITEMS>
__global__ __launch_bounds__(kSsThreads) void k_ss_scatter(
    const uint64_t* __restrict__ keys, const uint32_t* __restrict__ vals, uint64_t n,
    const unsigned long long* __restrict__ end, uint64_t in_cap, const uint64_t* __restrict__ spl, uint32_t bins,
    unsigned long long* __restrict__ cursor, uint64_t cap, uint64_t* __restrict__ keys_out,
    uint32_t* __restrict__ vals_out, SortFlags* __restrict__ flags) {
    constexpr uint32_t TILE = kSsThreads * ITEMS;
    __shared__ uint64_t skey[TILE];
    __shared__ uint32_t sval[TILE];
    __shared__ uint8_t sbin[TILE];
    __shared__ uint64_t cut[kSsBins];
    __shared__ uint64_t to[kSsBins], room[kSsBins];   // where a bin's run goes, and its region's end
    __shared__ uint32_t tcnt[kSsBins], toff[kSsBins], wsum[kSsBins / 64];
    const uint32_t tid = threadIdx.x;
    uint32_t seg = blockIdx.y, worker = blockIdx.x;
    if (gridDim.y > 1) {
        // all workers of a bucket on one XCD (workgroups are dealt to them in turn), where the lines that
        // several of their runs share meet
        const uint32_t l = seg * gridDim.x + worker, turn = l >> 3;
        if (l < (gridDim.y & ~7u) * gridDim.x) {
            seg = turn / gridDim.x * 8 + (l & 7u);
            worker = turn % gridDim.x;
        }
    }
    uint64_t lo = 0, hi = n;
    if (end) {
        lo = seg * in_cap;
        hi = min((uint64_t)end[seg], lo + in_cap);
        spl += (uint64_t)seg * kSsBins;
    }
    const uint64_t chunk = (hi - lo + gridDim.x - 1) / gridDim.x;
    const uint64_t a = min(hi, lo + worker * chunk), b = min(hi, a + chunk);
    if (tid < kSsBins) {
        cut[tid] = spl[tid];
        room[tid] = ((uint64_t)seg * bins + tid + 1) * cap;
    }
    uint32_t step0 = 1;
    while (step0 < bins) step0 <<= 1;
    uint64_t x[ITEMS];
    uint32_t v[ITEMS];
    auto load = [&](uint64_t ts) {
#pragma unroll
        for (uint32_t k = 0; k < ITEMS; ++k) {
            const uint64_t i = ts + tid + (uint64_t)k * kSsThreads;
            x[k] = i < b ? keys[i] : 0;
            v[k] = i < b ? vals[i] : 0;
        }
    };
    if (a < b) load(a);
    for (uint64_t ts = a; ts < b; ts += TILE) {
        if (tid < kSsBins) tcnt[tid] = 0;
        __syncthreads();
        uint32_t bin[ITEMS], rank[ITEMS];
#pragma unroll
        for (uint32_t k = 0; k < ITEMS; ++k) bin[k] = 0;
        for (uint32_t st = step0 >> 1; st; st >>= 1) {
#pragma unroll
            for (uint32_t k = 0; k < ITEMS; ++k) bin[k] += cut[bin[k] + st - 1] < x[k] ? st : 0u;
        }
#pragma unroll
        for (uint32_t k = 0; k < ITEMS; ++k)
            if (ts + tid + (uint64_t)k * kSsThreads < b) rank[k] = atomicAdd(&tcnt[bin[k]], 1u);
        __syncthreads();
        uint32_t c = 0, inc = 0;
        if (tid < kSsBins) {
            c = tcnt[tid];
            if (c) {
                const unsigned long long at = atomicAdd(&cursor[(uint64_t)seg * bins + tid], (unsigned long long)c);
                to[tid] = at;
                if (at + c > room[tid]) atomicOr(&flags->overflow, 1u);
            }
            inc = c;
#pragma unroll
            for (int d = 1; d < 64; d <<= 1) {
                const uint32_t u = __shfl_up(inc, d, 64);
                if ((tid & 63u) >= (uint32_t)d) inc += u;
            }
            if ((tid & 63u) == 63u) wsum[tid >> 6] = inc;
        }
        __syncthreads();
        if (tid < kSsBins) {
            uint32_t pre = inc - c;
            for (uint32_t w = 0; w < tid >> 6; ++w) pre += wsum[w];
            toff[tid] = pre;
        }
        __syncthreads();
#pragma unroll
        for (uint32_t k = 0; k < ITEMS; ++k) {
            if (ts + tid + (uint64_t)k * kSsThreads < b) {
                const uint32_t e = toff[bin[k]] + rank[k];
                skey[e] = x[k];
                sval[e] = v[k];
                sbin[e] = (uint8_t)bin[k];
            }
        }
        if (ts + TILE < b) load(ts + TILE);   // in flight during the writes
        __syncthreads();
        const uint32_t cnt = (uint32_t)min((uint64_t)TILE, b - ts);
        for (uint32_t e = tid; e < cnt; e += kSsThreads) {
            const uint32_t bb = sbin[e];
            const uint64_t dest = to[bb] + (e - toff[bb]);
            if (dest < room[bb]) {
                keys_out[dest] = skey[e];
                vals_out[dest] = sval[e];
            }
        }
        __syncthreads();
    }
}

// ---- leaves -------------------------------------------------------------------------------

// In-order position in the perfect tree of depth H = floor(log2 n) of the key of rank r in the
// complete tree on n keys, whose last level holds leaves = n - 2^H + 1 nodes (the last level's nodes
// are the even positions; those from 2 * leaves on do not exist, so later ranks stand at odd
// positions only), and the place (0-based, level order) of in-order position p.
__device__ __forceinline__ uint64_t perfect_position(uint64_t r, uint64_t leaves) {
    return r < 2 * leaves ? r : 2 * r - 2 * leaves + 1;
}
__device__ __forceinline__ uint64_t eytzinger_place(uint64_t p, uint32_t H) {
    const uint32_t z = (uint32_t)__ffsll((long long)(p + 1)) - 1;
    return (1ull << (H - z)) + ((p + 1) >> (z + 1)) - 1;
}

// One leaf sorted and written to its place, in order or in level order (a stretch of consecutive
// ranks is a stretch of every level, so those writes are runs too), with the separators among
// its keys.  Its first rank is summed here from the counts of the buckets and leaves before it.
template <bool EYTZ>
__global__ __launch_bounds__(kLeafThreads) void k_ss_leaf(
    const uint64_t* __restrict__ keys, const uint32_t* __restrict__ vals, uint64_t n,
    const unsigned long long* __restrict__ cur1, uint64_t cap1, uint32_t bins2,
    const unsigned long long* __restrict__ cur2, uint64_t last_level, uint64_t* __restrict__ keys_out,
    uint32_t* __restrict__ vals_out, SepIndex sep, uint64_t* __restrict__ index, SortFlags* __restrict__ flags) {
    __shared__ LdsSort<kLeafCap, kLeafBins, kLeafThreads, true> L;
    __shared__ uint64_t before[kLeafThreads / 64];
    uint64_t base = 0;
    uint32_t count = (uint32_t)n;
    if (cur2) {
        const uint64_t at = (uint64_t)blockIdx.x * kLeafCap;
        // after an overflow the cursors count dropped pairs too, but no pair twice: ranks stay below n
        count = (uint32_t)min((uint64_t)cur2[blockIdx.x] - at, (uint64_t)kLeafCap);
        keys += at;
        vals += at;
    }
    if (count == 0) return;   // the whole block
    auto sum_before = [&] {
        if (!cur2) return;
        const uint32_t bucket = blockIdx.x / bins2, leaf = blockIdx.x % bins2, tid = threadIdx.x;
        static_assert(kLeafThreads == 2 * kSsBins, "a thread per bucket and per leaf of the bucket");
        uint64_t c = 0;
        if (tid < bucket) {
            c = cur1[tid] - tid * cap1;
        } else if (tid >= kSsBins && tid - kSsBins < leaf) {
            const uint64_t l = (uint64_t)bucket * bins2 + (tid - kSsBins);
            c = cur2[l] - l * kLeafCap;
        }
        for (int d = 32; d >= 1; d >>= 1) c += (uint64_t)__shfl_xor((unsigned long long)c, d, 64);
        if ((tid & 63u) == 0) before[tid >> 6] = c;
    };
    const bool dup = lds_sort(
        L, count,
        [&](uint32_t i, uint64_t& x, uint32_t& v) {
            x = __builtin_nontemporal_load(keys + i);
            v = __builtin_nontemporal_load(vals + i);
        },
        sum_before,
        [&] {
            if (!cur2) return;
#pragma unroll
            for (uint32_t w = 0; w < kLeafThreads / 64; ++w) base += before[w];
        },
        [&](uint32_t r, uint64_t x, uint32_t v) {
            const uint64_t p = EYTZ ? perfect_position(base + r, last_level) : base + r;
            const uint64_t to = EYTZ ? eytzinger_place(p, sep.depth) : p;
            keys_out[to] = x;
            vals_out[to] = v;
            if (((p + 1) & ((1ull << sep.gran) - 1)) == 0) {
                uint64_t e = (p + 1) >> sep.gran;
                for (uint32_t l = 1; l <= sep.levels; ++l) {
                    if (e - 1 < sep.count[l]) index[sep.at[l] + e - 1] = x;
                    if (e & 15u) break;
                    e >>= 4;
                }
            }
        });
    if (dup) atomicOr(&flags->dup, 1u);
}

// ---- host ------------------------------------------------------------------------------------

struct SortScratch {
    uint64_t *k1, *k2, *spl, *sampled;
    uint32_t *v1, *v2;
    unsigned long long *cur1, *cur2;
};

static size_t carve_sort(const SortPlan& p, char* base, SortScratch& s) {
    size_t total = 0;
    auto carve = [&](auto*& field, size_t bytes) {
        if (base) field = reinterpret_cast<std::remove_reference_t<decltype(field)>>(base + total);
        total += (bytes + 255) & ~(size_t)255;
    };
    if (p.levels == 0) return 256;
    const uint64_t r1 = p.levels == 2 ? p.cap1 * p.bins1 : 0, r2 = (uint64_t)p.leaves * kLeafCap;
    carve(s.k1, 8 * r1);
    carve(s.v1, 4 * r1);
    carve(s.k2, 8 * r2);
    carve(s.v2, 4 * r2);
    carve(s.spl, 8 * (size_t)kSsBins * (1 + kSsBins));
    carve(s.sampled, 8 * (size_t)p.sample1);
    carve(s.cur1, 8 * (size_t)p.bins1);
    carve(s.cur2, 8 * (size_t)p.leaves);
    return total;
}

size_t sample_sort_scratch(uint64_t n) {
    SortScratch none{};
    return carve_sort(sort_plan(n), nullptr, none);
}

void sample_sort(const uint64_t* keys, const uint32_t* vals, uint64_t n, bool eytz, uint64_t* keys_out,
                 uint32_t* vals_out, const SepIndex& sep, uint64_t* index, SortFlags* flags, void* scratch,
                 hipStream_t st) {
    const SortPlan p = sort_plan(n);
    SortScratch s{};
    carve_sort(p, (char*)scratch, s);
    const bool two = p.levels == 2;
    const uint32_t splitters = p.levels == 0 ? 0 : kSsBins * (1 + (two ? p.bins1 : 0));
    hipLaunchKernelGGL(k_ss_setup, std::max(1u, (std::max({splitters, p.leaves, p.sample1}) + 255) / 256), 256, 0, st, keys, n,
                       p.levels ? p.sample1 : 0, s.sampled, s.cur1, two ? p.bins1 : 0, p.cap1, s.cur2, p.levels ? p.leaves : 0, s.spl, splitters, sep, index, flags);
    // tiles of 10240 pairs (133 KB with the bins, one workgroup per CU) where two of them per worker
    // give every CU a worker, else of 2048
    auto scatter = [&](const uint64_t* kin, const uint32_t* vin, const unsigned long long* end, uint64_t in_cap,
                       uint32_t segs, const uint64_t* spl, uint32_t bins, unsigned long long* cur, uint64_t cap,
                       uint64_t* kout, uint32_t* vout) {
        auto launch = [&](auto kernel, uint32_t items, uint32_t tiles) {
            const uint64_t worker = (uint64_t)tiles * items * kSsThreads, per = (n + segs - 1) / segs;
            uint64_t workers = std::max<uint64_t>(1, (per + worker - 1) / worker);
            // the first pass fills all 256 CUs the same number of times: 2^24 pairs 136 us with 820
            // workers, 126 with 1024
            if (segs == 1 && tiles == 2) workers = (workers + 255) & ~255ull;
            const dim3 grid((unsigned)workers, segs);
            FKS_TIMED("fks_sort_scatter", st,
                      hipLaunchKernelGGL(kernel, grid, kSsThreads, 0, st, kin, vin, n, end, in_cap, spl, bins, cur,
                                         cap, kout, vout, flags));
        };
        if (n >= 256ull * 2 * 10 * kSsThreads) launch(k_ss_scatter<10>, 10, 2);
        else if (n >= 256ull * 5 * kSsThreads) launch(k_ss_scatter<5>, 5, 1);
        else launch(k_ss_scatter<2>, 2, 1);
    };
    if (p.levels) {
        FKS_TIMED("fks_sort_splitters", st,
                  hipLaunchKernelGGL(k_ss_splitters, (p.sample1 + kRankKeys - 1) / kRankKeys, kSsThreads, 0, st,
                                     s.sampled, p.sample1, p.bins1, s.spl));
        if (!two) {
            scatter(keys, vals, nullptr, 0, 1, s.spl, p.bins1, s.cur2, kLeafCap, s.k2, s.v2);
        } else {
            scatter(keys, vals, nullptr, 0, 1, s.spl, p.bins1, s.cur1, p.cap1, s.k1, s.v1);
            FKS_TIMED("fks_sort_splitters", st,
                      hipLaunchKernelGGL(k_ss_bucket_splitters, p.bins1, kSsThreads, 0, st, s.k1, s.cur1, p.cap1,
                                         p.sample2, p.bins2, s.spl + kSsBins));
            scatter(s.k1, s.v1, s.cur1, p.cap1, p.bins1, s.spl + kSsBins, p.bins2, s.cur2, kLeafCap, s.k2, s.v2);
        }
    }
    const uint64_t* kin = p.levels ? s.k2 : keys;
    const uint32_t* vin = p.levels ? s.v2 : vals;
    const uint64_t last_level = n - ((1ull << sep.depth) - 1);
    const uint32_t bins2 = two ? p.bins2 : std::max(1u, p.leaves);
    auto leaf = [&](auto kernel) {
        FKS_TIMED("fks_sort_leaf", st,
                  hipLaunchKernelGGL(kernel, p.leaves, kLeafThreads, 0, st, kin, vin, n, s.cur1, p.cap1, bins2, s.cur2,
                                     last_level, keys_out, vals_out, sep, index, flags));
    };
    if (eytz) leaf(k_ss_leaf<true>);
    else leaf(k_ss_leaf<false>);
}

}  // namespace fks
