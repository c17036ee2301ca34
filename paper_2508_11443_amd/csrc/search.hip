// The comparison maps of Section 4: the same (key, value) pairs as a sorted
// array searched by binary search, or in Eytzinger (level-order) layout.
//
// Build: the sample sort of sort.hip, which writes the pairs in order or in level order
// and reports equal keys.  Beyond its largest size, with a caller's allocator (whose memory
// may have been sized for it) and after one of its regions overflowed: a
// least-significant-digit radix sort of the pairs, eight passes of
// 8-bit digits.  Each pass is a per-worker digit count, an exclusive scan of the
// (digit, worker) count matrix, and a stable scatter: inside a 4096-record tile
// every wave owns a contiguous stretch and ranks its records round by round
// with a ballot match of the digit bits, so equal digits keep their input
// order, and the tile is staged in LDS sorted by digit so every digit's run is
// written to consecutive addresses.  A check of neighbours then rejects equal
// keys.  The Eytzinger layout gathers the sorted pairs into the level order of
// the complete binary search tree, computing each node's in-order rank in
// closed form.
// Lookup: a search through an index of separators (every 16th key in order, every
// 256th and so on; Eytzinger: every 4th, every 64th), whose top level is staged in
// LDS, a line of sixteen at a time by eight lanes together; the last step runs on
// the keys themselves.  Many needles against few keys, which stay in the nearest
// caches, have no lines to save: each lane searches alone (a branch-free binary
// search, or the descent with the tree's top levels in LDS).
#include <hip/hip_runtime.h>

#include <algorithm>

#include "fks_internal.hpp"
#include "ordered.hpp"
#include "partition.hpp"
#include "prof.hpp"
#include "sort.hpp"

struct fks_sorted {
    uint64_t n;
    uint32_t layout;
    int device;
    uint64_t* keys;   // n keys in layout order
    uint32_t* vals;   // their values
    uint64_t* index;  // separators, level by level
    fks::SepIndex sep;
    fks_allocator alloc;   // where keys and vals came from (has_alloc == 0: the library's pool)
    int has_alloc;
};

namespace fks {

constexpr uint32_t kRB = 256;                 // threads per block
constexpr uint32_t kRItems = 16;              // records per thread per tile
constexpr uint32_t kRTile = kRB * kRItems;    // 4096 records per tile
constexpr uint32_t kWaveSpan = 64 * kRItems;  // records of one wave inside a tile
constexpr uint32_t kTopSeps = 4095;           // most separators of the top level, staged in LDS (12 steps)
constexpr uint32_t kSortedGran = 4, kEytzGran = 2;   // the lowest separators: every 16th and every 4th key

__device__ __forceinline__ void chunk_of(uint64_t n, uint32_t W, uint64_t& a, uint64_t& b) {
    const uint64_t chunk = (n + W - 1) / W;
    a = min(n, (uint64_t)blockIdx.x * chunk);
    b = min(n, a + chunk);
}

// counts of one worker per digit: cnt[digit * W + worker]
__global__ __launch_bounds__(kRB) void k_rs_count(const uint64_t* __restrict__ keys, uint64_t n, uint32_t W,
                                                    uint32_t shift, uint32_t* __restrict__ cnt) {
    __shared__ uint32_t hist[256];
    uint64_t a, b;
    chunk_of(n, W, a, b);
    hist[threadIdx.x] = 0;
    __syncthreads();
    for (uint64_t ts = a; ts < b; ts += kRTile) {
        uint64_t x[kRItems];
#pragma unroll
        for (uint32_t k = 0; k < kRItems; ++k) {
            const uint64_t i = ts + threadIdx.x + (uint64_t)k * kRB;
            x[k] = i < b ? keys[i] : 0;
        }
#pragma unroll
        for (uint32_t k = 0; k < kRItems; ++k)
            if (ts + threadIdx.x + (uint64_t)k * kRB < b) atomicAdd(&hist[(x[k] >> shift) & 255u], 1u);
    }
    __syncthreads();
    cnt[(uint64_t)threadIdx.x * W + blockIdx.x] = hist[threadIdx.x];
}

// exclusive scan of one value per thread across the 256-thread block
__device__ __forceinline__ uint32_t rs_block_exscan(uint32_t v, uint32_t* wsum) {
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
#pragma unroll
    for (int q = 0; q < 4; ++q) pre += q < w ? wsum[q] : 0u;
    __syncthreads();
    return pre + inc - v;
}

// Stable scatter of one worker's chunk by the digit at `shift`.
__global__ __launch_bounds__(kRB) void k_rs_scatter(const uint64_t* __restrict__ keys,
                                                      const uint32_t* __restrict__ vals, uint64_t n, uint32_t W,
                                                      uint32_t shift, const uint32_t* __restrict__ off,
                                                      uint64_t* __restrict__ keys_out,
                                                      uint32_t* __restrict__ vals_out) {
    __shared__ uint64_t skey[kRTile];
    __shared__ uint32_t sval[kRTile];
    __shared__ uint32_t wcnt[4][256];   // per wave and digit: records ranked so far, then the wave's prefix
    __shared__ uint32_t toff[256], run[256];
    __shared__ uint32_t wsum[4];
    uint64_t a, b;
    chunk_of(n, W, a, b);
    const uint32_t tid = threadIdx.x, lane = tid & 63u, wv = tid >> 6;
    const uint64_t lt = (1ull << lane) - 1ull;
    run[tid] = off[(uint64_t)tid * W + blockIdx.x];
    // wave wv reads records ts + wv*1024 + k*64 + lane: coalesced rounds, and the
    // (wave, round, lane) order is the input order
    uint64_t x[kRItems];
    uint32_t v[kRItems];
    auto load = [&](uint64_t ts) {
#pragma unroll
        for (uint32_t k = 0; k < kRItems; ++k) {
            const uint64_t i = ts + wv * kWaveSpan + k * 64 + lane;
            x[k] = i < b ? keys[i] : 0;
            v[k] = i < b ? vals[i] : 0;
        }
    };
    if (a < b) load(a);
    for (uint64_t ts = a; ts < b; ts += kRTile) {
#pragma unroll
        for (uint32_t w = 0; w < 4; ++w) wcnt[w][tid] = 0;
        __syncthreads();
        uint32_t rank[kRItems];
#pragma unroll
        for (uint32_t k = 0; k < kRItems; ++k) {
            const bool valid = ts + wv * kWaveSpan + k * 64 + lane < b;
            const uint32_t d = (uint32_t)(x[k] >> shift) & 255u;
            uint64_t peers = __ballot(valid);
#pragma unroll
            for (uint32_t bit = 0; bit < 8; ++bit) {
                const uint64_t m = __ballot((d >> bit) & 1u);
                peers &= ((d >> bit) & 1u) ? m : ~m;
            }
            if (valid) {
                const uint32_t before = wcnt[wv][d];
                rank[k] = before + (uint32_t)__popcll(peers & lt);
                if ((peers & lt) == 0) wcnt[wv][d] = before + (uint32_t)__popcll(peers);
            }
        }
        __syncthreads();
        // per digit: the tile's count, every wave's prefix, the digit's place in the tile
        uint32_t c = 0;
#pragma unroll
        for (uint32_t w = 0; w < 4; ++w) {
            const uint32_t cw = wcnt[w][tid];
            wcnt[w][tid] = c;
            c += cw;
        }
        toff[tid] = rs_block_exscan(c, wsum);
        __syncthreads();
#pragma unroll
        for (uint32_t k = 0; k < kRItems; ++k) {
            if (ts + wv * kWaveSpan + k * 64 + lane < b) {
                const uint32_t d = (uint32_t)(x[k] >> shift) & 255u;
                const uint32_t e = toff[d] + wcnt[wv][d] + rank[k];
                skey[e] = x[k];
                sval[e] = v[k];
            }
        }
        if (ts + kRTile < b) load(ts + kRTile);   // the next tile is in flight during the writes
        __syncthreads();
        const uint32_t cnt = (uint32_t)min((uint64_t)kRTile, b - ts);
        for (uint32_t e = tid; e < cnt; e += kRB) {
            const uint64_t key = skey[e];
            const uint32_t d = (uint32_t)(key >> shift) & 255u;
            const uint64_t dest = (uint64_t)run[d] + (e - toff[d]);
            keys_out[dest] = key;
            vals_out[dest] = sval[e];
        }
        __syncthreads();
        run[tid] += c;
    }
}

__global__ void k_rs_adjacent_equal(const uint64_t* __restrict__ k, uint64_t n, uint32_t* __restrict__ flag) {
    bool dup = false;
    for (uint64_t i = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x + 1; i < n;
         i += (uint64_t)gridDim.x * blockDim.x)
        dup |= k[i] == k[i - 1];
    if (dup) atomicOr(flag, 1u);
}

// Level order of the complete binary search tree on n sorted records.  Node i
// (1-based) at depth d = floor(log2 i) would have in-order position
// r = (2(i - 2^d) + 1) 2^(H-d) - 1 in the perfect tree of depth H = floor(log2 n);
// the last level holds only its first L = n - 2^H + 1 leaves, whose perfect
// positions are the even numbers below 2L, so r drops by the missing leaves
// (even positions in [2L, r)).
__global__ void k_eytzinger(const uint64_t* __restrict__ sk, const uint32_t* __restrict__ sv, uint64_t n,
                            uint32_t H, uint64_t L, uint64_t* __restrict__ ek, uint32_t* __restrict__ ev) {
    for (uint64_t i = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x + 1; i <= n;
         i += (uint64_t)gridDim.x * blockDim.x) {
        const uint32_t d = 63u - (uint32_t)__clzll(i);
        const int64_t r = (int64_t)((((i - (1ull << d)) << 1) + 1) << (H - d)) - 1;
        const int64_t gone = r > (int64_t)(2 * L) ? (r - (int64_t)(2 * L) + 1) >> 1 : 0;
        const uint64_t rank = (uint64_t)(r - gone);
        ek[i - 1] = sk[rank];
        ev[i - 1] = sv[rank];
    }
}

// in-order position p of the perfect tree of depth H: its node (1-based, level order)
__device__ __forceinline__ uint64_t node_at(uint64_t p, uint32_t H) {
    const uint32_t z = (uint32_t)__ffsll((long long)(p + 1)) - 1;
    return (1ull << (H - z)) + ((p + 1) >> (z + 1));
}

// the separators of every level, gathered from the keys in layout order
template <bool EYTZ>
__global__ void k_separators(const uint64_t* __restrict__ keys, SepIndex sep, uint64_t* __restrict__ index) {
    for (uint64_t e = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; e < sep.total;
         e += (uint64_t)gridDim.x * blockDim.x) {
        uint32_t l = 1;
        while (l < sep.levels && e >= sep.at[l + 1]) ++l;
        const uint64_t j = e - sep.at[l];
        uint64_t x = ~0ull;
        if (j < sep.count[l]) {
            const uint64_t p = ((j + 1) << (sep.gran + 4 * (l - 1))) - 1;
            x = keys[EYTZ ? node_at(p, sep.depth) - 1 : p];
        }
        index[e] = x;
    }
}

constexpr uint32_t kQ = 4;   // needles per lane in lockstep
constexpr uint32_t kTopLevels = 12;           // Eytzinger levels staged in LDS
constexpr uint32_t kTopNodes = (1u << kTopLevels) - 1;

// Whether each lane searches alone.  Kernel, alone and by lines: 2^22 needles over 16, 256 and 1024 keys
// in order 27 and 56 us, 54 and 60, 68 and 62; 2^20 over 64 and 256 keys 12.9 and 16.0, 17.0 and 16.0; 2^18 over
// 64 7.4 and 7.5.  In Eytzinger order 2^22 over 16, 4096, 16384 and 32768 keys 26 and 45, 44 and 53, 70 and 77,
// 87 and 76; 2^20 9.5 and 12.4, 14.2 and 17.0, 20.6 and 21.6, 25.0 and 22.8; 2^18 over 4096 10.6 and 8.1.
static bool search_alone(uint64_t n, uint64_t m, bool eytz) {
    return m >= (eytz ? 1u << 20 : 1u << 19) && n <= (eytz ? 1u << 14 : 1u << 8);
}

template <bool WANT_VALS>
__global__ __launch_bounds__(256) void k_bsearch(const uint64_t* __restrict__ sk, const uint32_t* __restrict__ sv,
                                                   uint64_t n, const uint64_t* __restrict__ q, uint64_t m,
                                                   uint32_t* __restrict__ out_vals, uint8_t* __restrict__ out_found,
                                                   uint32_t missing) {
    const uint64_t stride = (uint64_t)gridDim.x * blockDim.x * kQ;
    for (uint64_t j0 = ((uint64_t)blockIdx.x * blockDim.x + threadIdx.x) * kQ; j0 < m; j0 += stride) {
        uint64_t x[kQ], lo[kQ];
#pragma unroll
        for (uint32_t u = 0; u < kQ; ++u) {
            x[u] = j0 + u < m ? q[j0 + u] : 0;
            lo[u] = 0;
        }
        // the lower bound stays in [lo, lo + len]; len shrinks the same way for every needle
        uint64_t len = n;
        while (len > 1) {
            const uint64_t half = len >> 1;
#pragma unroll
            for (uint32_t u = 0; u < kQ; ++u) lo[u] = sk[lo[u] + half] < x[u] ? lo[u] + half : lo[u];
            len -= half;
        }
#pragma unroll
        for (uint32_t u = 0; u < kQ; ++u) {
            if (j0 + u >= m) break;
            // the lower bound is lo or lo + 1
            uint64_t pos = lo[u];
            bool hit = false;
            if (n) {
                const uint64_t kk = sk[pos];
                if (kk < x[u]) {
                    ++pos;
                    hit = pos < n && sk[pos] == x[u];
                } else {
                    hit = kk == x[u];
                }
            }
            out_found[j0 + u] = hit;
            if (WANT_VALS) out_vals[j0 + u] = hit ? sv[pos] : missing;
        }
    }
}

template <bool WANT_VALS>
__global__ __launch_bounds__(256) void k_eytz_search(const uint64_t* __restrict__ ek,
                                                       const uint32_t* __restrict__ ev, uint64_t n,
                                                       const uint64_t* __restrict__ q, uint64_t m,
                                                       uint32_t* __restrict__ out_vals,
                                                       uint8_t* __restrict__ out_found, uint32_t missing) {
    __shared__ uint64_t top[kTopNodes];
    const uint64_t ntop = min(n, (uint64_t)kTopNodes);
    for (uint32_t i = threadIdx.x; i < ntop; i += blockDim.x) top[i] = ek[i];
    __syncthreads();
    const uint64_t stride = (uint64_t)gridDim.x * blockDim.x * kQ;
    for (uint64_t j0 = ((uint64_t)blockIdx.x * blockDim.x + threadIdx.x) * kQ; j0 < m; j0 += stride) {
        uint64_t x[kQ], i[kQ];
#pragma unroll
        for (uint32_t u = 0; u < kQ; ++u) {
            x[u] = j0 + u < m ? q[j0 + u] : 0;
            i[u] = 1;
        }
        // descend: a right turn appends a 1 to the node number, a left turn a 0
        for (uint32_t lvl = 0; lvl < kTopLevels; ++lvl) {
#pragma unroll
            for (uint32_t u = 0; u < kQ; ++u)
                if (i[u] <= ntop) i[u] = 2 * i[u] + (top[i[u] - 1] < x[u] ? 1 : 0);
        }
        bool more = true;
        while (more) {
            more = false;
#pragma unroll
            for (uint32_t u = 0; u < kQ; ++u)
                if (i[u] <= n) {
                    i[u] = 2 * i[u] + (ek[i[u] - 1] < x[u] ? 1 : 0);
                    more = true;
                }
        }
#pragma unroll
        for (uint32_t u = 0; u < kQ; ++u) {
            if (j0 + u >= m) break;
            // the lower bound is the node of the last left turn (0: none)
            const uint64_t lb = i[u] >> (__ffsll((long long)~i[u]));
            const bool hit = lb != 0 && ek[lb - 1] == x[u];
            out_found[j0 + u] = hit;
            if (WANT_VALS) out_vals[j0 + u] = hit ? ev[lb - 1] : missing;
        }
    }
}

constexpr uint32_t kSBlock = 512;
constexpr int kSortAgain = 1;   // inside this file: the sample sort gave up

// sums over the eight lanes of a group, in every lane (all lanes active)
__device__ __forceinline__ uint32_t sum8(uint32_t v) {
    v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0xB1, 0xF, 0xF, false);    // lanes 1,0,3,2 of each four
    v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x4E, 0xF, 0xF, false);    // lanes 2,3,0,1
    v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x141, 0xF, 0xF, false);   // mirrored within eight lanes
    return v;
}

// the two entries of a line that lane `at` of its eight holds
struct Two {
    uint64_t a, b;
};

// The rest of a needle's search, once its place on one level of the separators is known: jm of the lane's
// own needle xm among the separators of `level`, x the needles of the lane's eight.  Returns whether the needle is a key, and its
// place.  All lanes of the wave take part.
template <bool EYTZ>
__device__ __forceinline__ bool sep_descend(const uint64_t* __restrict__ keys, uint64_t n,
                                            const uint64_t* __restrict__ index, const SepIndex& sep,
                                            uint32_t level, uint64_t xm, uint32_t jm, const uint64_t (&x)[8], uint64_t& at) {
    const uint32_t lane = threadIdx.x & 63u, l8 = lane & 7u, g8 = lane & 56u;
    uint32_t j[8];
#pragma unroll
    for (uint32_t s = 0; s < 8; ++s) j[s] = (uint32_t)__shfl((int)jm, (int)(g8 + s), 64);
    // counts of entries below the needles, four needles to a word
    auto count = [&](const Two (&e)[8]) {
#pragma unroll
        for (uint32_t h = 0; h < 8; h += 4) {
            uint32_t c = 0;
#pragma unroll
            for (uint32_t s = 0; s < 4; ++s)
                c += ((e[h + s].a < x[h + s] ? 1u : 0u) + (e[h + s].b < x[h + s] ? 1u : 0u)) << (8 * s);
            c = sum8(c);
#pragma unroll
            for (uint32_t s = 0; s < 4; ++s) j[h + s] = (j[h + s] << 4) + ((c >> (8 * s)) & 31u);
        }
    };
    for (uint32_t l = level - 1; l >= 1; --l) {
        const uint64_t* line = index + sep.at[l] + 2 * l8;
        Two e[8];
#pragma unroll
        for (uint32_t s = 0; s < 8; ++s) e[s] = *reinterpret_cast<const Two*>(line + ((uint64_t)j[s] << 4));
        count(e);
    }
    if (EYTZ) {
        // each lane's own needle down the tree below the separators: a right turn appends a 1 to
        // the node number, a left turn a 0; the lower bound is the node of the last left turn
        uint32_t jo = j[0];
#pragma unroll
        for (uint32_t s = 1; s < 8; ++s) jo = l8 == s ? j[s] : jo;
        uint64_t i = sep.first_node + jo, last = 0;
        bool left = false;
#pragma unroll
        for (uint32_t d = 0; d < kEytzGran; ++d) {
            if (i <= n) {
                const uint64_t k = keys[i - 1];
                const bool right = k < xm;
                if (!right) {
                    left = true;
                    last = k;
                }
                i = 2 * i + (right ? 1 : 0);
            }
        }
        const uint64_t lb = i >> __ffsll((long long)~i);   // 0: none
        if (!left && lb != 0) last = keys[lb - 1];         // a separator
        at = lb - 1;
        return lb != 0 && last == xm;
    }
    Two e[8];
#pragma unroll
    for (uint32_t s = 0; s < 8; ++s) {
        const uint64_t k = ((uint64_t)j[s] << 4) + 2 * l8;
        if (k + 1 < n) e[s] = *reinterpret_cast<const Two*>(keys + k);
        else e[s] = Two{k < n ? keys[k] : ~0ull, ~0ull};
    }
    // the line holds the lower bound, when a key equals the needle (entries past n are all
    // ones, and the needle of all ones is told by its position)
    uint32_t eq[2] = {0, 0};
#pragma unroll
    for (uint32_t s = 0; s < 8; ++s) eq[s >> 2] += (e[s].a == x[s] || e[s].b == x[s] ? 1u : 0u) << (8 * (s & 3));
    count(e);
    eq[0] = sum8(eq[0]);
    eq[1] = sum8(eq[1]);
    uint32_t jo = j[0], eo = eq[0] & 255u;
#pragma unroll
    for (uint32_t s = 1; s < 8; ++s) {
        jo = l8 == s ? j[s] : jo;
        eo = l8 == s ? (eq[s >> 2] >> (8 * (s & 3))) & 255u : eo;
    }
    at = jo;
    return eo != 0 && at < n;
}

// Every needle's lower bound.  The search is bound by 128-byte lines from beyond L1 (about 52 G/s
// from HBM, up to 270 G/s from L2), so a line is read once, whole, by eight lanes, which count its
// entries below the needle: lane l of a group answers needle l of the group, and for the lines all
// eight lanes work on the group's eight needles in turn, with eight lines in flight.  (With a lane
// per needle and four dependent reads in each line, the lines left the 32 KiB L1 between the reads:
// 2.19 ms for 2^24 needles and keys; a binary search over the bare array, 22 lines per needle,
// 3.93 ms.)
template <bool EYTZ, bool WANT_VALS>
__global__ __launch_bounds__(kSBlock) __attribute__((amdgpu_waves_per_eu(6))) void k_sep_search(
    const uint64_t* __restrict__ keys, const uint32_t* __restrict__ vals, uint64_t n,
    const uint64_t* __restrict__ index, SepIndex sep, const uint64_t* __restrict__ q, uint64_t m,
    uint32_t* __restrict__ out_vals, uint8_t* __restrict__ out_found, uint32_t missing) {
    __shared__ uint64_t top[kTopSeps + 1];
    const uint32_t ntop = (uint32_t)sep.count[sep.levels];
    uint32_t step0 = 1;   // smallest power of two above ntop
    while (step0 <= ntop) step0 <<= 1;
    {
        const uint64_t* src = index + sep.at[sep.levels];
        for (uint32_t i = threadIdx.x; i < step0; i += kSBlock) top[i] = i < ntop ? src[i] : ~0ull;
    }
    __syncthreads();
    const uint32_t lane = threadIdx.x & 63u, g8 = lane & 56u;
    const uint64_t wave = ((uint64_t)blockIdx.x * kSBlock + threadIdx.x) >> 6, waves = (uint64_t)gridDim.x * (kSBlock / 64);
    for (uint64_t i0 = wave * 64; i0 < m; i0 += waves * 64) {   // the same for all lanes of a wave
        const uint64_t mine = i0 + lane;
        const uint64_t xm = mine < m ? q[mine] : 0;
        uint64_t x[8];
#pragma unroll
        for (uint32_t s = 0; s < 8; ++s) x[s] = i0 + g8 + s < m ? q[i0 + g8 + s] : 0;
        uint32_t jm = 0;
        for (uint32_t st = step0 >> 1; st; st >>= 1) jm += top[jm + st - 1] < xm ? st : 0u;
        uint64_t at;
        const bool hit = sep_descend<EYTZ>(keys, n, index, sep, sep.levels, xm, jm, x, at);
        if (mine < m) {
            if (WANT_VALS) __builtin_nontemporal_store(hit ? vals[at] : missing, out_vals + mine);
            __builtin_nontemporal_store((uint8_t)hit, out_found + mine);
        }
    }
}

// ---- ordered search (ordered.hpp) -------------------------------------------------------------

// Part b takes the needles above top separator part_start(b) - 1 (part 0: all) and not above
// separator part_start(b + 1) - 1 (the last part: all): the stretches of top separators, and of
// the entries below them, that their searches can end in are the parts'.
__host__ __device__ inline uint32_t part_start(uint32_t b, uint32_t ntop, uint32_t bins) {
    return (uint32_t)((uint64_t)b * (ntop + 1) / bins);
}

struct SepPart {
    static constexpr uint32_t kLds = 256;
    const uint64_t* top;
    uint32_t ntop, bins;   // bins <= kLds, bins <= ntop
    __device__ void setup(uint64_t* cut) const {
        if (threadIdx.x < kLds)
            cut[threadIdx.x] = threadIdx.x + 1 < bins ? top[part_start(threadIdx.x + 1, ntop, bins) - 1] : ~0ull;
    }
    __device__ uint32_t of(const uint64_t* cut, uint64_t x, uint32_t) const {
        uint32_t b = 0;
#pragma unroll
        for (uint32_t st = kLds / 2; st; st >>= 1) b += cut[b + st - 1] < x ? st : 0u;
        return b;
    }
};

// Needles grouped by part: every line of the index and of the keys comes from beyond L2 about
// once, and the lowest level whose stretch for the part has at most kStretch entries is searched
// in LDS.  2^24 needles and keys: 437 us (780 us in the needles' order); 10^7 in Eytzinger order 243
// (775).  Bound by the chain of dependent reads at full occupancy: neither VALU, LDS nor L2 is busy
// a third of the time.  Stretches of 4096 entries 477 and 245 us, of 256 437 and 271; workgroups
// of 1024 threads 457 and 271, of 256 453 and 285.
constexpr uint32_t kSepBlock = 512, kStretch = 1024;
template <bool EYTZ>
__global__ __launch_bounds__(kSepBlock) void k_ord_sep(const uint64_t* __restrict__ keys,
                                                     const uint32_t* __restrict__ vals, uint64_t n,
                                                     const uint64_t* __restrict__ index, SepIndex sep, uint32_t level,
                                                     OrdArgs o, uint32_t missing) {
    __shared__ uint64_t cut[kTopSeps + 1];   // at most kStretch of them for a part
    __shared__ OrdRuns R;
    if (ord_idle(o)) return;   // the whole block
    uint32_t part;
    OrdSide side;
    const uint32_t total = ord_runs(o, R, side, part);
    if (side.begin == total) return;   // the whole block
    const uint32_t ntop = (uint32_t)sep.count[sep.levels], up = 4 * (sep.levels - level);
    // the part's stretch of `level`, or all of the top level for needles of any part
    uint32_t c0 = part_start(part, ntop, o.bins) << up;
    uint32_t c1 = (uint32_t)min((uint64_t)part_start(part + 1, ntop, o.bins) << up, sep.count[level] + 1) - 1;
    if (side.all_parts) {
        level = sep.levels;
        c0 = 0;
        c1 = ntop;
    }
    uint32_t step0 = 1;   // smallest power of two above the stretch's length
    while (step0 <= c1 - c0) step0 <<= 1;
    for (uint32_t i = threadIdx.x; i < step0; i += kSepBlock)
        cut[i] = i < c1 - c0 ? index[sep.at[level] + c0 + i] : ~0ull;
    __syncthreads();
    const uint32_t g8 = threadIdx.x & 56u;
    // the same for all lanes of a wave
    for (uint32_t i0 = side.begin + (threadIdx.x & ~63u); i0 < total; i0 += kSepBlock) {
        const uint32_t mine = i0 + (threadIdx.x & 63u);
        const uint64_t place = mine < total ? ord_place(R, mine) : 0;
        const uint64_t xm = mine < total ? side.x[place] : 0;
        uint64_t x[8];
#pragma unroll
        for (uint32_t s = 0; s < 8; ++s) x[s] = (uint64_t)__shfl((unsigned long long)xm, (int)(g8 + s), 64);
        uint32_t jm = 0;
        for (uint32_t st = step0 >> 1; st; st >>= 1) jm += cut[jm + st - 1] < xm ? st : 0u;
        uint64_t at;
        const bool hit = sep_descend<EYTZ>(keys, n, index, sep, level, xm, c0 + jm, x, at);
        if (mine < total) {
            if (side.val) ((uint32_t*)side.val)[place] = hit ? vals[at] : missing;
            side.found[place] = (uint8_t)hit;
        }
    }
}

__global__ void k_none_found(uint64_t m, uint32_t* __restrict__ vals, uint8_t* __restrict__ found, uint32_t missing) {
    for (uint64_t i = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; i < m; i += (uint64_t)gridDim.x * blockDim.x) {
        if (vals) vals[i] = missing;
        found[i] = 0;
    }
}

// levels of separators over n keys: up to the first that fits the LDS
static SepIndex sep_layout(uint64_t n, bool eytz) {
    SepIndex s{};
    s.gran = eytz ? kEytzGran : kSortedGran;
    uint64_t below = n, group = 1ull << s.gran;   // entries that the next level parts, and a group of them
    if (eytz) {
        while ((2ull << s.depth) <= n) ++s.depth;
        below = (2ull << s.depth) - 1;
        s.first_node = 1ull << (s.depth + 1 > s.gran ? s.depth + 1 - s.gran : 0);
    }
    do {
        below = (below + group - 1) / group - 1;
        group = 16;
        s.count[++s.levels] = below;
    } while (below > kTopSeps);
    for (uint32_t l = 1; l <= s.levels; ++l) {
        s.at[l] = s.total;
        // the lines of a level: one more than the separators that part them
        s.total += l < s.levels ? 16 * (s.count[l + 1] + 1) : (s.count[l] + 16) & ~15ull;
    }
    return s;
}

static unsigned sgrid(uint64_t items, uint64_t per_block, unsigned cap) {
    uint64_t g = (items + per_block - 1) / per_block;
    return (unsigned)(g < 1 ? 1 : g > cap ? cap : g);
}

// The whole lookup in the map's order; false: not worth it, no scratch, or a map in a caller's memory.
static bool ordered_search(const fks_sorted* S, const uint64_t* q, uint64_t m, uint32_t* vals, uint8_t* found,
                           uint32_t missing, hipStream_t st) {
    const uint32_t bins = ord_parts(m, 12 * S->n), ntop = (uint32_t)S->sep.count[S->sep.levels];
    if (bins == 0 || bins > SepPart::kLds || bins > ntop || S->has_alloc) return false;
    const uint64_t slice = std::min<uint64_t>(m, kOrdSlice);
    OrdScratch s(slice, bins, false, vals ? 4 : 0, true, st);
    if (!s) return false;
    const SepPart part{S->index + S->sep.at[S->sep.levels], ntop, bins};
    // the lowest level whose stretch for a part fits the LDS
    uint32_t level = S->sep.levels;
    while (level > 1 && ((ntop + bins) / bins << 4 * (S->sep.levels - level + 1)) <= kStretch) --level;
    for (uint64_t at = 0; at < m; at += slice) {
        const OrdArgs a = s.part(std::min(slice, m - at), q + at, nullptr, vals ? vals + at : nullptr, found + at);
        ord_group<SepPart, false>(part, a, st);
        auto launch = [&](auto kernel) {
            FKS_TIMED("fks_order_search", st,
                      hipLaunchKernelGGL(kernel, ord_grid(a), kSepBlock, 0, st, S->keys, S->vals, S->n, S->index,
                                         S->sep, level, a, missing));
        };
        if (S->layout == 1) launch(k_ord_sep<true>);
        else launch(k_ord_sep<false>);
        ord_return<uint32_t, false>(a, st);
    }
    return true;
}

static void separators(const fks_sorted* S, hipStream_t st) {
    const unsigned grid = sgrid(S->sep.total, 256, 8192);
    if (S->layout == 1)
        hipLaunchKernelGGL(k_separators<true>, grid, 256, 0, st, S->keys, S->sep, S->index);
    else
        hipLaunchKernelGGL(k_separators<false>, grid, 256, 0, st, S->keys, S->sep, S->index);
}

// The map by sample sort: everything is queued before the one wait for the outcome.
// kSortAgain: sort another way (a region overflowed, or there is no memory for the regions).
static int build_sampled(fks_sorted* S, const uint64_t* d_keys, const uint32_t* d_vals, hipStream_t st) {
    const uint64_t n = S->n;
    SortFlags* host = (SortFlags*)pinned_words();
    void* scratch = dev_alloc(sample_sort_scratch(n), st);
    SortFlags* flags = (SortFlags*)dev_alloc(sizeof(SortFlags), st);
    S->keys = (uint64_t*)dev_alloc(8 * n, st, kKept);
    S->vals = (uint32_t*)dev_alloc(4 * n, st, kKept);
    S->index = (uint64_t*)dev_alloc(8 * S->sep.total, st, kKept);
    int rc = host && scratch && flags && S->keys && S->vals && S->index ? FKS_OK : kSortAgain;
    bool settled = false;
    if (rc == FKS_OK) {
        sample_sort(d_keys, d_vals, n, S->layout == 1, S->keys, S->vals, S->sep, S->index, flags, scratch, st);
        hipError_t e = hipGetLastError();
        if (e == hipSuccess) e = words_to_host(host, flags, sizeof(SortFlags), st);
        settled = e == hipSuccess;
        if (e != hipSuccess) rc = hip_fail(e);
        else if (host->overflow) rc = kSortAgain;
        else if (host->dup) rc = FKS_EDUPKEY;
    }
    dev_free(scratch, st, settled);
    dev_free(flags, st, settled);
    if (rc != FKS_OK) {
        dev_free(S->keys, st, settled);
        dev_free(S->vals, st, settled);
        dev_free(S->index, st, settled);
        S->keys = S->index = nullptr;
        S->vals = nullptr;
    }
    return rc;
}

// The map by radix sort.
static int build_radix(fks_sorted* S, const uint64_t* d_keys, const uint32_t* d_vals, hipStream_t st) {
    const uint64_t n = S->n;
    const uint32_t layout = S->layout;
    const uint32_t W = (uint32_t)std::min<uint64_t>(4096, std::max<uint64_t>(1, n / (4 * (uint64_t)kRTile)));
    const uint64_t N = 256ull * W;
    uint64_t* kb[2] = {(uint64_t*)dev_alloc(8 * n, st, kKept), (uint64_t*)dev_alloc(8 * n, st, kKept)};   // a pair is kept
    uint32_t* vb[2] = {(uint32_t*)dev_alloc(4 * n, st, kKept), (uint32_t*)dev_alloc(4 * n, st, kKept)};
    uint32_t* cnt = (uint32_t*)dev_alloc(4 * N, st);
    uint32_t* off = (uint32_t*)dev_alloc(4 * N, st);
    uint32_t* tsum = (uint32_t*)dev_alloc(4 * exscan_tiles(N), st);
    uint64_t* tpre = (uint64_t*)dev_alloc(8 * (exscan_tiles(N) + 1), st);
    uint32_t* flag = (uint32_t*)dev_alloc(64, st);
    uint32_t* hflag = nullptr;
    auto cleanup = [&](bool settled) {
        for (int z = 0; z < 2; ++z) {
            dev_free(kb[z], st, settled);
            dev_free(vb[z], st, settled);
        }
        dev_free(cnt, st, settled);
        dev_free(off, st, settled);
        dev_free(tsum, st, settled);
        dev_free(tpre, st, settled);
        dev_free(flag, st, settled);
        if (hflag) (void)hipHostFree(hflag);
    };
    if (!kb[0] || !kb[1] || !vb[0] || !vb[1] || !cnt || !off || !tsum || !tpre || !flag ||
        hipHostMalloc((void**)&hflag, 4, hipHostMallocDefault) != hipSuccess) {
        cleanup(false);
        return FKS_ENOMEM;
    }
    const uint64_t* kin = d_keys;
    const uint32_t* vin = d_vals;
    int cur = 0;
    for (uint32_t pass = 0; pass < 8; ++pass) {
        const uint32_t shift = 8 * pass;
        FKS_TIMED("fks_sort_count", st, hipLaunchKernelGGL(k_rs_count, W, kRB, 0, st, kin, n, W, shift, cnt));
        exscan_u32(cnt, N, tsum, tpre, off, st);
        FKS_TIMED("fks_sort_scatter", st,
                  hipLaunchKernelGGL(k_rs_scatter, W, kRB, 0, st, kin, vin, n, W, shift, off, kb[cur], vb[cur]));
        kin = kb[cur];
        vin = vb[cur];
        cur ^= 1;
    }
    // kin/vin: the sorted pairs; the other buffer pair is free
    int rc = FKS_OK;
    hipError_t e = hipMemsetAsync(flag, 0, 4, st);
    if (e == hipSuccess) {
        hipLaunchKernelGGL(k_rs_adjacent_equal, sgrid(n, 256, 8192), 256, 0, st, kin, n, flag);
        e = hipGetLastError();
    }
    if (e == hipSuccess) e = hipMemcpyAsync(hflag, flag, 4, hipMemcpyDeviceToHost, st);
    if (e == hipSuccess) e = hipStreamSynchronize(st);
    if (e != hipSuccess) rc = hip_fail(e);
    else if (*hflag) rc = FKS_EDUPKEY;
    if (rc == FKS_OK && layout == 1) {
        uint32_t H = 0;
        while ((2ull << H) <= n) ++H;   // floor(log2 n)
        const uint64_t L = n - ((1ull << H) - 1);
        FKS_TIMED("fks_eytzinger", st,
                  hipLaunchKernelGGL(k_eytzinger, sgrid(n, 256, 65536), 256, 0, st, kin, vin, n, H, L, kb[cur],
                                     vb[cur]));
        kin = kb[cur];
        vin = vb[cur];
        cur ^= 1;
        e = hipGetLastError();
        if (e != hipSuccess) rc = hip_fail(e);
    }
    if (rc != FKS_OK) {
        cleanup(false);
        return rc;
    }
    S->index = (uint64_t*)dev_alloc(8 * S->sep.total, st, kKept);
    if (!S->index) {
        cleanup(false);
        return FKS_ENOMEM;
    }
    // keep the final pair of arrays, release the rest
    S->keys = const_cast<uint64_t*>(kin);
    S->vals = const_cast<uint32_t*>(vin);
    separators(S, st);
    kb[cur ^ 1] = nullptr;
    vb[cur ^ 1] = nullptr;
    e = hipStreamSynchronize(st);
    cleanup(e == hipSuccess);
    if (e != hipSuccess) {
        dev_free(S->keys, st);
        dev_free(S->vals, st);
        dev_free(S->index, st);
        return hip_fail(e);
    }
    return FKS_OK;
}

}  // namespace fks

using namespace fks;

extern "C" int fks_sorted_build_u64(const uint64_t* d_keys, const uint32_t* d_vals, uint64_t n, uint32_t layout,
                                    const fks_allocator* alloc, void* stream, fks_sorted** out) {
    if (!out || (n && (!d_keys || !d_vals)) || n >= (1ull << 32) || layout > 1 || !allocator_ok(alloc))
        return FKS_EINVAL;
    AllocScope scope(alloc);
    hipStream_t st = (hipStream_t)stream;
    fks_sorted* S = new fks_sorted{};
    keep_allocator(alloc, S->alloc, S->has_alloc);
    S->n = n;
    S->layout = layout;
    (void)hipGetDevice(&S->device);
    if (n == 0) {
        *out = S;
        return FKS_OK;
    }
    S->sep = sep_layout(n, layout == 1);
    int rc = kSortAgain;
    if (!alloc && n <= kSampleSortMax) rc = build_sampled(S, d_keys, d_vals, st);
    if (rc == kSortAgain) rc = build_radix(S, d_keys, d_vals, st);
    if (rc != FKS_OK) {
        delete S;
        return rc;
    }
    *out = S;
    return FKS_OK;
}

extern "C" int fks_sorted_lookup_u64(const fks_sorted* S, const uint64_t* d_q, uint64_t m, uint32_t* d_vals_out,
                                     uint8_t* d_found_out, uint32_t missing_value, void* stream) {
    if (!S || (m && (!d_q || !d_found_out))) return FKS_EINVAL;
    if (m == 0) return FKS_OK;
    hipStream_t st = (hipStream_t)stream;
    if (S->n == 0) {
        hipLaunchKernelGGL(k_none_found, sgrid(m, 256, 8192), 256, 0, st, m, d_vals_out, d_found_out, missing_value);
        const hipError_t e = hipGetLastError();
        return e == hipSuccess ? FKS_OK : hip_fail(e);
    }
    if (ordered_search(S, d_q, m, d_vals_out, d_found_out, missing_value, st)) {
        const hipError_t e = hipGetLastError();
        return e == hipSuccess ? FKS_OK : hip_fail(e);
    }
    if (search_alone(S->n, m, S->layout == 1)) {
        auto alone = [&](auto kernel) {
            hipLaunchKernelGGL(kernel, sgrid(m, 256 * kQ, 16384), 256, 0, st, S->keys, S->vals, S->n, d_q, m, d_vals_out,
                               d_found_out, missing_value);
        };
        if (S->layout == 0)
            FKS_TIMED("fks_bsearch_u64", st, d_vals_out ? alone(k_bsearch<true>) : alone(k_bsearch<false>));
        else
            FKS_TIMED("fks_eytzinger_u64", st, d_vals_out ? alone(k_eytz_search<true>) : alone(k_eytz_search<false>));
        const hipError_t e = hipGetLastError();
        return e == hipSuccess ? FKS_OK : hip_fail(e);
    }
    // at most four workgroups per CU, as many as its wave slots hold: each stages the top separators once
    const unsigned grid = sgrid(m, kSBlock, 1024);
    auto launch = [&](auto kernel) {
        hipLaunchKernelGGL(kernel, grid, kSBlock, 0, st, S->keys, S->vals, S->n, S->index, S->sep, d_q, m, d_vals_out,
                           d_found_out, missing_value);
    };
    if (S->layout == 0) {
        FKS_TIMED("fks_bsearch_u64", st,
                  d_vals_out ? launch(k_sep_search<false, true>) : launch(k_sep_search<false, false>));
    } else {
        FKS_TIMED("fks_eytzinger_u64", st,
                  d_vals_out ? launch(k_sep_search<true, true>) : launch(k_sep_search<true, false>));
    }
    const hipError_t e = hipGetLastError();
    return e == hipSuccess ? FKS_OK : hip_fail(e);
}

extern "C" int fks_sorted_export(const fks_sorted* S, uint64_t* h_keys, uint32_t* h_vals) {
    if (!S || (S->n && (!h_keys || !h_vals))) return FKS_EINVAL;
    if (S->n == 0) return FKS_OK;
    hipError_t e = hipMemcpy(h_keys, S->keys, 8 * S->n, hipMemcpyDeviceToHost);
    if (e == hipSuccess) e = hipMemcpy(h_vals, S->vals, 4 * S->n, hipMemcpyDeviceToHost);
    return e == hipSuccess ? FKS_OK : hip_fail(e);
}

extern "C" int fks_sorted_info(const fks_sorted* S, uint64_t* n, uint32_t* layout) {
    if (!S) return FKS_EINVAL;
    if (n) *n = S->n;
    if (layout) *layout = S->layout;
    return FKS_OK;
}

extern "C" void fks_sorted_destroy(fks_sorted* S) {
    if (!S) return;
    int prev = 0;
    (void)hipGetDevice(&prev);
    (void)hipSetDevice(S->device);
    {
        // back where the build took them from; frees are ordered on the null stream,
        // after all work already queued on it
        AllocScope scope(S->has_alloc ? &S->alloc : nullptr);
        dev_free(S->keys, nullptr);
        dev_free(S->vals, nullptr);
        dev_free(S->index, nullptr);
    }
    (void)hipSetDevice(prev);
    delete S;
}
