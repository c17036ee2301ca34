// Batched lookup and membership (Figure 2 lookup; Section 4 operations 2 and 3).
//
// Per needle: j = hash(A) q mod n selects a bucket; probe 1 reads the 16-byte
// record of the bucket's group (slot base, the eight 4-bit sizes, the eight
// trial indices); the bucket's cell is base + sum of the squared sizes before
// it + hash(C[t]) q mod s^2, with the level-two triples C staged in LDS; probe
// 2 reads that cell and compares keys (Section 2.2 membership test).  An empty
// bucket answers "absent" after one probe.  Each thread keeps several needles
// in flight so that their random probes overlap.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <type_traits>

#include "fks_internal.hpp"
#include "ordered.hpp"
#include "prof.hpp"

namespace fks {

constexpr int kLBlock = 256;
constexpr int kQ = 4;   // needles in flight per thread (integer needles: many of them)

__global__ void k_fill_outputs(uint64_t m, uint32_t* __restrict__ vals, uint64_t* __restrict__ vals64,
                               uint8_t* __restrict__ found, uint32_t missing, uint64_t missing64) {
    for (uint64_t i = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; i < m;
         i += (uint64_t)gridDim.x * blockDim.x) {
        if (vals) vals[i] = missing;
        if (vals64) vals64[i] = missing64;
        if (found) found[i] = 0;
    }
}

// V64: 64-bit values, the high half in the cell's aux word
// Q: needles in flight per thread
template <bool WANT_VALS, bool WANT_FOUND, bool V64, int Q>
__global__ __launch_bounds__(kLBlock) void k_lookup_u64(const Group* __restrict__ header,
                                                          const Cell* __restrict__ slots, Triple A,
                                                          uint64_t magic, uint32_t n,
                                                          const Triple* __restrict__ Cg, uint32_t T,
                                                          const uint64_t* __restrict__ q, uint64_t m,
                                                          uint32_t* __restrict__ vals,
                                                          uint8_t* __restrict__ found, uint32_t missing,
                                                          uint64_t* __restrict__ vals64 = nullptr,
                                                          uint64_t missing64 = 0) {
    __shared__ Triple C[kTMax];
    const uint64_t stride = (uint64_t)gridDim.x * kLBlock * Q, first = (uint64_t)blockIdx.x * kLBlock * Q;
    uint64_t x[Q];
    auto load = [&](uint64_t base) {
#pragma unroll
        for (int k = 0; k < Q; ++k) {
            const uint64_t i = base + threadIdx.x + (uint64_t)k * kLBlock;
            x[k] = i < m ? __builtin_nontemporal_load(q + i) : 0;   // needles and answers stream
        }
    };
    load(first);   // under way while the triples are staged
    for (uint32_t t = threadIdx.x; t < T; t += kLBlock) C[t] = Cg[t];
    __syncthreads();
    for (uint64_t base = first; base < m; base += stride) {
        if (base != first) load(base);
        Group h[Q];
        uint32_t kk[Q];
#pragma unroll
        for (int k = 0; k < Q; ++k) {
            const uint64_t i = base + threadIdx.x + (uint64_t)k * kLBlock;
            const uint32_t j = fastmod(mshash(A, x[k]), magic, n);
            kk[k] = j & 7u;
            if (i < m) h[k] = header[j >> 3];
            else h[k] = Group{0, 0, 0, 0};
        }
        Cell c[Q];
        uint32_t s[Q];
#pragma unroll
        for (int k = 0; k < Q; ++k) {
            uint32_t p;
            s[k] = cell_of(h[k], kk[k], C, x[k], p) ? 1u : 0u;
            // read once per needle: a streaming load, so that the cells do not push the group
            // records out of the caches
            c[k] = s[k] ? load_cell_once(slots + p) : Cell{~x[k], 0, 0};
        }
#pragma unroll
        for (int k = 0; k < Q; ++k) {
            const uint64_t i = base + threadIdx.x + (uint64_t)k * kLBlock;
            if (i < m) {
                const bool hit = s[k] && c[k].key == x[k];
                if (WANT_VALS && V64)
                    __builtin_nontemporal_store(hit ? ((uint64_t)c[k].aux << 32) | c[k].val : missing64, vals64 + i);
                if (WANT_VALS && !V64) __builtin_nontemporal_store(hit ? c[k].val : missing, vals + i);
                if (WANT_FOUND) __builtin_nontemporal_store((uint8_t)(hit ? 1 : 0), found + i);
            }
        }
    }
}

// ---- ordered lookups (ordered.hpp) ----------------------------------------------------------

OrdScratch::OrdScratch(uint64_t m, uint32_t bins, bool ids, uint32_t val_bytes, bool found, hipStream_t s, size_t more)
    : st_(s) {
    hipStreamCaptureStatus cap = hipStreamCaptureStatusNone;
    if (s != nullptr && hipStreamIsCapturing(s, &cap) != hipSuccess) {
        (void)hipGetLastError();
        return;
    }
    if (cap != hipStreamCaptureStatusNone) return;
    a_.tile = ord_tile(m, ids);
    a_.bins = bins;
    const size_t tiles = (m + a_.tile - 1) / a_.tile;
    size_t total = 0;
    auto carve = [&](size_t bytes) {
        const size_t at = total;
        total += (bytes + 255) & ~(size_t)255;
        return at;
    };
    const size_t x = carve(8 * m), id = carve(ids ? 4 * m : 0), slot = carve(2 * m),
                 start = carve(2 * tiles * (bins + 2)), val = carve((size_t)val_bytes * m),
                 fnd = carve(found ? m : 0), own = carve(more);
    base_ = pool_take(total, s, kTry);
    if (!base_) return;
    char* p = (char*)base_;
    a_.x = (uint64_t*)(p + x);
    a_.id = (uint32_t*)(p + id);
    a_.slot = (uint16_t*)(p + slot);
    a_.start = (uint16_t*)(p + start);
    a_.val = val_bytes ? p + val : nullptr;
    more_ = p + own;
    a_.found = found ? (uint8_t*)(p + fnd) : nullptr;
}

OrdScratch::~OrdScratch() {
    if (base_) pool_give(base_, st_, false, kTry);
}

// Needles in their own order against ordered, 50 % hits: over 4 * 10^6 keys 52 and 58 us for 2^21
// needles, 98 and 88 us for 2^22, 370 and 278 us for 2^24; 2^22 needles over 2^21 keys 84 and
// 83 us, over 2^25 keys 135 and 145 us (half the table's lines are not needed at all); 2^23 needles
// over 2^18 keys 138 and 126 us, over 2^25 keys 264 and 248 us.  The three launches and the table's one pass
// have to be paid back by 10-15 ps per needle.
uint32_t ord_parts(uint64_t m, uint64_t table_bytes) {
    constexpr uint32_t kParts = 256;
    if (m >= (1u << 23)) return table_bytes >= (8u << 20) && table_bytes / 136 <= m ? kParts : 0;
    return m >= (1u << 22) && table_bytes >= (128u << 20) && table_bytes / 68 <= m ? kParts : 0;
}

// part of the table that answers an integer needle: equal ranges of buckets
struct BucketPart {
    static constexpr uint32_t kLds = 0;
    Triple A;
    uint64_t magic;
    uint32_t n;
    uint32_t scale;   // floor(2^32 parts / n) with n > parts: parts come out below their number
    __device__ void setup(uint64_t*) const {}
    __device__ uint32_t of(const uint64_t*, uint64_t x, uint32_t) const {
        return __umulhi(fastmod(mshash(A, x), magic, n), scale);
    }
};

// Needles grouped by part, answered at their places.  Bound by the chain of a needle's two dependent
// reads, which the lines that miss L2 (the table once) lengthen: 10^7 needles over as many keys
// take 160 us, 80 of it without the cells and 45 without any table access, where their 1.4 to 2 requests each
// would take 51 to 75 us at the 270 G requests/s of L2.  Workgroups of 1024 threads with two needles each in
// flight keep few parts open at a time: with 256 threads and four needles 181 us; with 128 or
// 512 parts instead of 256 10-20 us more.
template <bool V64>
__global__ __launch_bounds__(kOrdBlock) void k_ord_lookup(const Group* __restrict__ header,
                                                        const Cell* __restrict__ slots, Triple A, uint64_t magic,
                                                        uint32_t n, const Triple* __restrict__ Cg, uint32_t T,
                                                        OrdArgs o, uint64_t missing) {
    __shared__ Triple C[kTMax];
    __shared__ OrdRuns R;
    if (ord_idle(o)) return;   // the whole block
    for (uint32_t t = threadIdx.x; t < T; t += kOrdBlock) C[t] = Cg[t];
    uint32_t part;
    OrdSide side;
    const uint32_t total = ord_runs(o, R, side, part);
    constexpr uint32_t Q = 2;
    for (uint32_t i0 = side.begin; i0 < total; i0 += kOrdBlock * Q) {
        uint64_t x[Q], at[Q];
        Group h[Q];
        uint32_t kk[Q];
#pragma unroll
        for (uint32_t k = 0; k < Q; ++k) {
            const uint32_t i = i0 + threadIdx.x + k * kOrdBlock;
            at[k] = i < total ? ord_place(R, i) : 0;
            x[k] = i < total ? __builtin_nontemporal_load(side.x + at[k]) : 0;
        }
#pragma unroll
        for (uint32_t k = 0; k < Q; ++k) {
            const uint32_t j = fastmod(mshash(A, x[k]), magic, n);
            kk[k] = j & 7u;
            if (i0 + threadIdx.x + k * kOrdBlock < total) h[k] = header[j >> 3];
            else h[k] = Group{0, 0, 0, 0};
        }
        Cell c[Q];
#pragma unroll
        for (uint32_t k = 0; k < Q; ++k) {
            uint32_t p;
            c[k] = cell_of(h[k], kk[k], C, x[k], p) ? slots[p] : Cell{~x[k], 0, 0};
        }
#pragma unroll
        for (uint32_t k = 0; k < Q; ++k) {
            if (i0 + threadIdx.x + k * kOrdBlock < total) {
                const bool hit = c[k].key == x[k];
                if (V64) {
                    if (side.val) ((uint64_t*)side.val)[at[k]] = hit ? ((uint64_t)c[k].aux << 32) | c[k].val : missing;
                } else {
                    if (side.val) ((uint32_t*)side.val)[at[k]] = hit ? c[k].val : (uint32_t)missing;
                }
                if (side.found) side.found[at[k]] = hit ? 1 : 0;
            }
        }
    }
}

// The whole lookup in table order; false: not worth it, no scratch, or a map in a caller's
// memory (whose lookups take none of the library's).
template <bool V64, typename V>
static bool ordered_lookup(const fks_map* map, const uint64_t* q, uint64_t m, V* vals, uint8_t* found, V missing,
                           hipStream_t st) {
    const uint32_t n = (uint32_t)map->n, bins = ord_parts(m, 2 * map->n + 16 * map->S);
    if (bins == 0 || n <= bins || map->has_alloc) return false;
    const uint64_t slice = std::min<uint64_t>(m, kOrdSlice);
    OrdScratch s(slice, bins, false, vals ? sizeof(V) : 0, found != nullptr, st);
    if (!s) return false;
    const BucketPart part{map->A, map->magic_n, n, (uint32_t)(((uint64_t)bins << 32) / n)};
    for (uint64_t at = 0; at < m; at += slice) {
        const OrdArgs a = s.part(std::min(slice, m - at), q + at, nullptr, vals ? vals + at : nullptr,
                                 found ? found + at : nullptr);
        ord_group<BucketPart, false>(part, a, st);
        FKS_TIMED("fks_order_lookup", st,
                  hipLaunchKernelGGL(k_ord_lookup<V64>, ord_grid(a), kOrdBlock, 0, st, map->header, map->slots, map->A,
                                     map->magic_n, n, map->C, map->T, a, (uint64_t)missing));
        ord_return<V, false>(a, st);
    }
    return true;
}

// String needles: fingerprint, probe, then compare the stored bytes on a fingerprint hit.
// The needle and the stored key are read 64 bytes at a time as aligned dwords, so each
// costs one memory round trip; a needle of at most 64 bytes stays in registers for the
// comparison.
template <bool WANT_VALS>
__global__ __launch_bounds__(kLBlock) void k_lookup_bytes(
    const Group* __restrict__ header, const Cell* __restrict__ slots, Triple A, uint64_t beta,
    uint64_t magic, uint32_t n, const Triple* __restrict__ Cg, uint32_t T,
    const int64_t* __restrict__ koff, const uint8_t* __restrict__ kbytes,
    const int64_t* __restrict__ qoff, const uint8_t* __restrict__ qbytes, uint64_t qn, uint64_t m,
    uint32_t* __restrict__ vals, uint8_t* __restrict__ found, uint32_t missing) {
    __shared__ Triple C[kTMax];
    for (uint32_t t = threadIdx.x; t < T; t += kLBlock) C[t] = Cg[t];
    __syncthreads();
    for (uint64_t i = (uint64_t)blockIdx.x * kLBlock + threadIdx.x; i < m;
         i += (uint64_t)gridDim.x * kLBlock) {
        const int64_t a = qoff[i], b = qoff[i + 1];
        if (a < 0 || b < a || (uint64_t)b > qn) {
            // not a range of the needle buffer: nothing is read through it
            if (WANT_VALS) vals[i] = missing;
            if (found) found[i] = 0;
            continue;
        }
        const uint64_t len = (uint64_t)(b - a);
        const uint8_t* s = qbytes + a;
        uint32_t w[kChunkWords];
        const uint64_t y = fingerprint_words(s, len, beta, w);
        const uint32_t j = fastmod(mshash(A, y), magic, n);
        const Group h = header[j >> 3];
        const uint32_t k = j & 7u;
        bool hit = false;
        uint32_t v = missing;
        uint32_t p;
        if (cell_of(h, k, C, y, p)) {
            const Cell c = load_cell_once(slots + p);
            if (c.key == y) {
                const int64_t ka = koff[c.aux], kb = koff[c.aux + 1];
                if ((uint64_t)(kb - ka) == len) {
                    bool eq;
                    if (len <= 4 * kChunkWords) {
                        uint32_t u[kChunkWords];
                        load_words<kChunkWords>(kbytes + ka, (uint32_t)len, u);
                        uint32_t diff = 0;
#pragma unroll
                        for (int q = 0; q < kChunkWords; ++q) diff |= u[q] ^ w[q];
                        eq = diff == 0;
                    } else {
                        eq = bytes_equal(kbytes + ka, s, len);
                    }
                    if (eq) {
                        hit = true;
                        v = c.val;
                    }
                }
            }
        }
        if (WANT_VALS) vals[i] = v;
        if (found) found[i] = hit ? 1 : 0;
    }
}

static unsigned lookup_grid(uint64_t m, uint64_t per_block) {
    uint64_t g = (m + per_block - 1) / per_block;
    if (g < 1) g = 1;
    if (g > 65536) g = 65536;
    return (unsigned)g;
}

// A lookup in the needles' own order.
template <bool V64>
static void launch_lookup(const fks_map* map, const uint64_t* q, uint64_t m, uint32_t* vals, uint64_t* vals64,
                          uint8_t* found, uint32_t missing, uint64_t missing64, hipStream_t st) {
    const bool want_vals = V64 ? vals64 != nullptr : vals != nullptr;
    auto launch = [&](auto kernel, uint64_t needles) {
        FKS_TIMED(V64 ? "fks_lookup_u64_v64" : want_vals ? "fks_lookup_u64" : "fks_contains_u64", st,
                  hipLaunchKernelGGL(kernel, lookup_grid(m, (uint64_t)kLBlock * needles), kLBlock, 0, st, map->header,
                                     map->slots, map->A, map->magic_n, (uint32_t)map->n, map->C, map->T, q, m, vals,
                                     found, missing, vals64, missing64));
    };
    auto with = [&](auto q_) {
        constexpr int Q = decltype(q_)::value;
        if (want_vals && found) launch(k_lookup_u64<true, true, V64, Q>, Q);
        else if (want_vals) launch(k_lookup_u64<true, false, V64, Q>, Q);
        else launch(k_lookup_u64<false, true, V64, Q>, Q);
    };
    // few needles are one thread's chain of dependent reads: one needle each, on as many CUs as there
    // are (kernel over 2^16 keys with one and four needles per thread: 1000 needles 2.5 and 5.0 us,
    // 2^16 3.3 and 6.2, 2^18 5.3 and 7.2, 2^19 8.9 and 8.7, 2^21 over 2^20 keys 38.4 and 37.7)
    if (m <= (1u << 19)) with(std::integral_constant<int, 1>{});
    else with(std::integral_constant<int, kQ>{});
}

}  // namespace fks

using namespace fks;

extern "C" int fks_lookup_u64(const fks_map* map, const uint64_t* d_queries, uint64_t m, uint32_t* d_vals_out,
                              uint8_t* d_found_out, uint32_t missing, void* stream) {
    // 32-bit values from a map with 32-bit values; membership from any integer-key map
    if (!map || (m && !d_queries)) return FKS_EINVAL;
    if (map->kind != 0 && !(map->kind == 2 && !d_vals_out)) return FKS_EINVAL;
    if (m == 0 || (!d_vals_out && !d_found_out)) return FKS_OK;
    hipStream_t st = (hipStream_t)stream;
    if (map->n == 0) {
        FKS_TIMED("fks_fill_outputs", st, hipLaunchKernelGGL(k_fill_outputs, lookup_grid(m, kLBlock), kLBlock, 0, st, m, d_vals_out, nullptr, d_found_out,
                           missing, 0ull));
    } else if (!ordered_lookup<false, uint32_t>(map, d_queries, m, d_vals_out, d_found_out, missing, st)) {
        launch_lookup<false>(map, d_queries, m, d_vals_out, nullptr, d_found_out, missing, 0, st);
    }
    hipError_t e = hipGetLastError();
    return e == hipSuccess ? FKS_OK : hip_fail(e);
}

extern "C" int fks_contains_u64(const fks_map* map, const uint64_t* d_queries, uint64_t m, uint8_t* d_found_out,
                                void* stream) {
    if (!d_found_out && m) return FKS_EINVAL;
    return fks_lookup_u64(map, d_queries, m, nullptr, d_found_out, 0, stream);
}

extern "C" int fks_lookup_u64_v64(const fks_map* map, const uint64_t* d_queries, uint64_t m, uint64_t* d_vals_out,
                                  uint8_t* d_found_out, uint64_t missing, void* stream) {
    if (!map || map->kind != 2 || (m && (!d_queries || !d_vals_out))) return FKS_EINVAL;
    if (m == 0) return FKS_OK;
    hipStream_t st = (hipStream_t)stream;
    if (map->n == 0) {
        FKS_TIMED("fks_fill_outputs", st,
                  hipLaunchKernelGGL(k_fill_outputs, lookup_grid(m, kLBlock), kLBlock, 0, st, m, nullptr, d_vals_out,
                                     d_found_out, 0u, missing));
    } else if (!ordered_lookup<true, uint64_t>(map, d_queries, m, d_vals_out, d_found_out, missing, st)) {
        launch_lookup<true>(map, d_queries, m, nullptr, d_vals_out, d_found_out, 0u, missing, st);
    }
    hipError_t e = hipGetLastError();
    return e == hipSuccess ? FKS_OK : hip_fail(e);
}

static int lookup_bytes_impl(const fks_map* map, const int64_t* d_q_offsets, const uint8_t* d_q_bytes,
                             uint64_t q_nbytes, uint64_t m, uint32_t* d_vals_out, uint8_t* d_found_out,
                             uint32_t missing, void* stream) {
    if (!map || map->kind != 1 || (m && !d_q_offsets) || (q_nbytes && !d_q_bytes)) return FKS_EINVAL;
    if (m == 0 || (!d_vals_out && !d_found_out)) return FKS_OK;
    hipStream_t st = (hipStream_t)stream;
    if (map->n == 0) {
        FKS_TIMED("fks_fill_outputs", st, hipLaunchKernelGGL(k_fill_outputs, lookup_grid(m, kLBlock), kLBlock, 0, st, m, d_vals_out, nullptr, d_found_out,
                           missing, 0ull));
    } else {
        const unsigned grid = lookup_grid(m, (uint64_t)kLBlock * 2);
        if (d_vals_out)
            FKS_TIMED("fks_lookup_bytes", st, hipLaunchKernelGGL(k_lookup_bytes<true>, grid, kLBlock, 0, st, map->header, map->slots, map->A,
                               map->beta, map->magic_n, (uint32_t)map->n, map->C, map->T, map->ctx_off,
                               map->ctx_bytes, d_q_offsets, d_q_bytes, q_nbytes, m, d_vals_out, d_found_out,
                               missing));
        else
            FKS_TIMED("fks_contains_bytes", st, hipLaunchKernelGGL(k_lookup_bytes<false>, grid, kLBlock, 0, st, map->header, map->slots, map->A,
                               map->beta, map->magic_n, (uint32_t)map->n, map->C, map->T, map->ctx_off,
                               map->ctx_bytes, d_q_offsets, d_q_bytes, q_nbytes, m, d_vals_out, d_found_out,
                               missing));
    }
    hipError_t e = hipGetLastError();
    return e == hipSuccess ? FKS_OK : hip_fail(e);
}

extern "C" int fks_lookup_bytes(const fks_map* map, const int64_t* d_q_offsets, const uint8_t* d_q_bytes,
                                uint64_t q_nbytes, uint64_t m, uint32_t* d_vals_out, uint8_t* d_found_out,
                                uint32_t missing, void* stream) {
    return lookup_bytes_impl(map, d_q_offsets, d_q_bytes, q_nbytes, m, d_vals_out, d_found_out, missing, stream);
}

extern "C" int fks_contains_bytes(const fks_map* map, const int64_t* d_q_offsets, const uint8_t* d_q_bytes,
                                  uint64_t q_nbytes, uint64_t m, uint8_t* d_found_out, void* stream) {
    return lookup_bytes_impl(map, d_q_offsets, d_q_bytes, q_nbytes, m, nullptr, d_found_out, 0, stream);
}
