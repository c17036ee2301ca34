// from_array (Figure 2): the constructor that accepts repeated keys.
//
// The input records (key, value, input index) are moved into partitions by the radix passes
// of partition.hip over a random level-one hash, so that all occurrences of a key lie in one
// partition; one workgroup per pair of partitions then collects its distinct keys in an LDS
// table, where every occurrence lowers the slot's smallest input index with an atomic minimum
// (a repeated key keeps the value of its first occurrence, in whatever order the threads
// arrive), and appends each key's first occurrence to a dense list.  Should keys crowd some pair
// under the hashes tried, one table in device memory, which has no such limit, collects them
// instead.  The list is handed to from_array_nodup, whose table does not depend on the order of its input.
#include <hip/hip_runtime.h>

#include <algorithm>

#include "fks_internal.hpp"
#include "partition.hpp"
#include "prof.hpp"

namespace fks {

constexpr uint64_t kEmpty = ~0ull;            // slot marker; the key ~0 itself is tracked on the side
constexpr uint32_t kDdThreads = 512;
constexpr uint32_t kDdParts = 2;              // partitions per workgroup
constexpr uint32_t kDdSlots = 4096;           // slots of a workgroup's table (about 2048 records without repeats)
constexpr uint32_t kDdHeld = 6;               // records per thread held in registers (3072; two regions hold 2944)
constexpr uint32_t kDdAttempts = 2;           // partition hashes tried before the table in device memory

// what the host reads back
struct DdCtrl {
    uint32_t count;      // distinct keys
    uint32_t full;       // a workgroup's table had no room for its keys
    uint32_t overflow;   // a region of the cursor passes overflowed
    uint32_t side;       // the table in device memory: all ones less the smallest index of the key kEmpty, or 0
};

__global__ void k_dd_clear(DdCtrl* c) {
    if (threadIdx.x == 0) *c = DdCtrl{0, 0, 0, 0};
}

// Distinct keys of partitions kDdParts * blockIdx.x on.  Bound by the LDS atomics' latency and
// by the one device atomic per workgroup that reserves its place in the list: those on one
// address take 11.4 ns each (65536 of them 747 us), which is why a workgroup takes two
// partitions (8192 partitions of 2^23 records: 47 us of atomics instead of 93).  A table in
// device memory with a compare-and-swap per record and a list position per occupied slot took
// 0.83 + 3.0 ms for 2^23 records of 2^22 keys; the two passes and this kernel take 0.2 ms.  Records
// held in registers between the table's two uses: 73 us, read and looked up twice 99.
__global__ __launch_bounds__(kDdThreads) void k_dd_distinct(
    const uint64_t* __restrict__ keys, const uint32_t* __restrict__ vals, const uint32_t* __restrict__ idx,
    const uint64_t* __restrict__ qbeg, const uint64_t* __restrict__ qend, uint64_t qcap, uint32_t Q, Triple H,
    uint64_t* __restrict__ out_keys, uint32_t* __restrict__ out_vals, uint64_t out_cap, DdCtrl* __restrict__ ctrl) {
    __shared__ uint64_t tkey[kDdSlots];
    __shared__ uint32_t tidx[kDdSlots];
    __shared__ uint32_t side;       // smallest index of the key kEmpty
    __shared__ uint32_t distinct, base, put, full;
    const uint32_t tid = threadIdx.x;
    for (uint32_t s = tid; s < kDdSlots; s += kDdThreads) {
        tkey[s] = kEmpty;
        tidx[s] = 0xFFFFFFFFu;
    }
    if (tid == 0) {
        side = 0xFFFFFFFFu;
        distinct = put = full = 0;
    }
    __syncthreads();
    const uint32_t q0 = blockIdx.x * kDdParts, q1 = min(Q, q0 + kDdParts);
    auto slot_of = [&](uint64_t x) { return mshash(H, x) >> (32 - 12); };
    static_assert(kDdSlots == 1u << 12, "the slot hash takes 12 bits");
    uint32_t claimed = 0;
    // the record's slot (kDdSlots: the key kEmpty), which keeps its key's smallest index; false: no room
    auto insert = [&](uint64_t x, uint32_t at, uint32_t& s) {
        if (x == kEmpty) {
            s = kDdSlots;
            if (atomicMin(&side, at) == 0xFFFFFFFFu) ++claimed;
            return true;
        }
        s = slot_of(x);
        for (uint32_t probe = 0; probe < kDdSlots; ++probe) {
            // a slot's key never changes once it is set: read before the swap
            unsigned long long old = tkey[s];
            if (old == kEmpty) {
                old = atomicCAS(reinterpret_cast<unsigned long long*>(&tkey[s]), (unsigned long long)kEmpty,
                                (unsigned long long)x);
                if (old == kEmpty) ++claimed;
            }
            if (old == kEmpty || old == x) {
                atomicMin(&tidx[s], at);
                return true;
            }
            s = (s + 1) & (kDdSlots - 1);
        }
        return false;
    };
    // the place of the workgroup's distinct keys in the list, once all are in the table
    auto reserve = [&]() {
        if (claimed) atomicAdd(&distinct, claimed);
        __syncthreads();
        if (tid == 0) {
            base = 0;
            if (full) atomicOr(&ctrl->full, 1u);
            else if (distinct) base = atomicAdd(&ctrl->count, distinct);
        }
        __syncthreads();
    };
    // the record that is its key's first occurrence goes to the list
    auto emit = [&](uint64_t x, uint32_t at, uint32_t v, uint32_t s) {
        if ((s == kDdSlots ? side : tidx[s]) != at) return;
        const uint64_t pos = (uint64_t)base + atomicAdd(&put, 1u);
        if (pos < out_cap) {
            out_keys[pos] = x;
            out_vals[pos] = v;
        }
    };
    auto end_of = [&](uint32_t q) { return qcap ? min(qend[q], qbeg[q] + qcap) : qend[q]; };
    uint64_t lo[kDdParts];
    uint32_t upto[kDdParts + 1];
    upto[0] = 0;
    bool small = true;
#pragma unroll
    for (uint32_t p = 0; p < kDdParts; ++p) {
        lo[p] = q0 + p < q1 ? qbeg[q0 + p] : 0;
        const uint64_t n = q0 + p < q1 ? end_of(q0 + p) - lo[p] : 0;
        small &= n <= kDdThreads * kDdHeld;
        upto[p + 1] = upto[p] + (uint32_t)n;
    }
    if (small && upto[kDdParts] <= kDdThreads * kDdHeld) {
        // the records stay in registers, with their slots, between the two halves
        uint64_t x[kDdHeld];
        uint32_t at[kDdHeld], v[kDdHeld], slot[kDdHeld];
#pragma unroll
        for (uint32_t k = 0; k < kDdHeld; ++k) {
            const uint32_t j = tid + k * kDdThreads;
            if (j < upto[kDdParts]) {
                uint64_t i = lo[0] + j;
#pragma unroll
                for (uint32_t p = 1; p < kDdParts; ++p)
                    if (j >= upto[p]) i = lo[p] + (j - upto[p]);
                x[k] = keys[i];
                at[k] = idx ? idx[i] : (uint32_t)i;
                v[k] = vals[i];
            }
        }
#pragma unroll
        for (uint32_t k = 0; k < kDdHeld; ++k)
            if (tid + k * kDdThreads < upto[kDdParts] && !insert(x[k], at[k], slot[k])) full = 1;
        reserve();
        if (full) return;   // the whole block: the host tries another hash
#pragma unroll
        for (uint32_t k = 0; k < kDdHeld; ++k)
            if (tid + k * kDdThreads < upto[kDdParts]) emit(x[k], at[k], v[k], slot[k]);
        return;
    }
    // crowded partitions (a key repeated very often): the records are read twice
    for (uint32_t q = q0; q < q1; ++q) {
        const uint64_t hi = end_of(q);
        for (uint64_t i = qbeg[q] + tid; i < hi; i += kDdThreads) {
            uint32_t s;
            if (!insert(keys[i], idx ? idx[i] : (uint32_t)i, s)) full = 1;
        }
    }
    reserve();
    if (full) return;   // the whole block: the host tries another hash
    for (uint32_t q = q0; q < q1; ++q) {
        const uint64_t hi = end_of(q);
        for (uint64_t i = qbeg[q] + tid; i < hi; i += kDdThreads) {
            const uint64_t x = keys[i];
            uint32_t s = kDdSlots;
            if (x != kEmpty)
                for (s = slot_of(x); tkey[s] != x;) s = (s + 1) & (kDdSlots - 1);
            emit(x, idx ? idx[i] : (uint32_t)i, vals[i], s);
        }
    }
}

// The table in device memory: linear probing at a load of at most 1/2, a compare-and-swap per record.
__global__ void k_dd_table(uint64_t* __restrict__ tkey, uint32_t* __restrict__ tidx, uint64_t cap) {
    for (uint64_t i = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; i < cap; i += (uint64_t)gridDim.x * blockDim.x) {
        tkey[i] = kEmpty;
        tidx[i] = 0xFFFFFFFFu;
    }
}
__global__ void k_dd_insert(const uint64_t* __restrict__ keys, uint64_t u, uint64_t* __restrict__ tkey,
                            uint32_t* __restrict__ tidx, uint64_t mask, DdCtrl* __restrict__ ctrl) {
    for (uint64_t i = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; i < u; i += (uint64_t)gridDim.x * blockDim.x) {
        const uint64_t x = keys[i];
        if (x == kEmpty) {
            atomicMax(&ctrl->side, 0xFFFFFFFFu - (uint32_t)i);
            continue;
        }
        uint64_t h = sm_fin(x) & mask;
        for (uint64_t probe = 0; probe <= mask; ++probe) {   // half the slots stay free
            const unsigned long long old = atomicCAS(reinterpret_cast<unsigned long long*>(tkey + h),
                                                     (unsigned long long)kEmpty, (unsigned long long)x);
            if (old == kEmpty || old == x) {
                atomicMin(tidx + h, (uint32_t)i);
                break;
            }
            h = (h + 1) & mask;
        }
    }
}
// the list of the table's keys, a wave's at a time; cap: a multiple of 64
__global__ void k_dd_compact(const uint64_t* __restrict__ tkey, const uint32_t* __restrict__ tidx, uint64_t cap,
                             const uint32_t* __restrict__ vals, uint64_t* __restrict__ out_keys,
                             uint32_t* __restrict__ out_vals, DdCtrl* __restrict__ ctrl) {
    const uint32_t lane = threadIdx.x & 63u;
    auto put = [&](bool have, uint64_t x, uint32_t at) {
        const uint64_t all = __ballot(have);
        uint32_t base = 0;
        if (lane == 0 && all) base = atomicAdd(&ctrl->count, (uint32_t)__popcll(all));
        base = (uint32_t)__builtin_amdgcn_readfirstlane((int)base);
        if (have) {
            const uint32_t pos = base + (uint32_t)__popcll(all & ((1ull << lane) - 1));
            out_keys[pos] = x;
            out_vals[pos] = vals[at];
        }
    };
    for (uint64_t i = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; i < cap; i += (uint64_t)gridDim.x * blockDim.x)
        put(tkey[i] != kEmpty, tkey[i], tidx[i]);
    if (blockIdx.x == 0 && threadIdx.x < 64) put(lane == 0 && ctrl->side, kEmpty, 0xFFFFFFFFu - ctrl->side);
}

// The distinct keys by the table in device memory, and their number.
static int dd_by_table(const uint64_t* d_keys, const uint32_t* d_vals, uint64_t u, uint64_t* dk, uint32_t* dv,
                       DdCtrl* ctrl, DdCtrl* pinned, hipStream_t st) {
    uint64_t cap = 64;
    while (cap < 2 * u) cap <<= 1;
    uint64_t* tkey = (uint64_t*)dev_alloc(8 * cap, st);
    uint32_t* tidx = (uint32_t*)dev_alloc(4 * cap, st);
    int rc = tkey && tidx ? FKS_OK : FKS_ENOMEM;
    if (rc == FKS_OK) {
        auto grid = [](uint64_t items) { return (unsigned)std::min<uint64_t>(65536, (items + 255) / 256); };
        hipLaunchKernelGGL(k_dd_clear, 1, 64, 0, st, ctrl);
        hipLaunchKernelGGL(k_dd_table, grid(cap), 256, 0, st, tkey, tidx, cap);
        FKS_TIMED("fks_dedup_insert", st,
                  hipLaunchKernelGGL(k_dd_insert, grid(u), 256, 0, st, d_keys, u, tkey, tidx, cap - 1, ctrl));
        FKS_TIMED("fks_dedup_compact", st,
                  hipLaunchKernelGGL(k_dd_compact, grid(cap), 256, 0, st, tkey, tidx, cap, d_vals, dk, dv, ctrl));
        hipError_t e = hipGetLastError();
        if (e == hipSuccess) e = words_to_host(pinned, ctrl, sizeof(DdCtrl), st);
        if (e != hipSuccess) rc = hip_fail(e);
    }
    dev_free(tkey, st, rc == FKS_OK);
    dev_free(tidx, st, rc == FKS_OK);
    return rc;
}

}  // namespace fks

using namespace fks;

extern "C" int fks_build_u64_from_array(const uint64_t* d_keys, const uint32_t* d_vals, uint64_t u, uint64_t seed,
                                        const fks_params* params, const fks_allocator* alloc, void* stream,
                                        fks_map** out) {
    if (!out || (u && (!d_keys || !d_vals)) || u >= (1ull << 30) || !allocator_ok(alloc)) return FKS_EINVAL;
    if (u == 0) return fks_build_u64(d_keys, d_vals, 0, seed, params, alloc, stream, out);
    AllocScope scope(alloc);
    hipStream_t st = (hipStream_t)stream;
    const PartPlan plan = part_plan(u, true);
    const bool cursor = plan.passes == 1 || plan.passes == 2;
    const size_t scratch_bytes = part_scratch(plan, u, true, cursor, false, nullptr, nullptr);
    char* scratch = (char*)dev_alloc(scratch_bytes, st);
    uint64_t* dk = (uint64_t*)dev_alloc(8 * u, st);
    uint32_t* dv = (uint32_t*)dev_alloc(4 * u, st);
    DdCtrl* ctrl = (DdCtrl*)dev_alloc(sizeof(DdCtrl), st);
    auto cleanup = [&](bool settled) {
        dev_free(scratch, st, settled);
        dev_free(dk, st, settled);
        dev_free(dv, st, settled);
        dev_free(ctrl, st, settled);
    };
    DdCtrl* const pinned = (DdCtrl*)pinned_words();
    if (!scratch || !dk || !dv || !ctrl || !pinned) {
        cleanup(false);
        return FKS_ENOMEM;
    }
    PartArgs a{};
    part_scratch(plan, u, true, cursor, false, scratch, &a);
    a.n = u;
    a.aux = true;
    a.magic = fastmod_magic((uint32_t)u);
    a.keys = d_keys;
    a.vals = d_vals;
    a.overflow = &ctrl->overflow;
    a.fused = true;   // no size pass: only the partitions' records are wanted
    a.cursor = cursor;
    uint32_t n = 0;
    int rc = FKS_OK;
    bool listed = false;
    for (uint32_t r = 0; r < kDdAttempts; ++r) {
        // partition and slot hashes of a stream of their own (~seed), fresh in every attempt
        a.A = level1_triple(~seed, r);
        const Triple H = level2_triple(~seed, r, 0);
        const bool with_passes = a.cursor || plan.passes == 0;
        a.start = with_passes ? AttemptStart{(uint32_t*)ctrl, sizeof(DdCtrl) / 4, nullptr, 0, 0, 0} : AttemptStart{};
        if (!with_passes) hipLaunchKernelGGL(k_dd_clear, 1, 64, 0, st, ctrl);
        PartOut o;
        if ((rc = part_prepare(a, st, o))) break;
        FKS_TIMED("fks_dedup_distinct", st,
                  hipLaunchKernelGGL(k_dd_distinct, (plan.Q + kDdParts - 1) / kDdParts, kDdThreads, 0, st, o.keys,
                                     o.vals, o.aux_is_pos ? nullptr : o.aux, o.qbeg, o.qend, o.qcap, plan.Q, H, dk,
                                     dv, u, ctrl));
        hipError_t e = hipGetLastError();
        if (e == hipSuccess) e = words_to_host(pinned, ctrl, sizeof(DdCtrl), st);
        if (e != hipSuccess) {
            rc = hip_fail(e);
            break;
        }
        const DdCtrl got = *pinned;
        if (got.overflow) {
            // a key repeated many times crowds its partition's region: the same hash again,
            // with counted passes, whose partitions hold any number of records
            a.cursor = false;
            --r;
            continue;
        }
        if (got.full) continue;   // more distinct keys than slots: another hash
        n = got.count;
        listed = true;
        break;
    }
    dev_free(scratch, st, rc == FKS_OK);
    scratch = nullptr;
    if (rc == FKS_OK && !listed && (rc = dd_by_table(d_keys, d_vals, u, dk, dv, ctrl, pinned, st)) == FKS_OK)
        n = pinned->count;
    if (rc == FKS_OK) rc = fks_build_u64(dk, dv, n, seed, params, alloc, stream, out);
    cleanup(rc == FKS_OK);   // the build has waited for its own last kernel
    return rc;
}
