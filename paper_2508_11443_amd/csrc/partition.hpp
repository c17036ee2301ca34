// Partitioned level-one attempt (partition.hip): plan, buffers, entry points.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "fks_internal.hpp"

namespace fks {

constexpr uint32_t kPartBits = 10;                   // 1024 buckets per partition
constexpr uint32_t kPartBuckets = 1u << kPartBits;

// A map of a batch built by the partition passes instead of a single workgroup
// ("wide" map, at most 65536 keys, so at most kSegParts partitions).
constexpr uint32_t kSegParts = 64;
struct WideSeg {
    Triple A;            // level-one triple of attempt 0
    uint64_t magic;      // remainder magic of n
    uint64_t seed;
    uint64_t in_lo, in_hi;   // the map's keys in the batch input
    uint64_t hdr_off;    // first group record of the map in the header pool
    uint64_t slot_off;   // first cell of the map in the cell pool
    uint32_t n, G;       // keys, groups of eight buckets
    uint32_t map;        // index of the map in the batch
    uint32_t c;          // space factor: the attempt fails when the map's cells exceed c*n
    uint32_t part0;      // its first entry in the list of partitions (ceil(n / 1024) of them) ...
    uint32_t tile0, tiles;   // ... and in the list of scatter tiles
};

// Device lists and scratch of wide_build.
struct WideLists {
    uint64_t* keys;      // records, a region per partition
    uint32_t* vals;
    unsigned long long* cursor;   // every partition's end
    uint64_t* state;     // look-back words
    uint64_t* S;         // cells of every map
    uint2* tiles;        // segment, first record within the map
    uint32_t* parts;     // segment * kSegParts + partition within the map
};

// Radix passes over the partition index q (bits_q bits), at most 8 bits (256 bins) each:
// one pass up to 2^8 partitions, two up to 2^16, three beyond (n < 2^30 gives q < 2^20).
struct PartPlan {
    uint32_t Q;        // partitions
    uint32_t bits_q;   // ceil(log2 Q)
    uint32_t passes;   // scatter passes: 0, 1, 2 or 3
    uint32_t shiftA;   // first-level bin = q >> shiftA
    uint32_t binsA;    // first-level bins
    uint32_t bitsB;    // two passes: second-level bin = q & (2^bitsB - 1); three: (q >> bitsC) & 255
    uint32_t binsAB;   // three passes: bins after the second pass (q >> bitsC)
    uint32_t bitsC;    // three passes: third-level bin = q & (2^bitsC - 1)
    uint32_t items;    // records per thread of a cursor pass's tile: 2, 4, or 0 for the largest tile
    uint32_t W1, W2, W3;   // workers of the first pass / per bin of the second and third passes
    uint64_t matrix;   // entries of the largest count matrix
    // two passes with cursors: capacity of a first-level region and of a partition's; first-level
    // regions, 2^subs of them (one for each XCD, or one) in a bin
    uint64_t cap1, capQ;
    uint32_t regions1, subs;
    uint32_t W2c;           // workers per first-level region
};

// What an attempt's set-up does beside the passes' own (nothing when zero): clears the first
// `words` (at most 256) words at `clear` and writes the T level-two triples of attempt r.
struct AttemptStart {
    uint32_t* clear;
    uint32_t words;
    Triple* C;
    uint64_t seed;
    uint32_t r, T;
};

// Inputs, scratch and outputs of one attempt (device pointers).
struct PartArgs {
    AttemptStart start;         // taken by the passes with cursors and by inputs without passes
    uint64_t n, G;
    bool aux;                   // an aux word travels with every key
    bool str;                   // keys are string fingerprints
    const uint32_t* aux_in;     // the input's aux words, or nullptr for the key index
    const uint64_t* pairs;      // passes with cursors: values and aux words as the halves of 64-bit words, or nullptr
    Triple A;
    uint64_t magic;
    const uint64_t* keys;       // the integers the construction hashes
    const uint32_t* vals;
    // scratch
    uint64_t *k1, *k2;          // partitioned keys after pass 1 / pass 2
    uint32_t *v1, *v2;          // values
    uint32_t *a1, *a2;          // string indices (string maps)
    uint32_t* cnt;              // per-worker bin counts (plan.matrix entries)
    uint32_t* off;              // their exclusive scan
    uint32_t* tsum;             // scan tile sums
    uint64_t* tpre;             // scanned tile sums
    uint64_t* offA;             // 257 first-level bin offsets
    uint64_t* offAB;            // three passes: binsAB+1 second-level bin offsets
    uint64_t* offQ;             // Q+1 partition offsets
    uint32_t* sqQ;              // Q sums of squared sizes
    uint64_t* cbase;            // Q+1 cell bases
    uint32_t* sizes;            // G size words (the headers' second word)
    uint64_t* S_dev;            // total cells
    uint32_t* oversize;         // a bucket above 15 keys
    uint32_t* outcome;          // pinned: where the host reads start.clear's words, or null
    uint32_t* done;             // one of those words, counting the final pass's workgroups
    bool fused;                 // the final pass sizes the partitions itself (no size pass and scan)
    // two passes without count passes: each tile reserves its runs on per-bin cursors in
    // fixed-capacity regions (k1/v1/a1 hold binsA * cap1 records, k2/v2/a2 Q * capQ)
    bool cursor;
    unsigned long long* cur1;   // binsA first-level cursors
    unsigned long long* cur2;   // Q partition cursors: each partition's end
    uint64_t* begA;             // binsA region starts
    uint64_t* begQ;             // Q partition starts
    uint32_t* overflow;         // a region overflowed: the attempt is redone with counts
};

struct PartOut {
    PartPlan plan;
    const uint64_t* keys;       // records in partition order
    const uint32_t* vals;
    const uint32_t* aux;
    int aux_is_pos;
    const uint64_t* qbeg;       // partition q's records are [qbeg[q], min(qend[q], qbeg[q] + qcap))
    const uint64_t* qend;
    uint64_t qcap;              // 0: no cap (counted passes)
    bool reported;              // the final pass writes the outcome to the host itself
    bool prezeroed;             // the fused pass's look-back words are already zero
};

// Exclusive prefix sum of N u32 counts whose total is below 2^32 (three launches):
// tsum holds exscan_tiles(N) words and tpre exscan_tiles(N) + 1 words of scratch.
uint64_t exscan_tiles(uint64_t N);
void exscan_u32(const uint32_t* in, uint64_t N, uint32_t* tsum, uint64_t* tpre, uint32_t* out, hipStream_t st);

PartPlan part_plan(uint64_t n, bool carry);   // carry: an aux word travels with every key

// Bytes of the passes' scratch for n keys (carry: an aux word travels; cursor: the cursor
// form's regions; sizes: the size words of the unfused form); with base given, a's scratch
// pointers are set into it.
size_t part_scratch(const PartPlan& plan, uint64_t n, bool carry, bool cursor, bool sizes, char* base, PartArgs* a);

// The partition passes over the wide maps of a batch (attempt 0 of each).  Inputs:
// d_keys/d_vals (the batch input), segs (nseg device descriptors), pools; Cpool receives the maps'
// level-two triples (T per map, at index map*T).  Per-map outcome words flags[4*seg + 0..3]: nonzero
// word 0 = attempt rejected (a bucket over 15 keys, more than c*n cells or an overflowing region), word 1 = a bucket exhausted its trials, word 2 = that bucket holds equal
// keys, word 3 = max trial.  *S points into the scratch, to every map's cells.
uint32_t wide_tiles(uint32_t n);      // scatter tiles of a map of n keys
uint64_t wide_parts_max();            // most partitions of a call
size_t wide_scratch_bytes(uint32_t nseg, uint64_t parts, uint64_t tiles);
int wide_build(const uint64_t* d_keys, const uint32_t* d_vals, const WideSeg* segs, uint32_t nseg, uint64_t parts,
               uint64_t tiles, Triple* Cpool, uint32_t T, Group* hdr_pool, Cell* slot_pool, uint32_t* flags,
               uint64_t** S, void* scratch, hipStream_t st);
uint64_t part_scan_tiles(const PartPlan& P);
// Polls of a predecessor's look-back word before the fused pass takes that sum from the records, for
// the calling thread's builds (0: at once; the table is the same).
void part_patience(uint32_t polls);
int part_prepare(const PartArgs& a, hipStream_t st, PartOut& o);
// given_t: trial index of every bucket decided elsewhere (n bytes), or nullptr to search.
// reject: two device words (a bucket above 15 keys, bad string offsets); when either is set
// the pass writes nothing (nullptr: never).  cap: cells allocated at slots; a partition
// whose cells would end beyond them writes nothing (the caller compares S with cap).
// The fused pass uses up o's cleared look-back words (o.prezeroed is reset).
int part_finish(const PartArgs& a, PartOut& o, const Triple* C, uint32_t T, Group* header, Cell* slots,
                uint32_t* flags, const int64_t* ctx_off, const uint8_t* ctx_bytes, const uint8_t* given_t,
                const uint32_t* reject, uint64_t cap, hipStream_t st);

}  // namespace fks
