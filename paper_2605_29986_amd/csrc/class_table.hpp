// Grouping by hash table, the first attempt of cfgzip_build_classes (paper Section 3.1
// "Pre-Computation").
//
// A class is a set of tokens with equal signatures, and equal signatures carry equal hashes, so the
// tokens are first gathered by 37 bits of it and, inside that, by first byte, because signatures
// that share the first byte are compared on short vectors.  Three launches, or two:
//   1. table_gather_kernel: a workgroup takes a run of tokens and gathers them in LDS: what it passes
//      on are the classes and the groups that it meets, an entry each, and no longer the tokens (a class
//      with a third of the vocabulary is then one entry of every run).  A small vocabulary does
//      without: its tokens are the entries;
//   2. table_merge_kernel: classes and groups are dealt out to buckets, a workgroup each.  Every
//      workgroup looks at all entries and keeps those of its bucket, which it then tells apart in LDS,
//      with each class's smallest token id and smallest (byte length, token id): nobody else has an
//      entry of these, so nothing in memory has to be cleared or shared;
//   3. table_settle_kernel: every token is compared with one member of its group, and every group's
//      member with one member of its class (equality is transitive, so all members are equal iff none
//      of these pairs differs); other workgroups number the classes: a class's id is the number of
//      classes with a smaller smallest member.
// If any pair differs (a hash collision), a bucket has no room for its classes, or the walk store turns
// out not to be usable, the host starts over with the sort, which settles collisions exactly; then
// nothing computed here is used.
//
// What bounds it: the chain of dependent launches (about 4.6 us each at the least) and, in the last, the comparisons.
// A table in memory that all workgroups share has to be cleared first and is paid for in atomics on its entries, and
// which tokens are the smallest of their class is known only at its end, which takes a launch more.  So it was before
// (clear, group, verify, assign); kernel times then and now, us:
//      4,096 tokens in 2,980 classes        28 (2 + 17 + 5 + 4)            14 (merge 7, settle 7)
//     32,000 tokens in   683 classes        22 (2 + 8 + 7 + 4)             20 (gather 6, merge 5, settle 9)
//    151,936 tokens in 2,559 classes        48 (5.5 + 15 + 23 + 4)         37 (7 + 6 + 24)
//    128,256 rows of 2 KB in 150 classes    56 (5.4 + 7 + 39 + 4.4)        49 (5 + 5 + 39)
//     32,000 rows of 8 KB                   73 (5 + 12 + 52 + 4)           51 (5.4 + 5 + 40.5)
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "classes_compare.hpp"
#include "common.hpp"

namespace cfgzip {
namespace {

// An entry is one 64-bit word, entered with one compare-and-swap: 37 hash bits, 8 bits of first byte
// and, below them, the id of the token that made it.  More tokens than this would not fit and go to the sort.
// 37 bits are what leaves one over, so that no entry looks like an empty slot.  A pair of classes that share
// them costs the whole attempt and then the sort: 32 bits did so for one vocabulary in two with 80,000 classes
// (151,936 tokens against 256 random states, such a seed: 368 us, 79 with 37 bits), 37 bits for one in forty.
constexpr int kTokenBits = 18;
constexpr int kTableHashBits = 37;
constexpr int32_t kTableMaxTokens = 1 << kTokenBits;
constexpr unsigned long long kTokenMask = kTableMaxTokens - 1;
constexpr unsigned long long kNoEntry = ~0ull;
static_assert(kTableHashBits + 8 + kTokenBits < 64, "an entry is never all ones");
constexpr int kCrossParts = 4;   // waves that share one comparison across two image rows
// Runs of tokens that the gathering workgroups take, a token per thread.
constexpr int kRunBits = 10;
constexpr int kRun = 1 << kRunBits;
constexpr int kMaxRuns = kTableMaxTokens / kRun;
// Up to here the tokens are the entries: every bucket then looks at every token, which takes longer than a launch from
// about here on (3,000 / 6,000 / 10,000 / 16,000 tokens: merge 6.9 / 10.1 / 12.4 / 15.8 us; gathered first, gather and
// merge 10.0 / 10.3 / 10.2 / 10.2 and the launch; calls of 7,000 tokens 46 to 50 and 50 us, of 8,000 48 and 47).
constexpr int32_t kDirectTokens = 7168;

// Buckets: at most as many as there are compute units, and 64 tokens in each on average (the lists of groups to be
// compared, kListedLeast a bucket, then stay small against the vocabulary).
constexpr int kMergeThreads = 1024;
constexpr int kMergeWaves = kMergeThreads / 64;
constexpr int kMaxBuckets = 256;
constexpr int kBucketTokens = 64;
// Workgroups that share the comparisons of a bucket's groups, and those that compare tokens with their groups' members, at
// the most: what a chip takes at a time is 768, and a workgroup costs its start.  Settling 151,936 / 128,256 tokens from the
// walk store with 4 and 2,048 23.8 / 17.2 us, 2 and 2,048 21.9 / 16.3, 2 and 1,280 21.6 / 15.4, 2 and 768 23.3 / 15.7, 1 and
// 2,048 26.0 / 18.6; whole builds with 2 and 768 / 1,280 / 2,048, 64,000 tokens 32.5 / 32.7 / 32.6, 96,000 35.5 / 35.5 / 35.8,
// 128,256 38.1 / 38.0 / 39.0, 151,936 44.2 / 43.5 / 43.9.  With fewer buckets than there may be the chip is not full, and four are better (a call on 4,096 tokens
// 38.9 us, with two 39.9).
constexpr int kPairBlocks = 1280;
inline int table_group_shift(int buckets) { return buckets < kMaxBuckets ? 2 : 1; }  // as a power of two
// A bucket's LDS table.  262,144 tokens of a class each put 1,024 into a bucket, give or take 32, and half full a run
// of kTableProbes taken slots has a chance of 1e-11 in each place.
constexpr int kTableSlotBits = 11;
constexpr int kTableSlots = 1 << kTableSlotBits;
constexpr int kTableProbes = 128;
constexpr uint32_t kNoSlot = 0x3FFF;  // fits above an entry's number in a word
static_assert(kTableSlots <= (int)kNoSlot && kTokenBits + 14 <= 32, "");
constexpr int kMergeList = 8192;  // entries of a bucket's list (LDS for two workgroups in a compute unit)
constexpr int kListedLeast = 512;

inline int table_buckets(int32_t V) {
    int b = 1;
    while (b < kMaxBuckets && 2 * b * kBucketTokens <= V) b *= 2;
    return b;
}
// Groups that a bucket may list: with what its table has room for, a list of 256 such would take more memory than the
// sort does on small vocabularies.
inline int table_list_room(int32_t V) {
    const int per = 4 * (V / table_buckets(V));
    return per < kListedLeast ? kListedLeast : (per < kTableSlots ? per : kTableSlots);
}

// The bucket of a class or a group.  A hash need only be a function of the signature (numbers in a row, a checksum, a value
// written twice), so it is mixed until every bit of the bucket hangs on every bit of its low half, and only hashes made
// for it fall together.  Those still give the exact classes, but one workgroup then works for all: 128,000 tokens in 4,000
// classes whose hashes fall into one bucket 1,520 us, 47 spread out.  (A weighted sum of the bytes did so for hashes that
// differ in their bytes and not in the sum.)  Of 262,144 regular hashes (multiples of small and large numbers, squares,
// floats, pairs) the fullest of 256 buckets gets 1,183, of random ones 1,123.  The products are of 24 bits, which run at
// full rate: on a small vocabulary every workgroup does this for all tokens (4,096 of them: 32-bit products 0.3 us more).
__device__ __forceinline__ uint32_t bucket_of(unsigned long long word, uint32_t mask) {
    static_assert(kMaxBuckets <= 256, "the last eight bits say which");
    const uint32_t low = (uint32_t)(word >> (8 + kTokenBits)), high = (uint32_t)(word >> (8 + kTokenBits + 32));
    const uint32_t fb = (uint32_t)(word >> kTokenBits) & 0xFFu;
    uint32_t x = __umul24(low, 0x9E3779u) + (low >> 8);
    x ^= x >> 11;
    x = __umul24(x, 0x85EBCBu) + (x >> 7);
    return ((x >> 24) + high * 37u + fb) & mask;
}

struct TableTokens {
    const uint64_t *hash;
    const int64_t *tok_off;
    const uint8_t *tok_bytes;
    int n;
    bool by_first_byte;  // false: rows are compared whole, the first byte does not matter
};

// A token's entry word and (byte length, id), the latter as one word that orders them.
struct TokenEntry {
    unsigned long long word, rep;
};
__device__ __forceinline__ TokenEntry token_entry(int t, unsigned long long hash, int64_t beg, int64_t end, uint32_t fb) {
    const int64_t len = min(max(end - beg, (int64_t)0), (int64_t)0x7FFFFFFF);
    return {((hash & ((1ull << kTableHashBits) - 1ull)) << (8 + kTokenBits)) | ((unsigned long long)fb << kTokenBits) | (uint32_t)t,
            ((unsigned long long)len << 32) | (uint32_t)t};
}

__device__ __forceinline__ unsigned long long class_word(unsigned long long word) {  // without the first byte
    return word & ~(0xFFull << kTokenBits);
}

// The slot of `mine`'s key in an LDS table, where the smallest token id with that key comes to stand.  False: there is
// no room.  `made`: this thread's was the first.
template <int SLOT_BITS, int PROBES>
__device__ __forceinline__ bool lds_enter(unsigned long long *table, unsigned long long mine, uint32_t &at, bool &made) {
    constexpr uint32_t mask = (1u << SLOT_BITS) - 1;
    at = (uint32_t)(((mine >> kTokenBits) * 0x9E3779B97F4A7C15ull) >> (64 - SLOT_BITS));
    made = false;
    for (int probe = 0; probe < PROBES; ++probe, at = (at + 1) & mask) {
        unsigned long long seen = *(volatile unsigned long long *)&table[at];
        if (seen == kNoEntry) {
            seen = atomicCAS(&table[at], kNoEntry, mine);
            made = seen == kNoEntry;
            if (made) return true;
        }
        if ((seen >> kTokenBits) == (mine >> kTokenBits)) {
            if (mine < seen) atomicMin(&table[at], mine);
            return true;
        }
    }
    return false;
}

// The entries of the runs, [runs][kRun] each, those of a run in the order of their buckets; `starts` [buckets + 1][runs]
// says where in its run a bucket's entries begin (the last row: where they all end).
struct RunEntries {
    unsigned long long *word;
    uint16_t *starts;
};

struct TableGatherArgs {
    TableTokens tok;
    RunEntries cls, group;        // out (groups only where the first byte matters)
    unsigned long long *cls_rep;  // out, beside cls.word
    int buckets;
    int2 *entry_of;               // [n] out: a token's entries, class and group
    uint8_t *tok_head;            // [n] cleared
};

// The entries are dealt out here: with their order a bucket's workgroup finds its own by two numbers a run.  (Looking
// for them by the entries' buckets took it 5 to 11 us on 151,936 tokens, looking at all tokens' hashes 160 us, most of
// that for the bucket with a third of the tokens.)
__global__ __launch_bounds__(kRun) void table_gather_kernel(TableGatherArgs a) {
    constexpr int kSlots = 2 * kRun;  // at most half full
    __shared__ unsigned long long cls[kSlots], rep[kSlots], group[kSlots];
    __shared__ uint16_t cls_number[kSlots], group_number[kSlots];
    __shared__ uint32_t in_bucket[2][kMaxBuckets];  // classes, groups; then where they begin
    __shared__ uint32_t wave_tot[2 * kMaxBuckets / 64];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int t = blockIdx.x * kRun + tid;
    const bool in = t < a.tok.n, groups = a.tok.by_first_byte;
    TokenEntry mine{0, 0};
    if (in) {
        const int64_t beg = a.tok.tok_off[t], end = a.tok.tok_off[t + 1];
        const unsigned long long h = a.tok.hash[t];
        const uint32_t fb = groups && end > beg ? (uint32_t)a.tok.tok_bytes[beg] : 0u;
        mine = token_entry(t, h, beg, end, fb);
        a.tok_head[t] = 0;
    }
#pragma unroll
    for (int s = tid; s < kSlots; s += kRun) {
        cls[s] = group[s] = kNoEntry;
        rep[s] = ~0ull;
    }
    if (tid < 2 * kMaxBuckets) in_bucket[tid / kMaxBuckets][tid % kMaxBuckets] = 0;
    __syncthreads();
    uint32_t c = 0, g = 0, c_bucket = 0, g_bucket = 0, c_at = 0, g_at = 0;
    bool made_c = false, made_g = false;
    if (in) {  // (there are more slots than tokens)
        lds_enter<kRunBits + 1, kSlots>(cls, class_word(mine.word), c, made_c);
        if (mine.rep < *(volatile unsigned long long *)&rep[c]) atomicMin(&rep[c], mine.rep);
        if (groups) lds_enter<kRunBits + 1, kSlots>(group, mine.word, g, made_g);
        if (made_c) {
            c_bucket = bucket_of(class_word(mine.word), (uint32_t)a.buckets - 1u);
            c_at = atomicAdd(&in_bucket[0][c_bucket], 1u);
        }
        if (made_g) {
            g_bucket = bucket_of(mine.word, (uint32_t)a.buckets - 1u);
            g_at = atomicAdd(&in_bucket[1][g_bucket], 1u);
        }
    }
    __syncthreads();
    // where the buckets begin: two scans of 256 counts, four waves each
    uint32_t count = 0, begin = 0;
    if (tid < 2 * kMaxBuckets) {
        count = in_bucket[tid / kMaxBuckets][tid % kMaxBuckets];
        begin = (uint32_t)wave_inclusive_sum((int)count);
        if (lane == 63) wave_tot[wave] = begin;
        begin -= count;
    }
    __syncthreads();
    if (tid < 2 * kMaxBuckets) {
        const int of = tid / kMaxBuckets, b = tid % kMaxBuckets;
        for (int w = of * (kMaxBuckets / 64); w < wave; ++w) begin += wave_tot[w];
        in_bucket[of][b] = begin;
        uint16_t *starts = of ? a.group.starts : a.cls.starts;
        if (b < a.buckets && (of == 0 || groups)) {
            starts[(size_t)b * gridDim.x + blockIdx.x] = (uint16_t)begin;
            if (b + 1 == a.buckets) starts[(size_t)(b + 1) * gridDim.x + blockIdx.x] = (uint16_t)(begin + count);
        }
    }
    __syncthreads();
    const uint32_t first = blockIdx.x * kRun;
    if (made_c) {
        c_at += in_bucket[0][c_bucket];
        cls_number[c] = (uint16_t)c_at;
        a.cls.word[first + c_at] = cls[c];
        a.cls_rep[first + c_at] = rep[c];
    }
    if (made_g) {
        g_at += in_bucket[1][g_bucket];
        group_number[g] = (uint16_t)g_at;
        a.group.word[first + g_at] = group[g];
    }
    __syncthreads();
    if (in) a.entry_of[t] = make_int2((int)(first + cls_number[c]), groups ? (int)(first + group_number[g]) : 0);
}

struct TableMergeArgs {
    TableTokens tok;  // DIRECT
    RunEntries cls, group;  // otherwise
    const unsigned long long *cls_rep;
    int n;
    int buckets;         // a power of two; the first workgroups merge classes, as many more groups
    int32_t *cls_of, *group_of;  // out, per entry: the smallest member of its class / group
    uint8_t *tok_head;   // [n] out: 1 for the smallest member of a class; DIRECT: cleared as well
    int32_t *rep_at;     // [n] out, at the smallest member of a class: its representative
    int32_t *listed_group;  // [buckets][list_room] out: the groups' smallest members
    int32_t *listed_count;  // [buckets]
    int list_room;
    Counters *host_ctr;  // pinned host memory
};

// DIRECT: the entries are the tokens.  Classes and groups have workgroups of their own: by the hash alone the groups of a
// class, and with a third of the tokens in it 6,600 of 45,000 entries, would all come to one bucket (27 us).
template <bool DIRECT>
__global__ __launch_bounds__(kMergeThreads, 8) void table_merge_kernel(TableMergeArgs a) {
    __shared__ unsigned long long table[kTableSlots], rep[kTableSlots];
    __shared__ uint32_t list[kMergeList];
    __shared__ int32_t wave_tot[kMaxRuns / 64];
    __shared__ int32_t picked, listed, no_room;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const bool groups = (int)blockIdx.x >= a.buckets;  // what this workgroup merges
    const uint32_t bucket = blockIdx.x - (groups ? (uint32_t)a.buckets : 0u), mask = (uint32_t)a.buckets - 1u;
    const RunEntries from = groups ? a.group : a.cls;
    int32_t *member_of = groups ? a.group_of : a.cls_of;
    const int runs = (a.n + kRun - 1) / kRun;
    for (int s = tid; s < kTableSlots; s += kMergeThreads) {
        table[s] = kNoEntry;
        rep[s] = ~0ull;
    }
    if (tid == 0) picked = 0, listed = 0, no_room = 0;
    // A run's entries of this bucket, a run per thread.
    int first_of = 0, left_of = 0;
    if (!DIRECT && tid < runs) {
        const int first = from.starts[(size_t)bucket * runs + tid], last = from.starts[(size_t)(bucket + 1) * runs + tid];
        first_of = tid * kRun + first;
        left_of = min(max(last - first, 0), kRun - first);
    }
    __syncthreads();
    // Lists this bucket's entries of runs [run0, run1); beyond the list's end they are counted only.  How many, the same
    // for everybody.
    auto pick = [&](int run0, int run1) -> int {
        if (DIRECT) {  // all tokens at once
            constexpr int kAhead = 4;
            for (int t0 = tid; t0 < a.n; t0 += kAhead * kMergeThreads) {
                unsigned long long hash[kAhead];
                uint32_t fb[kAhead];
#pragma unroll
                for (int u = 0; u < kAhead; ++u) {
                    const int t = min(t0 + u * kMergeThreads, a.n - 1);
                    hash[u] = a.tok.hash[t];
                    fb[u] = 0;
                    if (groups) {
                        const int64_t beg = a.tok.tok_off[t];
                        if (a.tok.tok_off[t + 1] > beg) fb[u] = (uint32_t)a.tok.tok_bytes[beg];
                    }
                }
#pragma unroll
                for (int u = 0; u < kAhead; ++u) {
                    const int t = t0 + u * kMergeThreads;
                    if (t < a.n && bucket_of(token_entry(t, hash[u], 0, 0, fb[u]).word, mask) == bucket)
                        list[atomicAdd(&picked, 1)] = (uint32_t)t;
                }
            }
            __syncthreads();
            return picked;
        }
        const bool mine = tid >= run0 && tid < run1;
        const int count = mine ? left_of : 0;
        int at = 0, all = 0;
        if (tid < kMaxRuns) {
            at = wave_inclusive_sum(count);
            if (lane == 63) wave_tot[wave] = at;
        }
        __syncthreads();
#pragma unroll
        for (int w = 0; w < kMaxRuns / 64; ++w) {
            at += w < wave ? wave_tot[w] : 0;
            all += wave_tot[w];
        }
        at -= count;
        for (int k = 0; k < count && at + k < kMergeList; ++k) list[at + k] = (uint32_t)(first_of + k);
        __syncthreads();
        return all;
    };
    // The list's entries into the table, where the smallest token of a class or group comes to stand for it; a list's
    // entry keeps its slot above the entry's number.
    auto enter = [&](int count) {
        constexpr int kTogether = 2;
        for (int i0 = tid; i0 < count; i0 += kTogether * kMergeThreads) {
            int32_t e[kTogether];
            TokenEntry x[kTogether];
#pragma unroll
            for (int u = 0; u < kTogether; ++u) {
                const int i = i0 + u * kMergeThreads;
                e[u] = i < count ? (int32_t)list[i] : 0;  // (an entry of its own: others' are being rewritten)
                if (DIRECT) {
                    const int64_t beg = a.tok.tok_off[e[u]], end = a.tok.tok_off[e[u] + 1];
                    const uint32_t fb = groups && end > beg ? (uint32_t)a.tok.tok_bytes[beg] : 0u;
                    x[u] = token_entry(e[u], a.tok.hash[e[u]], beg, end, fb);
                } else {
                    x[u] = {from.word[e[u]], groups ? 0ull : a.cls_rep[e[u]]};
                }
            }
#pragma unroll
            for (int u = 0; u < kTogether; ++u) {
                const int i = i0 + u * kMergeThreads;
                if (i >= count) continue;
                uint32_t s = kNoSlot;
                bool made;
                if (*(volatile int32_t *)&no_room != 0 ||
                    !lds_enter<kTableSlotBits, kTableProbes>(table, x[u].word, s, made)) {
                    s = kNoSlot;
                    no_room = 1;
                } else if (!groups && x[u].rep < *(volatile unsigned long long *)&rep[s]) {
                    atomicMin(&rep[s], x[u].rep);
                }
                list[i] = (uint32_t)e[u] | (s << kTokenBits);
                if (DIRECT && !groups) a.tok_head[e[u]] = 0;
            }
        }
        __syncthreads();
    };
    auto say_members = [&](int count) {
        for (int i = tid; i < count; i += kMergeThreads) {
            const uint32_t s = list[i] >> kTokenBits;
            member_of[list[i] & (uint32_t)kTokenMask] = s < (uint32_t)kTableSlots ? (int32_t)(table[s] & kTokenMask) : 0;
        }
    };
    const int found = pick(0, runs);
    static_assert(kDirectTokens <= kMergeList, "all tokens fit the list");
    if (DIRECT || found <= kMergeList) {
        enter(found);
        say_members(found);
    } else {
        // more than the list holds: a few runs at a time, and once more when it is known which tokens are the smallest
        constexpr int kTogether = kMergeList / kRun;
        for (int round = 0; round < 2; ++round) {
            for (int run0 = 0; run0 < runs; run0 += kTogether) {
                __syncthreads();  // everybody is done with the list
                const int count = pick(run0, min(run0 + kTogether, runs));
                enter(count);
                if (round == 1) say_members(count);
            }
        }
    }
    __syncthreads();
    for (int s = tid; s < kTableSlots; s += kMergeThreads) {
        const unsigned long long e = table[s];
        if (e == kNoEntry) continue;
        const int32_t smallest = (int32_t)(e & kTokenMask);
        if (groups) {
            const int at = atomicAdd(&listed, 1);
            if (at < a.list_room) a.listed_group[(size_t)bucket * a.list_room + at] = smallest;
            else no_room = 1;
        } else {
            a.rep_at[smallest] = (int32_t)(uint32_t)rep[s];
            a.tok_head[smallest] = 1;
        }
    }
    __syncthreads();
    if (tid == 0 && groups) a.listed_count[bucket] = min(listed, a.list_room);
    if (tid == 0 && no_room) a.host_ctr->no_room = 1;
}

constexpr int kTableThreads = 512;  // of the settling workgroups

struct TableSettleArgs {
    const int2 *entry_of;  // a token's entries, class and group, or null: the tokens are the entries
    const int32_t *cls_of, *group_of, *rep_at;
    const uint8_t *tok_head;
    int n;
    int number_blocks, buckets;  // the first workgroups number, the next compare a bucket's groups, the rest tokens
    int list_room, group_shift;
    const int32_t *listed_group, *listed_count;
    StoreSource store;    // from the walk store
    const uint16_t *sig;  // from rows: [n][S]
    int S;
    Counters *host_ctr;  // pinned host memory
    int32_t *class_of_token, *rep_of_class, *num_classes_dev;
};

// the smallest member of a token's class / group
__device__ __forceinline__ int32_t class_member(const TableSettleArgs &a, int t) {
    return a.cls_of[a.entry_of ? a.entry_of[t].x : t];
}
__device__ __forceinline__ int32_t group_member(const TableSettleArgs &a, int t) {
    return a.group_of[a.entry_of ? a.entry_of[t].y : t];
}

constexpr int kNumberPer = 2;                                // tokens per thread of the workgroups that number
constexpr int kRankWords = kTableMaxTokens / 64 / kTableThreads;  // 64 tokens' marks each, a thread's share at the most
// LDS of the workgroups that number: a bit per token, and the marks before every 64 of them.
inline size_t table_rank_bytes(int32_t V) {
    return (size_t)ceil_div(V, 64 * kRankWords) * kRankWords * (sizeof(uint64_t) + sizeof(uint32_t));
}

__device__ __forceinline__ void table_number(const TableSettleArgs &a, unsigned char *lds) {
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int shares = (a.n + 64 * kRankWords - 1) / (64 * kRankWords), words = shares * kRankWords;
    unsigned long long *bits = reinterpret_cast<unsigned long long *>(lds);        // [words]
    uint32_t *before = reinterpret_cast<uint32_t *>(lds + (size_t)words * 8);      // [words]
    __shared__ uint32_t wave_tot[kTableThreads / 64];
    const int base = (int)blockIdx.x * (kTableThreads * kNumberPer);
    int32_t smallest[kNumberPer];
#pragma unroll
    for (int j = 0; j < kNumberPer; ++j) {
        const int t = base + j * kTableThreads + tid;
        smallest[j] = class_member(a, min(t, a.n - 1));
    }
    // sixteen tokens' marks, a byte each, to sixteen bits
    for (int x = tid; x < words * 4; x += kTableThreads) {
        const uint4 v = reinterpret_cast<const uint4 *>(a.tok_head)[x];
        uint32_t lo = __builtin_amdgcn_udot4(v.x, 0x08040201u, 0u, false);
        lo = __builtin_amdgcn_udot4(v.y, 0x80402010u, lo, false);
        uint32_t hi = __builtin_amdgcn_udot4(v.z, 0x08040201u, 0u, false);
        hi = __builtin_amdgcn_udot4(v.w, 0x80402010u, hi, false);
        uint32_t m = (lo & 0xFFu) | (hi & 0xFFu) << 8;
        const int left = a.n - x * 16;  // what lies behind the last token is not a mark
        if (left < 16) m &= left > 0 ? (1u << left) - 1u : 0u;
        reinterpret_cast<uint16_t *>(bits)[x] = (uint16_t)m;
    }
    __syncthreads();
    uint32_t pop[kRankWords], mine = 0;
#pragma unroll
    for (int w = 0; w < kRankWords; ++w) {
        pop[w] = tid < shares ? (uint32_t)__popcll(bits[tid * kRankWords + w]) : 0u;
        mine += pop[w];
    }
    const uint32_t incl = (uint32_t)wave_inclusive_sum((int)mine);
    if (lane == 63) wave_tot[wave] = incl;
    __syncthreads();
    uint32_t run = incl - mine, total = 0;
#pragma unroll
    for (int w = 0; w < kTableThreads / 64; ++w) {
        run += w < wave ? wave_tot[w] : 0u;
        total += wave_tot[w];
    }
    if (tid < shares) {
#pragma unroll
        for (int w = 0; w < kRankWords; ++w) {
            before[tid * kRankWords + w] = run;
            run += pop[w];
        }
    }
    __syncthreads();
    if (blockIdx.x == 0 && tid == 0) {
        if (a.num_classes_dev) *a.num_classes_dev = (int32_t)total;
        a.host_ctr->num_classes = (int32_t)total;
    }
#pragma unroll
    for (int j = 0; j < kNumberPer; ++j) {
        const int t = base + j * kTableThreads + tid;
        if (t >= a.n) continue;
        const int32_t m = smallest[j];
        const int32_t k = (int32_t)(before[m >> 6] + (uint32_t)__popcll(bits[m >> 6] & ((1ull << (m & 63)) - 1ull)));
        a.class_of_token[t] = k;
        if (m == t) a.rep_of_class[k] = a.rep_at[t];
    }
}

// 16-byte units of a row that a wave compares at a time: of four rows each, or, where a row has that many, four times as many
// of one, so that what it asks for lies together.  Items go by fours of rows, then by parts, then, of long rows, by the four.
constexpr uint32_t kRowPart = 64;
constexpr int kLongRow = 4 * 8 * (int)kRowPart;  // entries
__host__ __device__ inline int64_t table_row_items(int32_t n, int32_t S) {
    if (S >= kLongRow) return ((int64_t)n + 3) / 4 * 4 * ((S + kLongRow - 1) / kLongRow);
    return ((int64_t)n + 3) / 4 * ((S + 8 * (int)kRowPart - 1) / (8 * (int)kRowPart));
}

// What the comparisons read: the walk store, rows of whole 16-byte units at multiples of that, or rows at any address (an
// instance each: 128,256 rows of 2 KB 39.5 us in whole units; at any address 42, and with both in one kernel's registers 49).
enum : int { SETTLE_STORE, SETTLE_UNITS, SETTLE_ROWS };
template <int FROM>
__global__ __launch_bounds__(kTableThreads) CFGZIP_OWN_PAGES void table_settle_kernel(TableSettleArgs a) {
    extern __shared__ __align__(16) unsigned char lds[];  // table_rank_bytes, or the waves' staged vectors
    if ((int)blockIdx.x < a.number_blocks) {
        table_number(a, lds);
        return;
    }
    constexpr bool STORE = FROM == SETTLE_STORE, UNITS = FROM == SETTLE_UNITS;
    constexpr int kWaves = kTableThreads / 64;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    uint16_t *staged = reinterpret_cast<uint16_t *>(lds) + (size_t)wave * 2 * kWalkStoreMaxStride;  // STORE only
    const int block = (int)blockIdx.x - a.number_blocks;
    const int group_blocks = STORE ? a.buckets << a.group_shift : 0, share = block & ((1 << a.group_shift) - 1);
    // where groups are compared: a lane's first group, asked for before the store's header is looked at
    const int parts = STORE && a.S >= 8 ? kCrossParts : 1;
    const int teams = (kWaves / parts) << a.group_shift, team = share * (kWaves / parts) + wave / parts;
    const int32_t *listed = a.listed_group + (size_t)(block >> a.group_shift) * a.list_room;
    int listed_here = 0, next_group = 0;
    if (block < group_blocks) {
        listed_here = min(max(a.listed_count[block >> a.group_shift], 0), a.list_room);
        next_group = listed[min(team + lane * teams, a.list_room - 1)];
    }
    uint32_t stride = 0;  // of the walk store
    if (STORE) {
        const int state = walk_store_state(a.store, stride);
        if (state) {
            if (block == 0 && tid == 0) a.host_ctr->store_state = state;
            return;
        }
    }
    bool differs = false;
    if (STORE && block < group_blocks) {
        // groups against a member of their class, a few workgroups per bucket: kCrossParts waves share a pair (S
        // >= 8).  A lane looks at a group, and where its smallest member is not its class's the wave compares
        // the two
        for (int x0 = team; x0 < listed_here; x0 += 64 * teams) {
            const int x = x0 + lane * teams;
            const int32_t group = x0 == team ? next_group : listed[min(x, listed_here - 1)];
            const int32_t t = x < listed_here ? group : 0, other = x < listed_here ? class_member(a, group) : 0;
            const uint32_t ra = store_row(a.store, t), rb = store_row(a.store, other);
            for (uint64_t left = __ballot(t != other); left; left &= left - 1) {
                const int l = __ffsll((unsigned long long)left) - 1;
                differs |= store_other_row_differ(a.store, stride, __builtin_amdgcn_readlane(t, l),
                                                  __builtin_amdgcn_readlane(other, l), __builtin_amdgcn_readlane(ra, l),
                                                  __builtin_amdgcn_readlane(rb, l), staged, staged + kWalkStoreMaxStride,
                                                  wave % parts, parts);
            }
        }
    } else {
        const int64_t gw = (int64_t)(block - group_blocks) * kWaves + wave;
        const int64_t waves = ((int64_t)gridDim.x - a.number_blocks - group_blocks) * kWaves;
        if (STORE) {
            // eight pairs per wave, eight lanes a pair, 16 bytes a lane and round: what a token's own entry says is
            // enough to ask for both vectors
            const uint32_t sub = lane & 7, pair = lane >> 3;
            for (int64_t t0 = gw * 8; t0 < a.n; t0 += waves * 8) {
                const int64_t t = min(t0 + pair, (int64_t)a.n - 1);  // repeats the last one past the end
                const int32_t ref = group_member(a, (int)t);
                const uint16_t pa = a.store.store.wrow[t];
                const uint4 *wa = reinterpret_cast<const uint4 *>(a.store.store.wvec + (size_t)t * stride);
                const uint4 *wb = reinterpret_cast<const uint4 *>(a.store.store.wvec + (size_t)ref * stride);
                const uint32_t n16 = min(walk_units_of(pa), stride / 8u);  // none of the empty token
                const uint16_t pb = a.store.store.wrow[ref];
                constexpr int kAhead = 2;
                uint32_t diff = 0;
                for (uint32_t u0 = sub; u0 < n16; u0 += 8 * kAhead) {
                    uint4 x[kAhead], y[kAhead];
#pragma unroll
                    for (int k = 0; k < kAhead; ++k) {
                        const uint32_t u = min(u0 + 8 * k, n16 - 1);
                        x[k] = wa[u];
                        y[k] = wb[u];
                    }
#pragma unroll
                    for (int k = 0; k < kAhead; ++k)
                        diff |= (x[k].x ^ y[k].x) | (x[k].y ^ y[k].y) | (x[k].z ^ y[k].z) | (x[k].w ^ y[k].w);
                }
                const uint32_t ra = min(walk_row_of(pa), 256u), rb = min(walk_row_of(pb), 256u);
                const bool cross = ra != rb;  // the empty token shares its key with tokens that begin with byte 0
                differs |= !cross && diff != 0u;
                uint64_t left = __ballot(cross && sub == 0);
                while (left) {
                    const int l = __ffsll((unsigned long long)left) - 1;
                    left &= left - 1;
                    differs |= store_other_row_differ(a.store, stride, __shfl((int32_t)t, l, 64), __shfl(ref, l, 64),
                                                      __shfl(ra, l, 64), __shfl(rb, l, 64), staged,
                                                      staged + kWalkStoreMaxStride);
                }
            }
        } else {
            // rows against their classes' members' rows, which many share (they stay in the caches); what there is to read is
            // every row once.  A wave takes four rows at a time, 1 KB of each, or 4 KB of one where a row has that: whole rows of
            // 8 KB, which all begin at the same memory channels, took longer than either.  Four waves next to each other then take
            // the same part of four rows, and so workgroups that go to different XCDs different parts: with rows of a power of two an
            // XCD's cache holds a part of every member's row, and not all of them.  Four rows / one, its parts by waves next to each
            // other / one, as here; calls on rows in whole units, us, with 150, 1,500 and 6,000 classes:
            //   32,000 rows of 4.5 KB     50.9 / 49.9 / 50.3     63.0 / 58.1 / 58.4     65.2 / 58.8 / 59.4
            //   32,000 rows of 8 KB       67.9 / 62.4 / 62.5     90.4 / 84.2 / 84.3     91.2 / 80.9 / 80.8
            //   30,000 rows of 16 KB     117.4 / 117.0 / 111.7  143.6 / 141.8 / 136.8  141.2 / 129.1 / 128.2
            //   16,000 rows of 16 KB      67.1 / 69.2 / 61.9     88.0 / 83.9 / 81.2     83.1 / 71.0 / 70.8
            //    8,000 rows of 32 KB      66.7 / 77.2 / 61.2     84.4 / 79.2 / 75.7
            //    4,000 rows of 60 KB      80.4 / 73.6 / 74.9     74.1 / 61.2 / 61.8
            // (eight rows, a part to a workgroup, 3 to 5 us less where rows are multiples of 8 KB, but up to 30 % more where the last
            // part has little: its workgroups have nothing to do), and relations with their classes, 32,000 x 256 states, 155.3 either
            // way of one.  Lanes behind the end of a row read nothing: what a row of a little over 4 KB has in its last part is a few
            // units, and asked for by all lanes they made 60,000 rows of 2,056 entries 71 us instead of 67, of 2,055 (at any address)
            // 106 instead of 79.
            const bool vec = UNITS || a.S >= 8;
            const uint32_t s8 = ((uint32_t)a.S + 7u) / 8u;
            const bool long_rows = a.S >= kLongRow;
            const int64_t items = table_row_items(a.n, vec ? a.S : 1), parts = items / (((int64_t)a.n + 3) / 4) / (long_rows ? 4 : 1);
            for (int64_t x = gw; x < items; x += waves) {
                const int64_t fours = long_rows ? x / 4 : x, t0 = fours / parts * 4 + (long_rows ? x % 4 : 0);
                int32_t t[4], ref[4];
                int cnt = 0;
#pragma unroll
                for (int u = 0; u < 4; ++u) {
                    t[u] = (int32_t)min(t0 + (long_rows ? 0 : u), (int64_t)a.n - 1);  // repeats the last one past the end
                    ref[u] = class_member(a, t[u]);
                    cnt += ref[u] != t[u];
                }
                if (!cnt) continue;  // all four are their classes' members (wave-uniform)
                if (vec) {
                    const uint32_t apart = long_rows ? kRowPart : 0u;  // of the four pieces, in their row
                    const uint32_t from = (uint32_t)(fours % parts) * (long_rows ? 4u * kRowPart : kRowPart) + lane;
                    if (from < s8) {
                        u32x4_any p[4], q[4];
                        auto piece = [&](uint32_t tok, uint32_t j) -> u32x4_any {  // of a token's row
                            if (UNITS) {
                                const uint4 v = reinterpret_cast<const uint4 *>(a.sig)[tok * s8 + j];  // (31 bits)
                                return u32x4_any{v.x, v.y, v.z, v.w};
                            }
                            const uint16_t *row = a.sig + (size_t)tok * a.S;
                            return *reinterpret_cast<const u32x4_any *>(row + min(8u * j, (uint32_t)a.S - 8u));
                        };
#pragma unroll
                        for (int u = 0; u < 4; ++u) {
                            p[u] = q[u] = u32x4_any{0u, 0u, 0u, 0u};
                            if (from + u * apart >= s8) continue;  // behind the row: of its last part there may be little
                            p[u] = piece((uint32_t)t[u], from + u * apart);
                            q[u] = piece((uint32_t)ref[u], from + u * apart);
                        }
#pragma unroll
                        for (int u = 0; u < 4; ++u)
                            differs |= (p[u].x != q[u].x) | (p[u].y != q[u].y) | (p[u].z != q[u].z) | (p[u].w != q[u].w);
                    }
                } else {
                    for (int j = lane; j < a.S; j += 64)
#pragma unroll
                        for (int u = 0; u < 4; ++u)
                            differs |= a.sig[(size_t)t[u] * a.S + j] != a.sig[(size_t)ref[u] * a.S + j];
                }
            }
        }
    }
    // whether any pair differs is all that is asked
    if (__ballot(differs) != 0ull && lane == 0) a.host_ctr->unresolved = 1;
}

}  // namespace
}  // namespace cfgzip
