// Grouping by hash table, the first attempt of cfgzip_build_classes (paper Section 3.1
// "Pre-Computation").
//
// A class is a set of tokens with equal signatures, and equal signatures carry equal hashes, so the
// tokens are first gathered by 37 bits of it and, inside that, by first byte, because signatures
// that share the first byte are compared on short vectors.  Four launches:
//   1. table_clear_kernel: the two tables start empty;
//   2. table_group_kernel: a workgroup first gathers its tokens in LDS (a class with a third of
//      the vocabulary then costs one access to its entry per workgroup and not one per token), then
//      enters its distinct (hash, first byte) groups and its distinct hashes into the tables, and
//      lowers each class's smallest token id and smallest (byte length, token id);
//   3. table_verify_kernel: every token is compared with one member of its group, and every group's
//      member with one member of its class (equality is transitive, so all members are equal iff none
//      of these pairs differs); other workgroups look the tokens' smallest class members up and mark
//      the tokens that are one;
//   4. table_assign_kernel: class id = number of marked tokens below the class's smallest member.
// If any pair differs (a hash collision), or the walk store turns out not to be usable, the host
// starts over with the sort, which settles collisions exactly; then nothing computed here is used.
//
// What bounds it: the chain of four dependent launches (about 4.6 us each at the least) and, inside
// each, three to five dependent memory accesses (on 151,936 tokens the waves of the group and verify kernels wait in
// 79 and 76 % of their cycles); with rows as the source, reading them once.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "classes_compare.hpp"
#include "common.hpp"

namespace cfgzip {
namespace {

// Tokens per workgroup in table_group_kernel, one per thread: 128 (2^7) or 1,024 (2^10).  Large workgroups meet
// a class less often, and the accesses to one entry are served one after the other; small ones put more compute
// units on a small vocabulary, most of whose tokens make an entry.  Measured with 64 / 128 / 1,024 threads:
// 4,096 tokens in 2,980 classes 14.8 / 14.7 / 22.4 us, 32,000 in 683 classes 16.2 / 8.4 / 8.3 us, 128,256 in
// 1,460 classes 59.9 / 25.8 / 12.8 us.
constexpr int kGroupBitsSmall = 7, kGroupBitsLarge = 10;
constexpr int32_t kGroupSmallTokens = 16384;
constexpr int kTableThreads = 256;
constexpr int kTableAssignThreads = 512;
constexpr int kTableAssignItems = 2;
// An entry is one 64-bit word, entered with one compare-and-swap: 37 hash bits, 8 bits of first byte
// and, below them, the id of the token that made it.  More tokens than this would not fit and go to the sort.
// 37 bits are what leaves one over, so that no entry looks like an empty slot.  A pair of classes that share
// them costs the whole attempt and then the sort: 32 bits did so for one vocabulary in two with 80,000 classes
// (151,936 tokens against 256 random states, such a seed: 368 us, 79 with 37 bits), 37 bits for one in forty.
constexpr int kTokenBits = 18;
constexpr int kTableHashBits = 37;
constexpr int32_t kTableMaxTokens = 1 << kTokenBits;
constexpr unsigned long long kNoEntry = ~0ull;
static_assert(kTableHashBits + 8 + kTokenBits < 64, "an entry is never all ones");
constexpr int kCrossParts = 4;  // waves that share one comparison across two image rows

// Open addressing, linear probing; the capacity is a power of two and at least 1.25 V, so an
// insertion always ends.
struct ClassTable {
    unsigned long long *group;    // (hash bits, first byte, one member)
    unsigned long long *cls;      // (hash bits, 0, one member)
    unsigned long long *cls_rep;  // smallest (byte length << 32 | token id)
    uint32_t *cls_min;            // smallest token id
    uint32_t mask;                // capacity - 1
    int shift;                    // 64 - log2(capacity)
};

inline uint32_t class_table_capacity(int32_t V) {
    uint32_t cap = 1024;
    if (V > kTableMaxTokens) return cap;  // not used
    while ((uint64_t)cap * 4 < (uint64_t)V * 5) cap <<= 1;
    return cap;
}

__device__ __forceinline__ uint32_t table_home(unsigned long long key, int shift) {
    return (uint32_t)((key * 0x9E3779B97F4A7C15ull) >> shift);
}

struct TableClearArgs {
    uint4 *words;  // the arrays of the table lie behind each other
    size_t n16;
    Counters *ctr;
};

__global__ __launch_bounds__(kTableThreads) void table_clear_kernel(TableClearArgs a) {
    if (blockIdx.x == 0 && threadIdx.x == 0) {
        a.ctr->unresolved = 0;
        a.ctr->num_classes = 0;
        a.ctr->store_state = 0;
        a.ctr->other_rows = 0;
    }
    const size_t step = (size_t)gridDim.x * kTableThreads;
    for (size_t i = (size_t)blockIdx.x * kTableThreads + threadIdx.x; i < a.n16; i += step)
        a.words[i] = make_uint4(~0u, ~0u, ~0u, ~0u);
}

struct TableGroupArgs {
    const uint64_t *hash;
    const int64_t *tok_off;
    const uint8_t *tok_bytes;
    int n;
    bool by_first_byte;  // false: rows are compared whole, the first byte does not matter
    ClassTable t;
    int32_t *tok_ref;    // [n] out: a member of the token's group, the same for the whole group
    int32_t *tok_cls;    // [n] out: its class's entry
    int2 *cross_list;    // (member of a group, member of its class), to be compared across first bytes
    Counters *ctr;       // other_rows counts the list
};

__device__ __forceinline__ unsigned long long table_look(const unsigned long long *entry) {
    return __hip_atomic_load(entry, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// The entry of `mine`'s key from slot `at` on, whose content was `seen` after any attempt to claim it
// (kNoEntry: `mine` has claimed it).  Returns the entry as it stands in the table.
__device__ __forceinline__ unsigned long long table_settle(unsigned long long *table, uint32_t mask, uint32_t &at,
                                                           unsigned long long mine, unsigned long long seen) {
    for (uint32_t probes = 0; probes <= mask; ++probes) {
        if (seen == kNoEntry) return mine;
        if ((seen >> kTokenBits) == (mine >> kTokenBits)) return seen;
        at = (at + 1) & mask;
        seen = table_look(&table[at]);
        if (seen == kNoEntry) seen = atomicCAS(&table[at], kNoEntry, mine);
    }
    return mine;  // not reached: the table has more slots than there are tokens
}

// The slot of the key in the workgroup's LDS table, at most half full; `made`: this thread's entry is there.
template <int SLOT_BITS>
__device__ __forceinline__ uint32_t lds_enter(unsigned long long *table, unsigned long long mine, bool &made) {
    constexpr uint32_t mask = (1u << SLOT_BITS) - 1;
    uint32_t at = table_home(mine >> kTokenBits, 64 - SLOT_BITS);
    made = false;
    for (uint32_t probes = 0; probes <= mask; ++probes, at = (at + 1) & mask) {
        unsigned long long seen = *(volatile unsigned long long *)&table[at];
        if (seen == kNoEntry) seen = atomicCAS(&table[at], kNoEntry, mine);
        if (seen == kNoEntry) {
            made = true;
            return at;
        }
        if ((seen >> kTokenBits) == (mine >> kTokenBits)) return at;
    }
    return at;
}

// The thread whose token made an entry of the LDS tables takes it on to the tables in memory: at most one group
// and one class per thread, both under way together, two dependent accesses in all.  (A loop over the LDS
// slots, two per thread, with a look before every compare-and-swap and minimum, and list entries reserved per
// wave: 45 us on 128,256 tokens with 512 threads; without the loop 24 us; without the looks, which cost a round
// trip and save nothing while all workgroups run at once, 12.8 us with 1,024 threads.)
template <int BITS>
__global__ __launch_bounds__(1 << BITS) void table_group_kernel(TableGroupArgs a) {
    constexpr int kGroupThreads = 1 << BITS;
    constexpr int kGroupSlots = 2 * kGroupThreads;  // the LDS tables are at most half full
    __shared__ unsigned long long group[kGroupSlots], cls[kGroupSlots], crep[kGroupSlots];
    __shared__ uint32_t cmin[kGroupSlots], centry[kGroupSlots];
    __shared__ int32_t gref[kGroupSlots], cref[kGroupSlots];
    __shared__ int32_t wave_listed[kGroupThreads / 64];
    __shared__ int32_t list_at;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
#pragma unroll
    for (int s = tid; s < kGroupSlots; s += kGroupThreads) {
        group[s] = kNoEntry;
        cls[s] = kNoEntry;
        crep[s] = ~0ull;
        cmin[s] = ~0u;
    }
    const int t = blockIdx.x * kGroupThreads + tid;
    const bool in = t < a.n;
    unsigned long long part = 0, packed = 0;
    uint32_t fb = 0;
    if (in) {
        const int64_t beg = a.tok_off[t];
        int64_t len = a.tok_off[t + 1] - beg;
        part = a.hash[t] & ((1ull << kTableHashBits) - 1ull);
        if (a.by_first_byte && len > 0) fb = (uint32_t)a.tok_bytes[beg];
        len = len < 0 ? 0 : (len > 0x7FFFFFFF ? 0x7FFFFFFF : len);
        packed = ((unsigned long long)len << 32) | (uint32_t)t;
    }
    const unsigned long long my_cls = (part << (8 + kTokenBits)) | (uint32_t)t;
    const unsigned long long my_group = my_cls | ((unsigned long long)fb << kTokenBits);
    __syncthreads();
    uint32_t g = 0, c = 0;
    bool made_g = false, made_c = false;
    if (in) {
        c = lds_enter<BITS + 1>(cls, my_cls, made_c);
        if (packed < *(volatile unsigned long long *)&crep[c]) atomicMin(&crep[c], packed);
        if ((uint32_t)t < *(volatile uint32_t *)&cmin[c]) atomicMin(&cmin[c], (uint32_t)t);
        g = lds_enter<BITS + 1>(group, my_group, made_g);
    }
    __syncthreads();
    bool new_group = false;
    {
        uint32_t ec = table_home(my_cls >> kTokenBits, a.t.shift), eg = table_home(my_group >> kTokenBits, a.t.shift);
        unsigned long long sc = 0, sg = 0;
        if (made_c) sc = atomicCAS(&a.t.cls[ec], kNoEntry, my_cls);
        if (made_g) sg = atomicCAS(&a.t.group[eg], kNoEntry, my_group);
        if (made_c) sc = table_settle(a.t.cls, a.t.mask, ec, my_cls, sc);
        if (made_g) sg = table_settle(a.t.group, a.t.mask, eg, my_group, sg);
        constexpr unsigned long long kToken = kTableMaxTokens - 1;
        if (made_g) {
            gref[g] = (int32_t)(sg & kToken);
            new_group = sg == my_group;
        }
        if (made_c) {
            centry[c] = ec;
            cref[c] = (int32_t)(sc & kToken);
            atomicMin(&a.t.cls_rep[ec], crep[c]);
            atomicMin(&a.t.cls_min[ec], cmin[c]);
        }
    }
    __syncthreads();
    // a group that this token has made is compared with its class's member, unless that is the token itself
    const bool listed = a.by_first_byte && new_group && cref[c] != t;
    const uint64_t lm = __ballot(listed);
    if (lane == 0) wave_listed[wave] = (int32_t)__popcll(lm);
    if (in) {
        a.tok_ref[t] = gref[g];
        a.tok_cls[t] = (int32_t)centry[c];
    }
    __syncthreads();
    int32_t before = 0, all = 0;
    for (int w = 0; w < kGroupThreads / 64; ++w) {
        before += w < wave ? wave_listed[w] : 0;
        all += wave_listed[w];
    }
    if (all == 0) return;  // the same for the whole workgroup
    if (tid == 0) list_at = atomicAdd(&a.ctr->other_rows, all);
    __syncthreads();
    if (listed) a.cross_list[list_at + before + __popcll(lm & ((1ull << lane) - 1ull))] = make_int2(t, cref[c]);
}

struct TableVerifyArgs {
    ClassTable t;
    const int32_t *tok_ref, *tok_cls;
    int n;
    int mark_blocks, cross_blocks;  // the first workgroups mark, the next compare the list, the rest tokens
    const int2 *cross_list;
    Counters *ctr;
    StoreSource store;    // from the walk store
    const uint16_t *sig;  // from rows: [n][S]
    int S;
    // out, per token and per word of 32 tokens / stretch of kTableThreads tokens
    int32_t *tok_min, *rep_at;
    uint2 *word_marks;  // the word's marks, and the number of marks before it in its stretch
    int32_t *stretch_marks;
};

__device__ __forceinline__ void table_mark(const TableVerifyArgs &a) {
    __shared__ uint32_t wave_marks[kTableThreads / 64];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int t = blockIdx.x * kTableThreads + threadIdx.x;
    bool head = false;
    if (t < a.n) {
        const int32_t c = a.tok_cls[t];
        const int32_t m = (int32_t)a.t.cls_min[c];
        a.tok_min[t] = m;
        head = m == t;
        if (head) a.rep_at[t] = (int32_t)(uint32_t)a.t.cls_rep[c];
    }
    const uint64_t marks = __ballot(head);
    if (lane == 0) wave_marks[wave] = (uint32_t)__popcll(marks);
    __syncthreads();
    uint32_t before = 0, all = 0;
    for (int w = 0; w < kTableThreads / 64; ++w) {
        before += w < wave ? wave_marks[w] : 0u;
        all += wave_marks[w];
    }
    if (lane < 2) {
        const uint32_t low = (uint32_t)__popcll(marks & 0xFFFFFFFFull);
        a.word_marks[(size_t)blockIdx.x * (kTableThreads / 32) + wave * 2 + lane] =
            make_uint2((uint32_t)(marks >> (32 * lane)), before + (lane ? low : 0u));
    }
    if (threadIdx.x == 0) a.stretch_marks[blockIdx.x] = (int32_t)all;
}

// STORE: the comparisons read the walk store, otherwise rows.
template <bool STORE>
__global__ __launch_bounds__(kTableThreads) void table_verify_kernel(TableVerifyArgs a) {
    __shared__ __align__(16) uint16_t staged[STORE ? kTableThreads / 64 : 1][2][STORE ? kWalkStoreMaxStride : 8];
    if ((int)blockIdx.x < a.mark_blocks) {
        table_mark(a);
        return;
    }
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int block = (int)blockIdx.x - a.mark_blocks;
    constexpr int kWaves = kTableThreads / 64;
    uint32_t stride = 0;  // of the walk store
    if (STORE) {
        const int state = walk_store_state(a.store, stride);
        if (state) {
            if (block == 0 && threadIdx.x == 0) a.ctr->store_state = state;
            return;
        }
    }
    bool differs = false;
    if (STORE && block < a.cross_blocks) {
        // groups against a member of their class: kCrossParts waves share a pair (S a multiple of 8)
        const int parts = (a.S % 8) == 0 ? kCrossParts : 1;
        const int count = min(a.ctr->other_rows, a.n);
        for (int64_t e = (int64_t)block * kWaves + wave; e < (int64_t)count * parts; e += (int64_t)a.cross_blocks * kWaves) {
            const int2 pair = a.cross_list[e / parts];
            const uint32_t ra = store_row(a.store, pair.x), rb = store_row(a.store, pair.y);
            if (ra == rb && ra != 256u) {
                if (e % parts == 0) differs |= store_same_row_differ(a.store, stride, pair.x, pair.y);
            } else {
                differs |= store_other_row_differ(a.store, stride, pair.x, pair.y, ra, rb, staged[wave][0], staged[wave][1],
                                                  (int)(e % parts), parts);
            }
        }
    } else {
        const int64_t gw = (int64_t)(block - a.cross_blocks) * kWaves + wave;
        const int64_t waves = ((int64_t)gridDim.x - a.mark_blocks - a.cross_blocks) * kWaves;
        if (STORE) {
            // eight pairs per wave, eight lanes a pair, 16 bytes a lane and round
            const uint32_t sub = lane & 7, pair = lane >> 3;
            for (int64_t t0 = gw * 8; t0 < a.n; t0 += waves * 8) {
                const int64_t t = t0 + pair;
                bool cross = false;
                uint32_t n16 = 0, ra = 256, rb = 256;
                int32_t ref = 0;
                const uint4 *wa = nullptr, *wb = nullptr;
                uint4 x0 = make_uint4(0, 0, 0, 0);
                if (t < a.n) {
                    ref = a.tok_ref[t];
                    const uint16_t pa = a.store.store.wrow[t];
                    wa = reinterpret_cast<const uint4 *>(a.store.store.wvec + (size_t)t * stride);
                    wb = reinterpret_cast<const uint4 *>(a.store.store.wvec + (size_t)ref * stride);
                    // (asked for before it is known to be wanted: every token has `stride` entries)
                    if (sub < stride / 8u) x0 = wa[sub];
                    const uint16_t pb = a.store.store.wrow[ref];
                    ra = min(walk_row_of(pa), 256u);
                    rb = min(walk_row_of(pb), 256u);
                    cross = ra != rb;  // the empty token shares its key with tokens that begin with byte 0
                    if (ref != t && ra == rb && ra != 256u) n16 = min(walk_units_of(pa), stride / 8u);
                }
                for (uint32_t u = sub; u < n16; u += 8) {
                    const uint4 x = u == sub ? x0 : wa[u], y = wb[u];
                    differs |= (x.x != y.x) | (x.y != y.y) | (x.z != y.z) | (x.w != y.w);
                }
                uint64_t list = __ballot(cross && sub == 0);
                while (list) {
                    const int l = __ffsll((unsigned long long)list) - 1;
                    list &= list - 1;
                    differs |= store_other_row_differ(a.store, stride, (int32_t)(t0 + (l >> 3)), __shfl(ref, l, 64),
                                                      __shfl(ra, l, 64), __shfl(rb, l, 64), staged[wave][0],
                                                      staged[wave][1]);
                }
            }
        } else {
            // four rows per wave and round against their groups' members' rows, which many share (they
            // stay in the caches); what there is to read is every row once
            const bool vec = (a.S % 8) == 0 && (reinterpret_cast<uintptr_t>(a.sig) % 16) == 0;
            for (int64_t t0 = gw * 4; t0 < a.n; t0 += waves * 4) {
                const uint16_t *x[4], *y[4];
                int cnt = 0;
#pragma unroll
                for (int u = 0; u < 4; ++u) {
                    const int64_t t = min(t0 + u, (int64_t)a.n - 1);  // repeats the last one past the end
                    const int32_t ref = a.tok_ref[t];
                    cnt += ref != t;
                    x[u] = a.sig + (size_t)t * a.S;
                    y[u] = a.sig + (size_t)ref * a.S;
                }
                if (!cnt) continue;  // all four are their groups' members (wave-uniform)
                if (vec) {
                    for (int j = lane; j < a.S / 8; j += 64) {
                        uint4 p[4], q[4];
#pragma unroll
                        for (int u = 0; u < 4; ++u) {
                            p[u] = reinterpret_cast<const uint4 *>(x[u])[j];
                            q[u] = reinterpret_cast<const uint4 *>(y[u])[j];
                        }
#pragma unroll
                        for (int u = 0; u < 4; ++u)
                            differs |= (p[u].x != q[u].x) | (p[u].y != q[u].y) | (p[u].z != q[u].z) |
                                       (p[u].w != q[u].w);
                    }
                } else {
                    for (int j = lane; j < a.S; j += 64)
#pragma unroll
                        for (int u = 0; u < 4; ++u) differs |= x[u][j] != y[u][j];
                }
            }
        }
    }
    // whether any pair differs is all that is asked
    if (__ballot(differs) != 0ull && lane == 0) atomicAdd(&a.ctr->unresolved, 1);
}

struct TableAssignArgs {
    int n, n_stretches;
    const int32_t *tok_min, *rep_at;
    const uint2 *word_marks;
    const int32_t *stretch_marks;
    const Counters *ctr;
    Counters *host_ctr;  // pinned host memory
    int32_t *class_of_token, *rep_of_class, *num_classes_dev;
};

__global__ __launch_bounds__(kTableAssignThreads) void table_assign_kernel(TableAssignArgs a) {
    extern __shared__ uint32_t before[];  // [n_stretches]: marks before each stretch
    __shared__ uint32_t wave_tot[kTableAssignThreads / 64];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int base = blockIdx.x * (kTableAssignThreads * kTableAssignItems);
    int32_t m[kTableAssignItems];
    uint2 marks[kTableAssignItems];
#pragma unroll
    for (int j = 0; j < kTableAssignItems; ++j) {
        const int t = base + j * kTableAssignThreads + tid;
        m[j] = t < a.n ? a.tok_min[t] : 0;
        m[j] = (uint32_t)m[j] < (uint32_t)a.n ? m[j] : 0;  // always: every class has a member
    }
#pragma unroll
    for (int j = 0; j < kTableAssignItems; ++j) marks[j] = a.word_marks[m[j] >> 5];
    // a scan per workgroup (1,024 stretches, two a thread, at the most) instead of a launch of its own
    uint32_t run = 0;
    for (int s0 = 0; s0 < a.n_stretches; s0 += kTableAssignThreads) {
        const int s = s0 + tid;
        const uint32_t v = s < a.n_stretches ? (uint32_t)a.stretch_marks[s] : 0u;
        const uint32_t incl = (uint32_t)wave_inclusive_sum((int)v);
        if (lane == 63) wave_tot[wave] = incl;
        __syncthreads();
        uint32_t pre = run, all = 0;
#pragma unroll
        for (int w = 0; w < kTableAssignThreads / 64; ++w) {
            pre += w < wave ? wave_tot[w] : 0u;
            all += wave_tot[w];
        }
        if (s < a.n_stretches) before[s] = pre + incl - v;
        run += all;
        __syncthreads();
    }
    if (blockIdx.x == 0 && tid == 0) {
        if (a.num_classes_dev) *a.num_classes_dev = (int32_t)run;
        a.host_ctr->unresolved = a.ctr->unresolved;
        a.host_ctr->store_state = a.ctr->store_state;
        a.host_ctr->other_rows = a.ctr->other_rows;
        a.host_ctr->num_classes = (int32_t)run;
    }
#pragma unroll
    for (int j = 0; j < kTableAssignItems; ++j) {
        const int t = base + j * kTableAssignThreads + tid;
        if (t >= a.n) continue;
        const int32_t k = (int32_t)(before[m[j] / kTableThreads] + marks[j].y +
                                    __popc(marks[j].x & ((1u << (m[j] & 31)) - 1u)));
        a.class_of_token[t] = k;
        if (m[j] == t) a.rep_of_class[k] = a.rep_at[t];
    }
}

}  // namespace
}  // namespace cfgzip
