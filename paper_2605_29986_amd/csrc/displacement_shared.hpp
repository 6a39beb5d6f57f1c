// Displacement sets by a walk over shared configuration sets: the first pass of cfgzip_displacements (paper
// Section 3.2.1, Algorithm 1).
//
// After p bytes of a token Algorithm 1 holds a SET of configurations (input queue, output stack, symbol consumed
// last), and the set after the next byte depends on nothing but that set and the byte.  Tokens of a vocabulary
// meet few different sets (the 128,256 tokens of the measured vocabulary 230 over the JSON grammar), so a
// workgroup keeps the sets it has met in LDS, numbers them, and remembers which set follows which on which byte.
// A lane then walks its token like a word over a deterministic automaton, one look-up a byte; only where a
// successor is not known yet do the 64 lanes of the wave work it out together, a lane per configuration, and add
// it to what all sixteen waves of the workgroup share.
//
// Queues and stacks are lists of shared cells: a cell is one 32-bit word (the rest of the list, a symbol, the
// length), its number is its slot in a hash table keyed by that very word, and equal lists have equal numbers.  A
// configuration is therefore one 32-bit word, a set some of them, and comparing two sets comparing words.  Cells and
// sets are entered by one compare-and-swap after what they refer to has been written, and two waves that enter the
// same thing at the same time agree on the first entry.
//
// What follows a set on a byte, and what a set is written as, is claimed first: a placeholder goes into the table, the
// wave works the answer out, and the answer takes the placeholder's place.  Who needs it meanwhile looks again until it
// is there.  So that every such wait ends, a wave waits for nothing between its claim and the answer, and does not leave
// without giving it.
//
// What a token's set is written as (the canonical row and its hash) is worked out once per set too; writing a row
// is then a copy out of LDS, and writing the rows is what bounds the kernel on a large vocabulary.
//
// Measured: 128,256 tokens over the JSON grammar with rows of 1,024 entries 109 us (a wave per token took 510 us for
// most tokens and 276 us for long digit runs), 32,000 over the statement grammar with rows of 256 71 us (210 us).
// What bounds it is instruction issue (with the JSON grammar the vector units are busy for 60 % of the kernel, and the scalar
// one about as long), and in the workgroup that is done last a chain of sets that nobody has met.  A step alone in its compute
// unit takes 2.2 us, 670 instructions and twenty LDS accesses (the steps of 32 digits over the JSON grammar, sets of 20 to 51
// configurations; 3.75 us with the pairs of configuration and production listed in LDS, the next set looked up and loaded
// again, and a production read through a pointer that may be global, which waits for all rows on their way to memory).  Slower:
// longest tokens first for some of the waves and shortest first for the others (JSON call 2 to 16 %; the
// rows then go out earlier, but the chain is what counts), rows two at a time, claims asked for ahead of a step's first
// look-ups (2 %: more instructions), the symbols of a set's lists in registers to bring them into order, a wave of few tokens
// that waits for all of them before it writes any (JSON 1 to 5 %).
//
// Everything in LDS is bounded.  A token that would need more (more than 128 successors at a byte, more cells,
// sets or row entries than there is room for) goes to the list of the passes behind this one, which take it alone.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include <type_traits>

#include "displacement_alone.hpp"
#include "displacement_common.hpp"

namespace cfgzip {
namespace {

constexpr int kShThreads = 1024;
constexpr int kShWaves = kShThreads / 64;
constexpr int kShCells = 2048;      // list cells (8 KB)
constexpr int kShNext = 2048;       // known successors (8 KB)
constexpr int kShSets = 1024;       // sets (8 KB, and 16 KB for what they are written as)
// Steps that a wave works out before its lanes try alone.  The waves of a workgroup with 125 tokens over the JSON or the
// statement grammar work out 6 to 8 steps, with 501 tokens 10 to 14; from the first step on it costs them 1.3 %, from
// the 7th 0.8, from here nothing that could be measured (from the 25th on tokens that share no sets take 5 to 30 % longer).
constexpr int kShShared = 12;
constexpr int kShPool = 6144;       // configurations of all sets (24 KB)
constexpr int kShOut = 18432;       // row entries of all sets written so far (36 KB)
constexpr int kShProds = 1024;      // productions kept in LDS (8 KB); of a larger grammar none are
constexpr int kShAdj = 512;         // words of the relation kept in LDS (2 KB); of a larger one none are
constexpr int kShPairs = 2048;      // (byte, symbol) pairs whose productions are looked up directly (4 KB)
constexpr int kShFollow = 2048;     // (byte, symbol consumed last) pairs whose backtracks are looked up directly, and a word
                                    // a byte (8 KB)
constexpr int kShFew = 32;          // productions a byte has at the most where they are: a bit each
constexpr int kShBatch = 1024;      // tokens a workgroup sorts by length at a time
constexpr int kShBytes = 6144;      // their bytes, kept in LDS; if there are more they are read from memory
constexpr int kShLengths = 64;      // lengths told apart in sorting
// Sorted tokens that a wave takes at a time, at the most: where the workgroup has up to kShFewTokens of them, and where it has
// more.  Few at a time spread the steps over the waves, many make the look-ups of short tokens cheaper.  Calls, four / eight at a
// time, us:
//   tokens a workgroup         188           250           256           313           375           501
//   statement grammar     94.0 /  96.7  101.0 / 104.7  102.3 / 106.1  113.4 / 113.2  118.9 / 117.9  136.6 / 131.9
//   JSON grammar         108.0 / 108.3  109.0 / 109.0  108.4 / 108.9  109.9 / 110.5  115.0 / 113.3  130.0 / 126.2
// (16 and 32 at a time 2 to 7 % more than eight with 501 over the JSON grammar.)
constexpr int kShTakeFew = 4, kShTakeMost = 8;
constexpr int kShFewTokens = 16 * kShWaves;
// Tokens for every wave up to which they are not sorted and a wave takes its share at once.  Calls sorted / not, rows of 1,024
// entries with the JSON grammar, of 256 with the statement grammar, us:
//   tokens a workgroup       47          63          78          94         109         125
//   statement grammar     71 /  67    75 /  72    85 /  82    79 /  85    88 /  94    80 /  87
//   JSON grammar         104 / 113   104 / 107   105 / 115   105 / 116   106 / 123   106 / 129
// The statement grammar's tokens are of much the same length, and what sorting costs it up to 78 tokens the JSON grammar
// gains; tokens that share no sets lose 2 to 7 % from the line on (32,000 of 4 / 8 / 12 bytes).
constexpr int kShOnce = 4;
constexpr int kShSeen = 256;        // slots of a wave's table of the successors found so far: at most half full
constexpr int kShProbes = 48;       // slots looked at before a table counts as full
constexpr int kShFrontier = 128;    // successors of a set at one byte: two a lane
constexpr int kShMaxList = 32;      // symbols of a queue or stack (the interface's bound)
constexpr int kShMaxSymbols = 255;  // symbols, and "none", fit a byte

typedef unsigned long long u64;

// a configuration: queue and stack as cell numbers (slot + 1, 0 = empty; 12 bits each), the symbol consumed last
constexpr int kCellIdBits = 12;
constexpr uint32_t kCellIdMask = (1u << kCellIdBits) - 1;
constexpr uint32_t kNoSymbol = 0xFF;
__device__ __forceinline__ uint32_t sh_config(uint32_t queue, uint32_t stack, uint32_t last) {
    return queue | (stack << kCellIdBits) | (last << (2 * kCellIdBits));
}
__device__ __forceinline__ uint32_t sh_queue(uint32_t c) { return c & kCellIdMask; }
__device__ __forceinline__ uint32_t sh_stack(uint32_t c) { return (c >> kCellIdBits) & kCellIdMask; }
__device__ __forceinline__ uint32_t sh_last(uint32_t c) { return c >> (2 * kCellIdBits); }

// a cell: the number of the rest (12 bits), the symbol (8), the length of the list (6); never 0
__device__ __forceinline__ uint32_t cell_rest(uint32_t w) { return w & kCellIdMask; }
__device__ __forceinline__ uint32_t cell_symbol(uint32_t w) { return (w >> kCellIdBits) & 0xFFu; }
__device__ __forceinline__ uint32_t cell_length(uint32_t w) { return w >> (kCellIdBits + 8); }

// a set: 24 hash bits, the position of its configurations in the pool (16 bits), how many (8)
constexpr u64 kShEmpty = ~0ull;
__device__ __forceinline__ uint32_t set_at(u64 w) { return (uint32_t)(w >> 8) & 0xFFFFu; }
__device__ __forceinline__ uint32_t set_size(u64 w) { return (uint32_t)w & 0xFFu; }

// a known successor: set (10 bits) and byte (8) above the following set (14 bits) or one of these
constexpr uint32_t kNextBits = 14;
constexpr uint32_t kGiveUp = 0x3FFE;    // more room needed than there is: the token goes to the next pass
constexpr uint32_t kCrossed = 0x3FFD;   // a bound of the interface is broken: the token overflows
constexpr uint32_t kWorkedOut = 0x3FFC; // another wave is at it
constexpr uint32_t kByTheWave = 0x3FFB; // never published: what follows takes a whole wave to work out
constexpr uint32_t kNextEmpty = ~0u;

// what a set is written as: position of its row entries (in units of eight) above their number (13 bits), or one of these
constexpr uint32_t kRowUnknown = ~0u;
constexpr uint32_t kRowGiveUp = ~0u - 1;
constexpr uint32_t kRowTooLong = ~0u - 2;
constexpr uint32_t kRowWorkedOut = ~0u - 3;  // another wave is at it
constexpr int kRowBits = 13;
static_assert(kShOut / 8 < 1 << (32 - kRowBits - 1), "no place looks like one of these");
__device__ __forceinline__ uint32_t row_entries(uint32_t row) { return row & ((1u << kRowBits) - 1u); }
__device__ __forceinline__ uint32_t row_at(uint32_t row) { return (row >> kRowBits) * 8u; }

struct SharedLds {
    __align__(16) uint16_t out[kShOut];
    uint32_t pool[kShPool];
    u64 sets[kShSets];
    uint32_t row[kShSets];
    u64 row_hash[kShSets];
    __align__(16) uint32_t work[kShWaves][2 * kShFrontier];
    uint32_t seen[kShWaves][kShSeen];
    uint32_t cells[kShCells];
    uint32_t next[kShNext];
    u64 prods[kShProds];
    union {
        uint32_t adj[kShAdj];   // as long as `follow` is not kept
        uint32_t follow[kShFollow];  // [number of the byte][symbol consumed last, N: none]: which of the byte's productions may
    };                          // come next where the stack is empty, a bit each; [N + 1]: the first of them
    uint32_t byte_off[257];
    uint16_t pair[kShPairs];  // [number of the byte among those with productions of their own][symbol]: first production
                              // (10 bits), how many (6)
    uint8_t byte_number[256];  // the bytes that are the first with their productions numbered, the others as the first
    uint32_t own[8];           // bytes that are their own byte_like
    uint32_t pairs_kept;      // whether `pair` holds what the productions say
    uint32_t few_each;        // no byte has more productions than `follow` has bits
    uint32_t follow_kept;     // whether `follow` holds what the relation says
    uint32_t pool_top, out_top, cursor;
    uint32_t start_set, dead_set;  // nothing consumed and nothing pushed; no configuration left
    uint32_t scattered;      // some token's bytes do not lie where the token before ends
    uint32_t of_length[kShLengths];
    uint16_t order[kShBatch], start[kShBatch + 2];  // the batch's tokens, longest first; where each one's bytes begin
    uint8_t like_of[256];  // [number]: the byte that has it
    uint8_t bytes[kShBytes];  // already as byte_number has them
};

// The kernel's arguments (its first), loaded anew: where they are seldom needed they then take no scalar registers in
// between, of which the walk has too few (107 of them moved to and from vector registers otherwise, and back).
__device__ __forceinline__ DisplacementArgs sh_arguments() {
    auto from = reinterpret_cast<const __attribute__((address_space(4))) uint32_t *>(
        reinterpret_cast<uintptr_t>(__builtin_amdgcn_kernarg_segment_ptr()));
    asm volatile("" : "+s"(from));
    DisplacementArgs a;
    static_assert(sizeof(a) % 4 == 0, "");
#pragma unroll
    for (size_t i = 0; i < sizeof(a) / 4; ++i) {
        const uint32_t w = from[i];
        __builtin_memcpy(reinterpret_cast<char *>(&a) + 4 * i, &w, 4);
    }
    return a;
}

template <typename T>
__device__ __forceinline__ T lds_look(const T *p) {
    return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
}
// What this wave has written to LDS comes before what it publishes next, and what it reads after a look at something
// published is what was written before that: LDS does the operations of a wave in the order in which they are issued, so
// only the compiler has to be told (a fence for the workgroup also waits until all of them are done, an access's time each).
__device__ __forceinline__ void lds_order() { __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront"); }

__device__ __forceinline__ uint32_t wave_read(uint32_t v, int lane) { return __builtin_amdgcn_readlane(v, lane); }
__device__ __forceinline__ u64 wave_read64(u64 v, int lane) {
    return ((u64)wave_read((uint32_t)(v >> 32), lane) << 32) | wave_read((uint32_t)v, lane);
}
// Sum over the 64 lanes (all of them active), the same for every lane: row shifts by 1, 2, 4, 8, then across rows.
__device__ __forceinline__ u64 wave_sum64(u64 v) {
    auto moved = [](u64 x, auto ctrl, auto rows) -> u64 {
        const uint32_t lo = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)(uint32_t)x, decltype(ctrl)::value, decltype(rows)::value, 0xF, true);
        const uint32_t hi = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)(uint32_t)(x >> 32), decltype(ctrl)::value, decltype(rows)::value, 0xF, true);
        return ((u64)hi << 32) | lo;
    };
    v += moved(v, std::integral_constant<int, 0x111>{}, std::integral_constant<int, 0xF>{});
    v += moved(v, std::integral_constant<int, 0x112>{}, std::integral_constant<int, 0xF>{});
    v += moved(v, std::integral_constant<int, 0x114>{}, std::integral_constant<int, 0xF>{});
    v += moved(v, std::integral_constant<int, 0x118>{}, std::integral_constant<int, 0xF>{});
    v += moved(v, std::integral_constant<int, 0x142>{}, std::integral_constant<int, 0xA>{});
    v += moved(v, std::integral_constant<int, 0x143>{}, std::integral_constant<int, 0xC>{});
    return wave_read64(v, 63);
}
// Sum over the lanes up to this one (all 64 are active): row shifts by 1, 2, 4, 8, then across rows.
__device__ __forceinline__ uint32_t wave_upto32(uint32_t v) {
    v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x111, 0xF, 0xF, true);
    v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x112, 0xF, 0xF, true);
    v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x114, 0xF, 0xF, true);
    v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x118, 0xF, 0xF, true);
    v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x142, 0xA, 0xF, true);
    v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x143, 0xC, 0xF, true);
    return v;
}
// Sum over all of them, the same for every lane.
__device__ __forceinline__ uint32_t wave_sum32(uint32_t v) { return wave_read(wave_upto32(v), 63); }
// OR over the 64 lanes (all of them active), the same for every lane.
__device__ __forceinline__ uint32_t wave_or32(uint32_t v) {
    v |= (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x111, 0xF, 0xF, true);
    v |= (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x112, 0xF, 0xF, true);
    v |= (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x114, 0xF, 0xF, true);
    v |= (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x118, 0xF, 0xF, true);
    v |= (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x142, 0xA, 0xF, true);
    v |= (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x143, 0xC, 0xF, true);
    return wave_read(v, 63);
}

// The largest of the lanes' values (all of them active), the same for every lane.
__device__ __forceinline__ uint32_t wave_max32(uint32_t v) {
    auto with = [&](auto ctrl, auto rows) {
        const uint32_t x = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, decltype(ctrl)::value, decltype(rows)::value, 0xF, true);
        v = v > x ? v : x;
    };
    with(std::integral_constant<int, 0x111>{}, std::integral_constant<int, 0xF>{});
    with(std::integral_constant<int, 0x112>{}, std::integral_constant<int, 0xF>{});
    with(std::integral_constant<int, 0x114>{}, std::integral_constant<int, 0xF>{});
    with(std::integral_constant<int, 0x118>{}, std::integral_constant<int, 0xF>{});
    with(std::integral_constant<int, 0x142>{}, std::integral_constant<int, 0xA>{});
    with(std::integral_constant<int, 0x143>{}, std::integral_constant<int, 0xC>{});
    return wave_read(v, 63);
}

__device__ __forceinline__ uint32_t cell_word(uint32_t rest, uint32_t symbol, uint32_t length) {
    return rest | (symbol << kCellIdBits) | (length << (kCellIdBits + 8));
}
__device__ __forceinline__ uint32_t cell_slot(uint32_t w) {
    static_assert(kShCells == 1 << 11, "eleven bits of hash; a number (slot + 1) fits twelve");
    return (w * 0x9E3779B1u) >> (32 - 11);
}
// The numbers of two cells, of which either may be 0 (none wanted, none comes back); 0 and `full` if the table is full.
// They are claimed together, so that the attempts of one do not wait for the other's.
__device__ __forceinline__ void sh_two_cells(SharedLds &L, uint32_t w0, uint32_t w1, uint32_t &id0, uint32_t &id1, bool &full) {
    uint32_t at0 = cell_slot(w0), at1 = cell_slot(w1), seen0 = 0, seen1 = 0;
    if (w0) seen0 = atomicCAS(&L.cells[at0], 0u, w0);
    if (w1) seen1 = atomicCAS(&L.cells[at1], 0u, w1);
    bool open0 = seen0 != 0u && seen0 != w0, open1 = seen1 != 0u && seen1 != w1;
#pragma unroll 1
    for (int probe = 1; (open0 || open1) && probe < kShProbes; ++probe) {
        if (open0) {
            at0 = (at0 + 1) & (kShCells - 1);
            seen0 = atomicCAS(&L.cells[at0], 0u, w0);
        }
        if (open1) {
            at1 = (at1 + 1) & (kShCells - 1);
            seen1 = atomicCAS(&L.cells[at1], 0u, w1);
        }
        open0 = open0 && seen0 != 0u && seen0 != w0;
        open1 = open1 && seen1 != 0u && seen1 != w1;
    }
    full = full || open0 || open1;
    id0 = w0 && !open0 ? at0 + 1 : 0u;
    id1 = w1 && !open1 ? at1 + 1 : 0u;
}
// The number of the list of `length` symbols that is `symbol` in front of `rest`; 0 if the table is full.
__device__ __forceinline__ uint32_t sh_cons(SharedLds &L, uint32_t rest, uint32_t symbol, uint32_t length, bool &full) {
    uint32_t id, none;
    sh_two_cells(L, cell_word(rest, symbol, length), 0u, id, none, full);
    return id;
}

__device__ __forceinline__ uint32_t next_slot(uint32_t key) { return (key * 0x9E3779B1u) >> (32 - 11); }
static_assert(kShNext == 1 << 11, "eleven bits of hash");

// The set that follows `set` on byte `like`, if known: its number, kGiveUp or kCrossed; kNextEmpty if not.
__device__ __forceinline__ uint32_t sh_known(const SharedLds &L, uint32_t set, uint32_t like) {
    const uint32_t key = (set << 8) | like;
    uint32_t at = next_slot(key);
#pragma unroll 1
    for (int probe = 0; probe < kShProbes; ++probe, at = (at + 1) & (kShNext - 1)) {
        const uint32_t w = lds_look(&L.next[at]);
        if (w == kNextEmpty) return kNextEmpty;
        if ((w >> kNextBits) == key) return w & ((1u << kNextBits) - 1);
    }
    return kNextEmpty;
}

// Takes on working out what follows `set` on `like`: the slot to publish it in, -1 if it is known or another wave was
// faster, -2 if the table is full (the successor is then worked out again by everybody who comes here).
__device__ __forceinline__ int sh_claim(SharedLds &L, uint32_t set, uint32_t like) {
    const uint32_t key = (set << 8) | like;
    uint32_t at = next_slot(key);
#pragma unroll 1
    for (int probe = 0; probe < kShProbes; ++probe, at = (at + 1) & (kShNext - 1)) {
        const uint32_t seen = atomicCAS(&L.next[at], kNextEmpty, (key << kNextBits) | kWorkedOut);
        if (seen == kNextEmpty) return (int)at;
        if ((seen >> kNextBits) == key) return -1;
    }
    return -2;
}

// Says what follows `set` on `like`, unless somebody has or is about to.
__device__ __forceinline__ void sh_publish(SharedLds &L, uint32_t set, uint32_t like, uint32_t following) {
    const uint32_t key = (set << 8) | like;
    uint32_t at = next_slot(key);
#pragma unroll 1
    for (int probe = 0; probe < kShProbes; ++probe, at = (at + 1) & (kShNext - 1)) {
        const uint32_t seen = atomicCAS(&L.next[at], kNextEmpty, (key << kNextBits) | following);
        if (seen == kNextEmpty || (seen >> kNextBits) == key) return;
    }
}

// Different words of a wave, two a lane at the most: which of them are the first of their value, where they go when
// packed, how many there are, and a hash that does not depend on their order.
template <int PER>
struct Different {
    uint32_t word[PER];
    bool first[PER];
    int at[PER];
    int n;
    uint32_t sum;
};
constexpr uint32_t kNoWord = ~0u;  // no configuration: cell numbers are below 2^12 - 1

__device__ __forceinline__ uint32_t word_hash(uint32_t w) {
    return (w * 0x85EBCA6Bu) ^ (w >> 13) ^ ((w >> 7) * 0x9E3779B1u);
}
__device__ __forceinline__ uint32_t seen_slot(uint32_t word) { return (word * 0x9E3779B1u) >> 24; }
static_assert(kShSeen == 256, "eight bits of hash");

// `seen` starts empty (all kNoWord) and holds the words afterwards; seen_clear empties it.  One pass of
// compare-and-swaps instead of a sort: comparing 45 words with each other one readlane after the other took as long as
// all the rest of a step.
template <int PER>
__device__ __forceinline__ Different<PER> find_different(uint32_t *seen, const uint32_t (&words)[PER], int lane) {
    Different<PER> d;
    uint32_t h = 0;
    d.n = 0;
#pragma unroll
    for (int u = 0; u < PER; ++u) {
        const uint32_t w = d.word[u] = words[u];
        d.first[u] = false;
        if (w != kNoWord) {
            uint32_t at = seen_slot(w);
#pragma unroll 1
            for (int probe = 0; probe < kShSeen; ++probe, at = (at + 1) & (kShSeen - 1)) {
                const uint32_t old = atomicCAS(&seen[at], kNoWord, w);
                d.first[u] = old == kNoWord;
                if (old == kNoWord || old == w) break;
            }
            if (d.first[u]) h += word_hash(w);
        }
        const u64 mask = __ballot(d.first[u]);
        d.at[u] = d.n + (int)__popcll(mask & ((1ull << lane) - 1ull));
        d.n += (int)__popcll(mask);
    }
    d.sum = wave_sum32(h);
    return d;
}
__device__ __forceinline__ bool seen_has(const uint32_t *seen, uint32_t word) {
    uint32_t at = seen_slot(word);
    for (int probe = 0; probe < kShSeen; ++probe, at = (at + 1) & (kShSeen - 1)) {
        const uint32_t x = seen[at];
        if (x == word) return true;
        if (x == kNoWord) return false;
    }
    return false;
}
__device__ __forceinline__ void seen_clear(uint32_t *seen, int lane) {
#pragma unroll
    for (int u = 0; u < kShSeen / 64; ++u) seen[lane + 64 * u] = kNoWord;
    lds_order();
}

__device__ __forceinline__ uint32_t set_hash(uint32_t sum, uint32_t n) { return (sum ^ (sum >> 15)) * 0x2C1B3C6Du + n; }

// Room in the pool that a wave has reserved and not used yet.
struct PoolRoom {
    int at, n;
    bool none_left;
};
// Sees to it that there is room for n configurations, as far as there is any.  Asked for before it is known whether the set
// is new; what a known set leaves unused is there for the next.  As many as are different, and not as there are successors, for
// what is left of too little is lost: over a grammar with 64 successors for sets of eight the pool was full after a hundred
// steps, and 19,700 of 32,000 tokens were handed on (965 us a call; 360 of them and 292 us so).
__device__ __forceinline__ void sh_reserve(SharedLds &L, PoolRoom &room, int n, int lane) {
    if (room.n >= n || room.none_left) return;
    int top = 0;
    if (lane == 0) top = (int)atomicAdd(&L.pool_top, (uint32_t)n);
    room.at = __builtin_amdgcn_readfirstlane(top);
    room.n = n;
}
// The number of the set of the words `d` (which `seen` holds); kGiveUp if there is no room.  Two sets of equal size
// are equal if each word of one is in the other.
template <int PER>
__device__ __forceinline__ uint32_t sh_set_number(SharedLds &L, PoolRoom &room, const uint32_t *seen, const Different<PER> &d,
                                                  int lane) {
    if (room.n && room.at + room.n > kShPool) {
        room.n = 0;
        room.none_left = true;
    }
    const bool fits = d.n <= room.n;
    if (fits) {
#pragma unroll
        for (int u = 0; u < PER; ++u)
            if (d.first[u]) L.pool[room.at + d.at[u]] = d.word[u];
        lds_order();
    }
    const uint32_t h = set_hash(d.sum, (uint32_t)d.n);
    const u64 tag = (u64)(h >> 8) << 24, mine = tag | ((u64)room.at << 8) | (u64)d.n;
    uint32_t at = h & (kShSets - 1);
#pragma unroll 1
    for (int probe = 0; probe < kShProbes; ++probe, at = (at + 1) & (kShSets - 1)) {
        // one lane's access for the whole wave: the lanes of a read need not see the same moment of a slot that another
        // wave is filling, and the branches below take the whole wave
        u64 found = 0;
        if (lane == 0) found = fits ? atomicCAS(&L.sets[at], kShEmpty, mine) : lds_look(&L.sets[at]);
        found = wave_read64(found, 0);
        if (found == kShEmpty) {
            if (!fits) return kGiveUp;
            room.at += d.n;
            room.n -= d.n;
            return at;
        }
        if ((found >> 24 << 24) == tag && (int)set_size(found) == d.n) {
            lds_order();
            const uint32_t *other = L.pool + set_at(found);
            bool same = true;
            for (int i = lane; i < d.n; i += 64) same = same && seen_has(seen, other[i]);
            if (__ballot(!same) == 0ull) return at;
        }
    }
    return kGiveUp;
}

__device__ __forceinline__ u64 sh_production(const DisplacementArgs &a, const SharedLds &L, int i) {
    // (looks that the compiler cannot join into one access through a generic pointer, which would wait for the rows too)
    return a.g.P <= kShProds ? lds_look(&L.prods[i]) : a.prod_packed[i];
}
// Whether the head of production `p` may come right after the symbol `last` when the stack is empty.
__device__ __forceinline__ bool sh_may_follow(const DisplacementArgs &a, const SharedLds &L, u64 p, uint32_t last) {
    const uint32_t word = packed_head(p) * (uint32_t)a.g.W + (last >> 5);
    return ((a.g.N * a.g.W <= kShAdj && !L.follow_kept ? lds_look(&L.adj[word]) : a.adj[word]) >> (last & 31)) & 1u;
}

// Where `follow` has what may come after the symbol `last` on a byte; behind a byte's symbols, the byte's first production.
__device__ __forceinline__ uint32_t sh_follow(const DisplacementArgs &a, uint32_t byte_number, uint32_t last) {
    return byte_number * (uint32_t)(a.g.N + 2) + (last == kNoSymbol ? (uint32_t)a.g.N : last);
}
__device__ __forceinline__ uint32_t sh_follow_first(const DisplacementArgs &a, uint32_t byte_number) {
    return byte_number * (uint32_t)(a.g.N + 2) + (uint32_t)a.g.N + 1u;
}

// The cell that says what may come next of a configuration: the top of its stack, or the end of its queue where the
// stack is empty; 0 where both are.
__device__ __forceinline__ uint32_t sh_end_cell(const SharedLds &L, uint32_t config) {
    const uint32_t id = sh_stack(config) ? sh_stack(config) : sh_queue(config);
    return id ? lds_look(&L.cells[id - 1]) : 0u;
}

// A configuration, whose end is `cell`, after a production with the head `head` and a body of `length` symbols.
// `crossed`: a bound of the interface is broken; `full`: there is no room.
template <typename Symbol>
__device__ __forceinline__ uint32_t sh_carry_out(SharedLds &L, uint32_t config, uint32_t cell, uint32_t head, int length,
                                                 const Symbol &symbol, bool &full, bool &crossed) {
    const bool pops = sh_stack(config) != 0u;
    uint32_t queue = sh_queue(config), rest = pops ? cell_rest(cell) : 0u, rest_length = pops ? cell_length(cell) - 1u : 0u;
    const uint32_t queued = pops ? 0u : cell_length(cell) + 1u;
    if (queued > (uint32_t)kShMaxList || rest_length + (uint32_t)length > (uint32_t)kShMaxList) {
        crossed = true;
        return kNoWord;
    }
    // the queue's new cell and the stack's first: neither needs the other
    uint32_t queue_end, top;
    sh_two_cells(L, queued ? cell_word(queue, head, queued) : 0u,
                 length ? cell_word(rest, symbol(length - 1), rest_length + 1u) : 0u, queue_end, top, full);
    if (queued) queue = queue_end;
    if (length) {
        rest = top;
        ++rest_length;
#pragma unroll 1
        for (int k = length - 2; k >= 0; --k) rest = sh_cons(L, rest, symbol(k), ++rest_length, full);
    }
    return sh_config(queue, rest, head);
}
// The same after production i, whose body may be of any length.
__device__ __forceinline__ uint32_t sh_carry_out(const DisplacementArgs &a, SharedLds &L, uint32_t config, uint32_t cell, int i,
                                                 bool &full, bool &crossed) {
    const u64 p = sh_production(a, L, i);
    const bool is_long = packed_length(p) == kLongBody;
    const int off = is_long ? a.g.body_off[i] : 0;
    return sh_carry_out(
        L, config, cell, packed_head(p), is_long ? body_len(a.g, i) : (int)packed_length(p),
        [&](int k) -> uint32_t { return is_long ? (uint32_t)a.g.body[off + k] & 0xFFu : packed_symbol(p, k); }, full, crossed);
}

// One byte of Algorithm 1 by one lane, where it is simple enough: a set of one configuration that one production at
// the most applies to.  The number of the set that follows, or kByTheWave.  Every lane has a token of its own here, so
// a vocabulary whose tokens share no sets (every prefix of every token a set of its own: 32,000 tokens of 4, 8, 12 bytes
// over such a grammar) is not worked out one token after the other: 111, 200, 420 us; a wave per token, without the shared
// walk, 125, 172, 220.  What is left is that the tables fill up (from 8 bytes on) and that
// every token's row is its own.  Nothing is claimed first: two lanes that work out the same come to the same.
constexpr int kFewProductions = 4;
__device__ __forceinline__ uint32_t sh_step_alone(const DisplacementArgs &a, SharedLds &L, uint32_t set, uint32_t number,
                                                  uint32_t dead) {
    const u64 w = lds_look(&L.sets[set]);
    lds_order();
    if (set_size(w) != 1u) return kByTheWave;
    const uint32_t config = L.pool[set_at(w)], stack = sh_stack(config), last = sh_last(config), cell = sh_end_cell(L, config);
    int i = 0, n = 0;
    if (stack) {
        if (L.pairs_kept == 0u) return kByTheWave;
        const uint32_t e = L.pair[number * (uint32_t)a.g.N + cell_symbol(cell)];
        i = (int)(e & 0x3FFu);
        n = (int)(e >> 10);
    } else if (L.follow_kept) {
        const uint32_t may = L.follow[sh_follow(a, number, last)];
        n = __popc(may);
        i = (int)L.follow[sh_follow_first(a, number)] + (n ? __ffs(may) - 1 : 0);
    } else {
        const uint32_t like = L.like_of[number];
        const int lo = (int)L.byte_off[like], hi = (int)L.byte_off[like + 1];
        if (hi - lo > kFewProductions) return kByTheWave;
        for (int k = lo; k < hi; ++k) {
            if (last != kNoSymbol && !sh_may_follow(a, L, sh_production(a, L, k), last)) continue;
            i = k;
            ++n;
        }
    }
    if (n == 0) return dead;
    if (n > 1) return kByTheWave;
    bool full = false, crossed = false;
    const uint32_t word = sh_carry_out(a, L, config, cell, i, full, crossed);
    if (crossed) return kCrossed;
    if (full) return kGiveUp;
    const uint32_t h = set_hash(word_hash(word), 1u);
    const u64 tag = (u64)(h >> 8) << 24;
    uint32_t at = h & (kShSets - 1);
    int reserved = -1;
#pragma unroll 1
    for (int probe = 0; probe < kShProbes; ++probe, at = (at + 1) & (kShSets - 1)) {
        u64 found = lds_look(&L.sets[at]);
        if (found == kShEmpty) {
            if (reserved < 0) {
                reserved = (int)atomicAdd(&L.pool_top, 1u);
                if (reserved >= kShPool) return kGiveUp;
                L.pool[reserved] = word;
            }
            lds_order();
            found = atomicCAS(&L.sets[at], kShEmpty, tag | ((u64)reserved << 8) | 1ull);
            if (found == kShEmpty) return at;
        }
        lds_order();
        if ((found >> 24 << 24) == tag && set_size(found) == 1u && L.pool[set_at(found)] == word) return at;
    }
    return kGiveUp;
}

// The pairs of the set's configurations and the productions of `ch` that apply to them, listed in `work`: how many there
// are (of more than kShFrontier only the first are listed).  `seen` starts empty and is left so.
__device__ __forceinline__ int sh_list_pairs(const DisplacementArgs &a, SharedLds &L, uint32_t *work, uint32_t *seen,
                                             uint32_t set, int byte_number, int lane) {
    const Grammar &g = a.g;
    const u64 w = wave_read64(lds_look(&L.sets[set]), 0);  // (what is the same for every lane: in scalar registers)
    lds_order();
    const int n = (int)set_size(w);
    const uint32_t *configs = L.pool + set_at(w);
    const int ch = (int)L.like_of[byte_number];
    const int lo = __builtin_amdgcn_readfirstlane((int)L.byte_off[ch]);
    const int hi = __builtin_amdgcn_readfirstlane((int)L.byte_off[ch + 1]), per = hi - lo;
    const bool pairs_kept = __builtin_amdgcn_readfirstlane(L.pairs_kept) != 0u;
    auto prod = [&](int i) -> u64 { return sh_production(a, L, i); };
    const u64 below = (1ull << lane) - 1ull;
    uint32_t *pair_config = work, *pair_production = work + kShFrontier, *empty = seen;
    int m = 0, empties = 0;
    auto list = [&](bool on, uint32_t config, int i) {
        const u64 mask = __ballot(on);
        const int slot = m + (int)__popcll(mask & below);
        if (on && slot < kShFrontier) {
            pair_config[slot] = config;
            pair_production[slot] = (uint32_t)i;
        }
        m += (int)__popcll(mask);
    };
    // pops: the productions of (byte, top of the stack), which lie behind each other
    for (int c0 = 0; c0 < n; c0 += 64) {
        const int c = c0 + lane;
        const uint32_t config = c < n ? configs[c] : 0u, stack = sh_stack(config);
        uint32_t top = 0;
        if (stack) top = cell_symbol(lds_look(&L.cells[stack - 1]));
        if (pairs_kept) {
            const uint32_t e = stack ? L.pair[(uint32_t)byte_number * (uint32_t)g.N + top] : 0u;
            const int first = (int)(e & 0x3FFu), count = (int)(e >> 10);
            for (int k = 0; __ballot(k < count); ++k) list(k < count, config, first + k);
        } else {
            int i = hi;
            if (stack) {
                i = lo;
                for (int count = per; count > 0;) {  // the first whose head is not below `top`
                    const int half = count >> 1;
                    const bool right = packed_head(prod(i + half)) < top;
                    i = right ? i + half + 1 : i;
                    count = right ? count - half - 1 : half;
                }
            }
            for (;;) {
                const bool on = i < hi && packed_head(prod(i)) == top;
                if (!__ballot(on)) break;
                list(on, config, i);
                i = on ? i + 1 : hi;
            }
        }
        const bool is_empty = c < n && !stack;
        const u64 mask = __ballot(is_empty);
        if (is_empty) empty[empties + __popcll(mask & below)] = config;
        empties += (int)__popcll(mask);
    }
    lds_order();
    // stack backtracks: every production of the byte whose head may come right after the symbol consumed last, for
    // every configuration with an empty stack
    // (four looks at a time, none of which waits for another)
    constexpr int kAhead = 4;
    const float inverse = 1.0f / (float)per;
    for (int x0 = 0; x0 < empties * per && m <= kShFrontier; x0 += 64 * kAhead) {
        bool on[kAhead];
        uint32_t config[kAhead];
        int i[kAhead];
#pragma unroll
        for (int u = 0; u < kAhead; ++u) {
            const int x = x0 + 64 * u + lane;
            on[u] = x < empties * per;
            int e = min((int)(((float)x + 0.5f) * inverse), empties - 1);  // x / per, up to rounding where x is large
            e = e * per > x ? e - 1 : ((e + 1) * per <= x ? e + 1 : e);
            config[u] = on[u] ? empty[e] : 0u;
            i[u] = on[u] ? lo + (x - e * per) : lo;
        }
#pragma unroll
        for (int u = 0; u < kAhead; ++u) {
            if (on[u]) {
                const uint32_t last = sh_last(config[u]);
                if (last != kNoSymbol) on[u] = sh_may_follow(a, L, prod(i[u]), last);
            }
        }
#pragma unroll
        for (int u = 0; u < kAhead; ++u) list(on[u], config[u], i[u]);
    }
    if (empties) {
        seen[lane] = kNoWord;
        seen[lane + 64] = kNoWord;
        static_assert(kShFrontier == 128, "as many configurations a set has at the most");
    }
    return m;
}

// One byte of Algorithm 1 on a whole set, by the whole wave: the number of the set that follows.  The listed pairs are
// carried out together, a lane each: the chain of LDS accesses is what this costs, and it is gone through once.
__device__ __forceinline__ uint32_t sh_step(const DisplacementArgs &a, SharedLds &L, uint32_t *work, uint32_t *seen,
                                            PoolRoom &room, uint32_t set, int number_of_byte, int lane) {
    const int m = sh_list_pairs(a, L, work, seen, set, number_of_byte, lane);
    // (the passes behind this one also find whether a bound is broken)
    if (m > kShFrontier) return kGiveUp;
    lds_order();
    uint32_t *pair_config = work, *pair_production = work + kShFrontier;
    bool full = false, crossed = false;
    auto carry_out = [&](int x) -> uint32_t {
        if (x >= m) return kNoWord;
        return sh_carry_out(a, L, pair_config[x], sh_end_cell(L, pair_config[x]), (int)pair_production[x], full, crossed);
    };
    uint32_t words[2] = {carry_out(lane), kNoWord};
    if (m > 64) words[1] = carry_out(lane + 64);
    if (__ballot(crossed)) return kCrossed;
    if (__ballot(full)) return kGiveUp;
    const Different<2> d = find_different<2>(seen, words, lane);
    sh_reserve(L, room, d.n, lane);
    const uint32_t number = sh_set_number(L, room, seen, d, lane);
    seen_clear(seen, lane);
    return number;
}

// The place of the k-th (from 0) of the bits that are set in `w`, which has more than k of them.
__device__ __forceinline__ int nth_bit(uint32_t w, int k) {
    int at = 0;
#pragma unroll
    for (int half = 16; half; half >>= 1) {
        const int below = __popc(w & ((1u << half) - 1u));
        const bool up = k >= below;
        k -= up ? below : 0;
        at += up ? half : 0;
        w = up ? w >> half : w;
    }
    return at;
}

// A set whose configurations the lanes hold, one each (kNoWord: none), with the cells that their ends are.
struct LaneSet {
    uint32_t word, cell;
};

// One byte of Algorithm 1 on such a set, where `pair` and `follow` are kept: the number of the set that follows, which the
// lanes then hold; kByTheWave, and nothing is done, if it takes more than 64 successors or a long body to make it.  Which
// productions apply to a configuration is one look-up of a bit for each of the byte's productions; the successors are dealt
// out to the lanes by a prefix sum of how many there are.  JSON call 237 -> 208 us, statement grammar 157 -> 143 with the sets' order by
// a word of their first symbols, 2,000 to 64,000 tokens with the JSON grammar 0.71 to 0.80 of the time.
__device__ __forceinline__ uint32_t sh_step_lanes(const DisplacementArgs &a, SharedLds &L, uint32_t *work, uint32_t *seen,
                                                  PoolRoom &room, LaneSet &set, uint32_t byte_number, uint32_t dead, int lane) {
    const uint32_t lo = L.follow[sh_follow_first(a, byte_number)];  // (the same for every lane)
    uint32_t may = 0;
    if (set.word != kNoWord) {
        if (sh_stack(set.word)) {
            const uint32_t e = L.pair[byte_number * (uint32_t)a.g.N + cell_symbol(set.cell)];
            may = ((1u << (e >> 10)) - 1u) << (((e & 0x3FFu) - lo) & 31u);
            may = e >> 10 == 32u ? ~0u : may;
        } else {
            may = L.follow[sh_follow(a, byte_number, sh_last(set.word))];
        }
    }
    uint4 *each = reinterpret_cast<uint4 *>(work);
    static_assert(sizeof(uint4) * 64 <= sizeof(uint32_t) * 2 * kShFrontier, "");
    const int count = __popc(may);
    const int upto = (int)wave_upto32((uint32_t)count), m = __builtin_amdgcn_readlane(upto, 63), first = upto - count;
    if (m > 64) return kByTheWave;
    if (!m) return dead;
    // a configuration that something applies to is put where its first successor comes to stand, and the lanes of those look
    // which it is
    each[lane].w = 0;
    lds_order();
    if (count) each[first] = make_uint4(set.word, set.cell, may, 1u);
    lds_order();
    const u64 begins = __ballot(each[lane].w != 0u);
    const int from = 63 - __clzll(begins & (~0ull >> (63 - lane)));  // (lane 0's begins)
    uint4 e = make_uint4(0, 0, 0, 0);
    u64 p = 0;
    if (lane < m) {
        e = each[from];
        p = L.prods[lo + nth_bit(e.z, lane - from)];
    }
    lds_order();
    // (a body of more than four symbols lies in memory, and what waits for that waits for the rows on their way there)
    if (__ballot(packed_length(p) == kLongBody)) return kByTheWave;
    uint32_t words[1] = {kNoWord};
    bool full = false, crossed = false;
    if (lane < m)
        words[0] = sh_carry_out(L, e.x, e.y, packed_head(p), (int)packed_length(p),
                                [&](int k) -> uint32_t { return packed_symbol(p, k); }, full, crossed);
    if (__ballot(crossed)) return kCrossed;
    if (__ballot(full)) return kGiveUp;
    const Different<1> d = find_different<1>(seen, words, lane);
    sh_reserve(L, room, d.n, lane);
    set.word = d.first[0] ? words[0] : kNoWord;
    set.cell = d.first[0] ? sh_end_cell(L, set.word) : 0u;
    const uint32_t number = sh_set_number(L, room, seen, d, lane);
    seen_clear(seen, lane);
    return number;
}
// The lanes take a set of up to 64 configurations.
__device__ __forceinline__ bool sh_load_set(const SharedLds &L, uint32_t number, LaneSet &set, int lane) {
    const u64 w = wave_read64(lds_look(&L.sets[number]), 0);
    lds_order();
    const int n = (int)set_size(w);
    set.word = kNoWord;
    set.cell = 0;
    if (n > 64) return false;
    if (lane < n) {
        set.word = L.pool[set_at(w) + lane];
        set.cell = sh_end_cell(L, set.word);
    }
    return true;
}

// Which of two different lists of one length comes first: queues (a cell holds the LAST symbol) ...
__device__ __forceinline__ bool queue_less(const SharedLds &L, uint32_t x, uint32_t y) {
    bool less = false;
    while (x != y) {  // the difference closest to the front decides
        const uint32_t a = lds_look(&L.cells[x - 1]), b = lds_look(&L.cells[y - 1]);
        if (cell_symbol(a) != cell_symbol(b)) less = cell_symbol(a) < cell_symbol(b);
        x = cell_rest(a);
        y = cell_rest(b);
    }
    return less;
}
// ... and stacks (a cell holds the FIRST symbol)
__device__ __forceinline__ bool stack_less(const SharedLds &L, uint32_t x, uint32_t y) {
    while (x != y) {
        const uint32_t a = lds_look(&L.cells[x - 1]), b = lds_look(&L.cells[y - 1]);
        if (cell_symbol(a) != cell_symbol(b)) return cell_symbol(a) < cell_symbol(b);
        x = cell_rest(a);
        y = cell_rest(b);
    }
    return false;
}

// What the set is written as: the row's entries and the hash, by the whole wave.  The canonical order is (length of the
// queue, of the stack), then the queue's and the stack's symbols, front first: one word of the two lengths and the first
// six and a half symbols is compared with everybody's, and only records that are alike so far are compared list by list.
__device__ __forceinline__ void sh_write_set(const DisplacementArgs &a, SharedLds &L, uint32_t *work, uint32_t *seen,
                                             uint32_t set, int lane) {
    const u64 w = wave_read64(lds_look(&L.sets[set]), 0);
    lds_order();
    int n = (int)set_size(w);
    // the displacement forgets the symbol consumed last
    constexpr uint32_t kPair = (1u << (2 * kCellIdBits)) - 1;
    const uint32_t *configs = L.pool + set_at(w);
    {
        const uint32_t pairs[2] = {lane < n ? configs[lane] & kPair : kNoWord,
                                   lane + 64 < n ? configs[lane + 64] & kPair : kNoWord};
        const Different<2> d = find_different<2>(seen, pairs, lane);
        n = d.n;
#pragma unroll
        for (int u = 0; u < 2; ++u)
            if (d.first[u]) work[d.at[u]] = d.word[u];
        seen_clear(seen, lane);
    }
    uint32_t mine[2], ni[2], no[2], start[2] = {1, 1}, total = 1;
    u64 key[2] = {0, 0};
    uint32_t q[2] = {0, 0}, t[2] = {0, 0};  // the lists' first cells
#pragma unroll
    for (int u = 0; u < 2; ++u) {
        mine[u] = ni[u] = no[u] = 0;
        if (64 * u >= n) break;  // the same for every lane
        mine[u] = lane + 64 * u < n ? work[lane + 64 * u] : 0u;
        if (sh_queue(mine[u])) q[u] = lds_look(&L.cells[sh_queue(mine[u]) - 1]);
        if (sh_stack(mine[u])) t[u] = lds_look(&L.cells[sh_stack(mine[u]) - 1]);
        ni[u] = cell_length(q[u]), no[u] = cell_length(t[u]);
    }
    lds_order();
    // The lists' symbols, front first: four of a lane's in a word, the words of all lanes behind each other.  (The records'
    // places are known only when all have been compared, and going through the lists a second time took as long as the first.)
    constexpr int kNotedWords = 2 * kShFrontier / 64;  // in `work`, and as many in `seen`
    static_assert(kNotedWords >= 2 && kNotedWords * 64 <= kShSeen, "");
    const bool noted = n <= 64 && __ballot(ni[0] + no[0] > 8u * kNotedWords) == 0ull;
    const bool past_work = __ballot(ni[0] + no[0] > 4u * kNotedWords) != 0ull;
    if (noted) {
        auto note = [&](uint32_t at, uint32_t symbol) {
            uint32_t *words = at < 4u * kNotedWords ? work : seen;
            reinterpret_cast<uint8_t *>(words)[((at / 4u) % kNotedWords) * 256u + (uint32_t)lane * 4u + at % 4u] = (uint8_t)symbol;
        };
        work[lane] = work[64 + lane] = 0;  // where the comparison looks
        lds_order();
        uint32_t qc = q[0], tc = t[0], at_q = ni[0], at_t = ni[0];
        while (qc | tc) {
            if (qc) note(--at_q, cell_symbol(qc));
            if (tc) note(at_t++, cell_symbol(tc));
            const uint32_t queue = cell_rest(qc), stack = cell_rest(tc);
            qc = queue ? lds_look(&L.cells[queue - 1]) : 0u;
            tc = stack ? lds_look(&L.cells[stack - 1]) : 0u;
        }
        lds_order();
        const uint32_t w0 = __builtin_bswap32(work[lane]), w1 = __builtin_bswap32(work[64 + lane]);
        key[0] = ((u64)ni[0] << 58) | ((u64)no[0] << 52) | ((((u64)w0 << 32) | w1) >> 12);
    } else {
#pragma unroll
        for (int u = 0; u < 2; ++u) {
            if (64 * u >= n) break;
            uint32_t queue, stack, qc = q[u], tc = t[u];
            u64 front = 0, behind = 0;  // the first eight symbols of the queue, of the stack
            int shift = 56;
            while (qc || (tc && shift >= 0)) {
                if (qc) front = (front >> 8) | ((u64)cell_symbol(qc) << 56);
                if (shift >= 0) behind |= (u64)cell_symbol(tc) << shift;
                shift -= 8;
                queue = cell_rest(qc);
                stack = cell_rest(tc);
                qc = queue ? lds_look(&L.cells[queue - 1]) : 0u;
                tc = stack && shift >= 0 ? lds_look(&L.cells[stack - 1]) : 0u;
            }
            if (ni[u] < 8) front |= behind >> (8 * ni[u]);
            key[u] = ((u64)ni[u] << 58) | ((u64)no[u] << 52) | (front >> 12);
        }
    }
    static_assert(kShMaxList < 64, "a length fits six bits");
    auto entries_of = [](u64 k) -> uint32_t { return 2u + (uint32_t)(k >> 58) + ((uint32_t)(k >> 52) & 63u); };
    if (n == 1) total += 2u + wave_read(ni[0], 0) + wave_read(no[0], 0);
    for (int j = 0; n > 1 && j < n; ++j) {
        const u64 other = j < 64 ? wave_read64(key[0], j) : wave_read64(key[1], j - 64);
        const uint32_t entries = entries_of(other);
        start[0] += other < key[0] ? entries : 0u;
        if (n > 64) start[1] += other < key[1] ? entries : 0u;
        total += entries;
    }
    uint32_t result;
    if (total > (uint32_t)a.row_len) {
        result = kRowTooLong;
    } else {
        const uint32_t room = (total + 7u) & ~7u;  // whole 16-byte units, zeros behind the entries
        uint32_t at = 0;
        if (lane == 0) at = atomicAdd(&L.out_top, room);
        at = __builtin_amdgcn_readfirstlane(at);
        if (at + room > (uint32_t)kShOut) {
            result = kRowGiveUp;
        } else {
            // records that are alike so far have come to the same place
            bool tie = false;
#pragma unroll
            for (int u = 0; u < 2; ++u)
                if (lane + 64 * u < n && n > 1) L.out[at + start[u]] = (uint16_t)(lane + 64 * u);
            lds_order();
#pragma unroll
            for (int u = 0; u < 2; ++u)
                if (lane + 64 * u < n && n > 1) tie = tie || L.out[at + start[u]] != (uint16_t)(lane + 64 * u);
            lds_order();
            if (__ballot(tie)) {
                for (int j = 0; j < n; ++j) {
                    const u64 other = j < 64 ? wave_read64(key[0], j) : wave_read64(key[1], j - 64);
                    const uint32_t c = j < 64 ? wave_read(mine[0], j) : wave_read(mine[1], j - 64);
#pragma unroll
                    for (int u = 0; u < 2; ++u)
                        if (lane + 64 * u < n && other == key[u] && c != mine[u] &&
                            (sh_queue(c) != sh_queue(mine[u]) ? queue_less(L, sh_queue(c), sh_queue(mine[u]))
                                                              : stack_less(L, sh_stack(c), sh_stack(mine[u]))))
                            start[u] += entries_of(other);
                }
            }
            if (lane == 0) L.out[at] = (uint16_t)n;
            if (lane < 8 && total + lane < room) L.out[at + total + lane] = 0;
            u64 h = 0;
            if (noted) {
                if (lane < n) {
                    uint16_t *rec = L.out + at + start[0];
                    rec[0] = (uint16_t)ni[0];
                    rec[1] = (uint16_t)no[0];
                    const uint32_t symbols = ni[0] + no[0];
                    RecordMix mix(a.seed);
                    mix.add(ni[0]);
                    mix.add(no[0]);
#pragma unroll 1
                    for (uint32_t k0 = 0; k0 < symbols; k0 += 4) {
                        const uint32_t *words = k0 < 4u * kNotedWords ? work : seen;
                        const uint32_t four = words[((k0 / 4u) % kNotedWords) * 64u + (uint32_t)lane];
#pragma unroll
                        for (uint32_t k = 0; k < 4; ++k) {
                            const uint32_t symbol = (four >> (8 * k)) & 0xFFu;
                            if (k0 + k < symbols) {
                                rec[2 + k0 + k] = (uint16_t)symbol;
                                mix.add(symbol);
                            }
                        }
                    }
                    h = mix.done();
                }
            } else {
#pragma unroll
                for (int u = 0; u < 2; ++u) {
                    if (lane + 64 * u >= n) continue;
                    uint16_t *rec = L.out + at + start[u];
                    rec[0] = (uint16_t)ni[u];
                    rec[1] = (uint16_t)no[u];
                    uint32_t queue = sh_queue(mine[u]), stack = sh_stack(mine[u]);
                    for (int k = 0; queue || stack; ++k) {
                        const uint32_t q = queue ? lds_look(&L.cells[queue - 1]) : 0u;
                        const uint32_t s = stack ? lds_look(&L.cells[stack - 1]) : 0u;
                        if (queue) rec[1 + (int)ni[u] - k] = (uint16_t)cell_symbol(q);
                        if (stack) rec[2 + (int)ni[u] + k] = (uint16_t)cell_symbol(s);
                        queue = cell_rest(q);
                        stack = cell_rest(s);
                    }
                    lds_order();
                    RecordMix mix(a.seed);
                    const int length = 2 + (int)ni[u] + (int)no[u];
                    constexpr int kAhead = 8;  // reads that wait for nothing
                    for (int k0 = 0; k0 < length; k0 += kAhead) {
                        uint32_t x[kAhead];
#pragma unroll
                        for (int k = 0; k < kAhead; ++k) x[k] = rec[min(k0 + k, length - 1)];
#pragma unroll
                        for (int k = 0; k < kAhead; ++k)
                            if (k0 + k < length) mix.add(x[k]);
                    }
                    h += mix.done();
                }
            }
            h = wave_sum64(h);
            if (lane == 0) L.row_hash[set] = h;
            result = ((at / 8u) << kRowBits) | total;
        }
    }
    if (noted && past_work) seen_clear(seen, lane);
    lds_order();
    if (lane == 0) __hip_atomic_store(&L.row[set], result, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
}

// A workgroup takes `per_group` consecutive tokens, the longest first: what a token of 25 bytes needs, set after set that
// nobody has met, is a chain that nothing shortens, and begun last it is what the workgroup waits for.  The lanes of a wave
// hold tokens in all stages.  The wave works out a step that one of them waits for, of the token with most bytes to go, and
// the steps behind it; if there is none, writes the rows of those that are through; if none is, takes more tokens; and waits
// only if there are none left.
template <bool ROWS16>  // rows start at multiples of 16 bytes
__global__ __launch_bounds__(kShThreads) CFGZIP_OWN_PAGES void displacement_shared_kernel(DisplacementArgs a, int per_group) {
    __shared__ SharedLds L;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int64_t group0 = (int64_t)blockIdx.x * per_group;
    const int in_group = (int)min((int64_t)per_group, (int64_t)a.V - group0);
    // a batch of tokens, and the thread's share of their bytes: the first is asked for before the tables are set up
    int64_t from_byte = 0, bytes_here = 0, begins = 0, ends = 0;
    constexpr int kShare = kShBytes / kShThreads;
    static_assert(kShBytes % kShThreads == 0, "");
    uint8_t share[kShare];
    int batch_size = 0;
    auto fetch = [&](int batch0) {
        const int64_t first_token = group0 + batch0;
        const int in_batch = min(in_group - batch0, kShBatch);
        batch_size = in_batch;
        from_byte = a.tok_off[first_token];
        bytes_here = a.tok_off[first_token + in_batch] - from_byte;
        begins = a.tok_off[first_token + min(tid, in_batch - 1)] - from_byte;
        ends = a.tok_off[first_token + min(tid, in_batch - 1) + 1] - from_byte;
#pragma unroll
        for (int k = 0; k < kShare; ++k) {
            const int x = tid + k * kShThreads;
            share[k] = 0;
            if (bytes_here <= kShBytes && x < bytes_here) share[k] = a.tok_bytes[from_byte + x];
        }
    };
    // the tables, an entry each: asked for before anything that was asked for is waited for (of an invalid grammar they hold
    // anything, and nothing looks at them)
    const int relation_words = a.g.N * a.g.W;
    int32_t invalid_there = a.hdr->invalid;
    uint32_t like = a.byte_like[tid & 255], first_of_byte = (uint32_t)a.byte_off[min(tid, 256)], relation = 0;
    uint32_t byte_of = 0;
    u64 production = 0;
    static_assert(kShProds <= kShThreads && kShAdj <= kShThreads, "an entry each");
    if (a.g.P <= kShProds) {
        production = a.prod_packed[min(tid, a.g.P - 1)];
        byte_of = a.g.byte[min(tid, a.g.P - 1)];
    }
    if (relation_words <= kShAdj) relation = a.adj[min(tid, relation_words - 1)];
    fetch(0);
    const bool invalid = invalid_there != 0;  // the same for everybody
    const bool sorted = in_group > kShOnce * kShWaves;  // otherwise every wave takes its tokens at once
    // sorting a batch: four parts with a barrier between them
    uint32_t shorter = 0, rank = 0;
    auto fit = [&]() { return bytes_here >= 0 && bytes_here <= kShBytes; };
    auto clear_batch = [&]() {
        if (tid == 0) L.cursor = L.scattered = 0;
        if (tid < kShLengths) L.of_length[tid] = 0;
    };
    auto count_lengths = [&]() {
        if (invalid) from_byte = bytes_here = begins = ends = 0;
        if (tid < batch_size) {
            // a number that is smaller for longer ones
            shorter = (uint32_t)(kShLengths - 1 - min(max(ends - begins, (int64_t)0), (int64_t)kShLengths - 1));
            if (sorted) rank = atomicAdd(&L.of_length[shorter], 1u);
            if (begins < 0 || ends < begins || ends > bytes_here) L.scattered = 1;
        }
    };
    auto stage_bytes = [&]() {
        if (fit())
#pragma unroll
            for (int k = 0; k < kShare; ++k)
                if (tid + k * kShThreads < bytes_here) L.bytes[tid + k * kShThreads] = L.byte_number[share[k]];
    };
    auto sum_lengths = [&]() {
        if (!sorted || wave != 0) return;
        const uint32_t count = L.of_length[lane];
        L.of_length[lane] = wave_upto32(count) - count;
    };
    auto put_in_order = [&]() {
        if (tid >= batch_size) return;
        L.order[sorted ? L.of_length[shorter] + rank : (uint32_t)tid] = (uint16_t)tid;
        if (fit() && L.scattered == 0) {
            L.start[tid] = (uint16_t)begins;
            L.start[tid + 1] = (uint16_t)ends;  // (where the next one begins: the same value from both)
        }
    };
    for (int i = tid; i < kShCells; i += kShThreads) L.cells[i] = 0;
    for (int i = tid; i < kShNext; i += kShThreads) L.next[i] = kNextEmpty;
    for (int i = tid; i < kShSets; i += kShThreads) {
        L.sets[i] = kShEmpty;
        L.row[i] = kRowUnknown;
    }
    if (tid < 257) L.byte_off[tid] = first_of_byte;
    if (tid < a.g.P && a.g.P <= kShProds) L.prods[tid] = production;
    if (tid < relation_words && relation_words <= kShAdj) L.adj[tid] = relation;
    {
        const u64 own = __ballot(!invalid && (int)like == tid);  // bytes that are their own like
        if (wave < 4 && lane == 0) {
            L.own[2 * wave] = (uint32_t)own;
            L.own[2 * wave + 1] = (uint32_t)(own >> 32);
        }
    }
    for (int i = tid; i < kShPairs; i += kShThreads) L.pair[i] = 0;
    if (tid == 0) {
        L.pool_top = 0;
        L.out_top = 0;
        L.few_each = 1;
        L.follow_kept = 0;
    }
    uint32_t *work = L.work[wave], *seen = L.seen[wave];
    seen_clear(seen, lane);
    clear_batch();
    __syncthreads();
    count_lengths();
    PoolRoom room = {0, 0, false};
    if (wave == kShWaves - 1) {
        // the start set: nothing consumed, nothing pushed; and the set that no configuration is left in (there is room
        // for these two: they are the first)
        const uint32_t one[1] = {lane == 0 ? sh_config(0, 0, kNoSymbol) : kNoWord}, none[1] = {kNoWord};
        sh_reserve(L, room, 1, lane);
        const uint32_t first = sh_set_number(L, room, seen, find_different<1>(seen, one, lane), lane);
        seen_clear(seen, lane);
        const uint32_t second = sh_set_number(L, room, seen, find_different<1>(seen, none, lane), lane);
        if (lane == 0) {
            L.start_set = first;
            L.dead_set = second;
        }
    }
    // the productions of a (byte, symbol) lie behind each other: where, if all of this fits
    int own = 0;
    for (int w = 0; w < 8; ++w) own += __popc(L.own[w]);
    const bool fits = !invalid && a.g.P <= kShProds && own * a.g.N <= kShPairs;
    if (tid == 0) L.pairs_kept = fits ? 1u : 0u;
    if (tid < 256) {
        int number = 0;
        for (int w = 0; w < (int)(like >> 5); ++w) number += __popc(L.own[w]);
        number += __popc(L.own[like >> 5] & ((1u << (like & 31)) - 1u));
        L.byte_number[tid] = (uint8_t)number;
        if ((int)like == tid) {
            L.like_of[number] = (uint8_t)tid;
            if (fits && L.byte_off[tid + 1] - L.byte_off[tid] > (uint32_t)kShFew) L.few_each = 0;
        }
    }
    __syncthreads();
    sum_lengths();
    if (fits && tid < a.g.P && ((L.own[byte_of >> 5] >> (byte_of & 31)) & 1u)) {
        const int i = tid, lo = (int)L.byte_off[byte_of], hi = (int)L.byte_off[byte_of + 1];
        const uint32_t head = packed_head(production);
        if (i == lo || packed_head(L.prods[i - 1]) != head) {
            if (i + 63 < hi && packed_head(L.prods[i + 63]) == head) {  // more than six bits say
                L.pairs_kept = 0;  // (not counted out: of one pair's 676 productions that took 50 us)
            } else {
                int end = i + 1;
                while (end < hi && packed_head(L.prods[end]) == head) ++end;
                L.pair[L.byte_number[byte_of] * (uint32_t)a.g.N + head] = (uint16_t)(i | ((end - i) << 10));
            }
        }
    }
    stage_bytes();
    // which of a byte's productions may come right after a symbol: where this fits it takes the relation's place
    const int follows = fits && L.few_each && own * (a.g.N + 2) <= kShFollow && relation_words <= kShAdj ? own * (a.g.N + 2) : 0;
    constexpr int kFollowEach = kShFollow / kShThreads;
    uint32_t may[kFollowEach];
#pragma unroll
    for (int u = 0; u < kFollowEach; ++u) {
        const int x = tid + u * kShThreads;
        may[u] = 0;
        if (x >= follows) continue;
        const int number = x / (a.g.N + 2), last = x - number * (a.g.N + 2), b = (int)L.like_of[number];
        const int lo = (int)L.byte_off[b], count = last <= a.g.N ? min((int)L.byte_off[b + 1] - lo, kShFew) : 0;
        for (int k = 0; k < count; ++k)
            if (last == a.g.N || sh_may_follow(a, L, L.prods[lo + k], (uint32_t)last)) may[u] |= 1u << k;
        if (last > a.g.N) may[u] = (uint32_t)lo;
    }
    __syncthreads();
    put_in_order();
    const bool follow_kept = follows && L.pairs_kept;  // the same for everybody
    if (follow_kept) {
#pragma unroll
        for (int u = 0; u < kFollowEach; ++u)
            if (tid + u * kShThreads < follows) L.follow[tid + u * kShThreads] = may[u];
        if (tid == 0) L.follow_kept = 1;
    }
    __syncthreads();
    const uint32_t start = __builtin_amdgcn_readfirstlane(L.start_set), dead = __builtin_amdgcn_readfirstlane(L.dead_set);

    int steps = 0;  // that this wave has worked out
    for (int batch0 = 0; batch0 < in_group; batch0 += kShBatch) {
        const int64_t first_token = group0 + batch0;
        const int in_batch = min(in_group - batch0, kShBatch);
        if (batch0) {  // (the first has been sorted while the tables were set up)
            __syncthreads();  // the last batch is done with
            fetch(batch0);
            clear_batch();
            __syncthreads();
            count_lengths();
            stage_bytes();
            __syncthreads();
            sum_lengths();
            __syncthreads();
            put_in_order();
            __syncthreads();
        }
        const bool staged = fit() && L.scattered == 0;
        // (the address is kept: loaded with the other arguments at each byte it was a trip to memory in front of another one,
        // 2,000 strings of 400 bytes over the JSON grammar 241 us a call, 225 so)
        const uint8_t *text = a.tok_bytes + from_byte;
        auto byte_at = [&](int64_t p) -> uint32_t { return staged ? (uint32_t)lds_look(&L.bytes[p]) : (uint32_t)L.byte_number[text[p]]; };

        // the lane's token
        int token = -1;                         // its number in the batch, -1: none
        int64_t pos = 0, end = 0;               // its bytes from here on
        uint32_t set = start, like = 0, after = 0;  // where it is, the next byte and the one behind it
        bool give_up = false, crossed = false;
        bool by_the_wave = false;               // the next step has turned out to take a whole wave
        uint32_t row = kRowUnknown;
        // how many the wave takes next: of sorted ones the longest one by one, else all that are its
        int take = sorted ? 1 : (in_group + kShWaves - 1) / kShWaves;
        bool more = true;
        for (;;) {
            __builtin_amdgcn_wave_barrier();  // the wave goes round together: no branch on the lane is joined with the next one
            // every lane as far as what follows is known
            uint32_t waits = 0;  // kNextEmpty or kWorkedOut: what the lane has come to
            auto advance = [&](uint32_t following) {
                if (following >= kCrossed) {
                    give_up = following == kGiveUp;
                    crossed = following == kCrossed;
                    pos = end;
                } else {
                    set = following;
                    by_the_wave = false;
                    like = after;
                    if (++pos + 1 < end) after = byte_at(pos + 1);
                }
            };
            while (pos < end && !waits) {
                if (set == dead) {  // so it stays
                    pos = end;
                    break;
                }
                const uint32_t following = sh_known(L, set, like);
                if (following == kNextEmpty || following == kWorkedOut) waits = following;
                else advance(following);
            }
            // where the tokens share few sets: what follows by the lanes alone, as far as it is simple
            const bool alone = waits == kNextEmpty && !by_the_wave && steps > kShShared;
            if (__ballot(alone)) {
                if (alone) {
                    const uint32_t following = sh_step_alone(sh_arguments(), L, set, like, dead);
                    if (following == kByTheWave) {
                        by_the_wave = true;
                    } else {
                        sh_publish(L, set, like, following);
                        waits = 0;
                        advance(following);
                    }
                }
                if (__ballot(alone && !by_the_wave)) continue;
            }
            if (__ballot(waits == kNextEmpty)) {
                // by the whole wave what the lane with most bytes to go waits for
                const uint32_t to_go = (uint32_t)min(end - pos, (int64_t)0xFFFFFF);
                const uint32_t key = waits == kNextEmpty ? (to_go << 6) | (uint32_t)(lane ^ 63) : 0u;
                const int chosen = sorted ? (int)(wave_max32(key) & 63u) ^ 63
                                          : __ffsll(__ballot(waits == kNextEmpty)) - 1;
                uint32_t from = wave_read(set, chosen), on = wave_read(like, chosen);
                // Before the waves that look things up or wait for this one: calls of 20,000 to 64,000 tokens 2 to 4 % (statement
                // grammar, 32,000 tokens, with classes 115.8 -> 112.7 us); also where sets are written out: no more.
                __builtin_amdgcn_s_setprio(2);
                LaneSet held;
                bool holds = false;  // the lanes have the set's configurations
                for (;;) {
                    int slot = 0;
                    if (lane == 0) slot = sh_claim(L, from, on);
                    slot = __builtin_amdgcn_readfirstlane(slot);
                    if (slot == -1) break;  // known, or taken meanwhile
                    if (follow_kept && !holds) holds = sh_load_set(L, from, held, lane);
                    uint32_t following = kByTheWave;
                    if (holds) following = sh_step_lanes(a, L, work, seen, room, held, on, dead, lane);
                    if (following == kByTheWave) {
                        holds = false;
                        following = sh_step(sh_arguments(), L, work, seen, room, from, (int)on, lane);
                    }
                    ++steps;
                    lds_order();
                    if (slot >= 0 && lane == 0)
                        __hip_atomic_store(&L.next[slot], (((from << 8) | on) << kNextBits) | following, __ATOMIC_RELAXED,
                                           __HIP_MEMORY_SCOPE_WORKGROUP);
                    if (pos < end && set == from && like == on) advance(following);
                    // The token's next byte right away: where a token makes set after set that nobody has met, that chain
                    // is what the workgroup waits for
                    if (!((__ballot(pos < end) >> chosen) & 1ull) || following == dead) break;
                    from = following;
                    on = wave_read(like, chosen);
                }
                __builtin_amdgcn_s_setprio(0);
                continue;
            }
            // What the sets reached are written as.
            bool through = token >= 0 && pos >= end;
            const bool wanted = through && !invalid && !give_up && !crossed;
            for (;;) {
                if (wanted && (row == kRowUnknown || row == kRowWorkedOut)) row = lds_look(&L.row[set]);
                const u64 unknown = __ballot(wanted && row == kRowUnknown);
                if (!unknown) break;
                const uint32_t s = wave_read(set, __ffsll(unknown) - 1);
                uint32_t state = 0;
                if (lane == 0) state = atomicCAS(&L.row[s], kRowUnknown, kRowWorkedOut);
                if (wave_read(state, 0) == kRowUnknown) sh_write_set(sh_arguments(), L, work, seen, s, lane);
            }
            if (wanted && row == kRowWorkedOut) through = false;  // another wave is at it
            if (__ballot(through)) {
                const DisplacementArgs a = sh_arguments();
                lds_order();
                const int64_t t = first_token + token;
                if (wanted && row == kRowGiveUp) give_up = true;
                if (wanted && row == kRowTooLong) crossed = true;
                const bool done = through && !give_up;
                if (done) {
                    u64 h = 0;
                    int32_t status = kStatusOk;
                    if (invalid) {
                        status = kStatusBadGrammar;
                    } else if (crossed) {
                        h = overflow_hash(a.seed, (int)t);
                        status = kStatusOverflow;
                    } else {
                        h = L.row_hash[set];
                    }
                    a.hash[t] = h;
                    if (a.status) a.status[t] = status;
                }
                const u64 handed = __ballot(through && give_up);
                if (handed) {
                    int32_t at = 0;
                    if (lane == 0) at = (int32_t)atomicAdd(&a.hdr->retry_count[0], (int32_t)__popcll(handed));
                    at = __builtin_amdgcn_readfirstlane(at);
                    if (through && give_up)
                        a.retry_list[0][at + __popcll(handed & ((1ull << lane) - 1ull))] = (int32_t)t;
                }
                // the rows, one after the other by the whole wave
                const u64 plain = __ballot(done && !invalid && !crossed);
                for (u64 left = __ballot(done); left; left &= left - 1) {
                    const int k = __ffsll(left) - 1;
                    const int64_t tk = first_token + (int)wave_read((uint32_t)token, k);
                    uint16_t *out_row = a.rows + (size_t)tk * a.row_len;
                    const bool copy = (plain >> k) & 1ull;
                    const uint32_t rk = wave_read(row, k);
                    const uint32_t units = copy ? (row_entries(rk) + 7u) / 8u : 0u;  // 16 bytes each
                    const uint4 *src = reinterpret_cast<const uint4 *>(L.out + (copy ? row_at(rk) : 0u));
                    const bool marked = !copy && !invalid;  // the row of a token that overflowed
                    for (uint32_t u = lane; u < (uint32_t)a.row_len / 8u; u += 64) {
                        uint4 v = make_uint4(0, 0, 0, 0);
                        if (u < units) v = src[u];
                        if (marked && u == 0) v = make_uint4(0xFFFFu | ((uint32_t)tk << 16), (uint32_t)tk >> 16, 0, 0);
                        if (ROWS16) {
                            reinterpret_cast<uint4 *>(out_row)[u] = v;
                        } else {
                            reinterpret_cast<uint2 *>(out_row)[2 * u] = make_uint2(v.x, v.y);
                            reinterpret_cast<uint2 *>(out_row)[2 * u + 1] = make_uint2(v.z, v.w);
                        }
                    }
                }
                if (through) token = -1;
                continue;
            }
            const u64 idle = __ballot(token < 0);
            if (more && idle) {
                const int want = min(take, (int)__popcll(idle));
                int taken = 0;
                if (lane == 0) taken = (int)atomicAdd(&L.cursor, (uint32_t)want);
                taken = __builtin_amdgcn_readfirstlane(taken);
                const int count = min(want, in_batch - taken);
                more = sorted && count > 0;  // (else the wave has had all that is its)
                const int rank_idle = (int)__popcll(idle & ((1ull << lane) - 1ull));
                if (token < 0 && rank_idle < count) {
                    token = (int)L.order[taken + rank_idle];
                    if (staged) {
                        pos = L.start[token];
                        end = L.start[token + 1];
                    } else {
                        pos = end = 0;
                        if (!invalid) {
                            const DisplacementArgs a = sh_arguments();
                            pos = a.tok_off[first_token + token] - from_byte;
                            end = a.tok_off[first_token + token + 1] - from_byte;
                        }
                    }
                    set = start;
                    give_up = crossed = by_the_wave = false;
                    row = kRowUnknown;
                    if (pos < end) like = byte_at(pos);
                    if (pos + 1 < end) after = byte_at(pos + 1);
                }
                take = min(2 * take, in_group > kShFewTokens ? kShTakeMost : kShTakeFew);
                continue;
            }
            if (idle == ~0ull) break;
            __builtin_amdgcn_s_sleep(2);  // another wave is at all that is left; it waits for nothing while it works
        }
    }
}

}  // namespace
}  // namespace cfgzip
