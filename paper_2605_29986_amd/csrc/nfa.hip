// Signatures over a non-deterministic byte automaton (paper Section 3.2.1 for a right-linear grammar with
// several productions q -> a q' per state and byte).  The displacement of token t is then the relation
// R_t = {(q, q') : q' reachable from q on bytes(t)}, the boolean product of the per-byte transition relations; it is
// kept as one bit row per start state.
//
// Start states that the first byte sends to the same set of states have the same row for the whole token, and a
// lexer's bytes leave few different sets (about 30 of 256 states).  Up to 256 states a wave therefore walks its token
// from the different successor sets of the first byte only, a lane each, and every start state's row is a copy of its
// set's (the image walk of the deterministic case).  A set is W words in registers; per byte the successor rows of
// its members are ORed together, so the cost follows the size of the sets and not S.  Up to 64 states, and with few
// pairs of token and state, a thread takes a pair instead (kWalkPairs).  Automata of more than 256 states
// (up to 1,024) walk from every state and keep the sets in LDS.  The 64-bit hash is the same multilinear form as for
// the byte walk, over the relation read as 16-bit entries, so any split over threads gives the same bits.

#include <algorithm>

#include "common.hpp"
#include "walk_device.hpp"  // splitmix64_at: the multipliers of the signature hash

namespace cfgzip {
namespace {

constexpr int kThreads = 256;
constexpr int kMaxRegisterStates = 256;  // up to here a thread keeps its set in registers
constexpr int kMaxNfaStates = 1024;
constexpr int kStagedBytes = 64;  // token bytes read once into LDS by nfa_walk_kernel; longer tokens go on from memory

struct NfaArgs {
    const uint8_t *tok_bytes;
    const int64_t *tok_off;
    const uint32_t *nfa;  // [256][S][W]
    uint32_t *rel;        // [V][S][W]
    uint64_t *hash;       // [V] or null
    uint64_t seed;
    int V, S;
    uint32_t last_word_mask;  // the bits of a row's last word that are states
};

// Up to here a thread per (token, start state) is faster than walking from the different successor sets only.  It fills
// the chip (524,288 threads) less than twice, so what counts is the chain of a token, and telling sets apart comes on
// top: lexers of 96 / 128 / 200 / 256 states with 4,000 tokens 30 / 32 / 44 / 48 us against 33 / 35 / 46 / 46, with
// 1,000 tokens 28 / 28 / 33 / 34 against 32 / 34 / 44 / 43; with 32,000 tokens 73 / 83 / 151 / 167 against 63 / 66 /
// 108 / 104.  With up to 64 states a wave has all of a token's states in its lanes, and walking fewer saves nothing: 24
// states 38 us against 42, 64 states 51 against 55 (32,000 tokens).
constexpr int64_t kWalkPairs = 7 << 17;
constexpr int kWalkStates = 64;

constexpr int kImageThreads = 1024;
constexpr int kImageWaves = kImageThreads / 64;
constexpr int kImageSets = 96;           // different successor sets of a byte that the walk shares
constexpr int kImageSlots = 512;         // slots of the table in which a byte's sets are told apart (256 states at most)
constexpr int kImageBytes = 64;          // first bytes that a workgroup keeps the sets of
constexpr int kImageGroup = 96;          // tokens of a workgroup at the most; those that begin with a byte beyond the
                                         // kImageBytes first met are walked from every state
constexpr uint32_t kImageUnknown = 0, kImageWorkedOut = 1, kImageMany = 2;  // ready: how many in bits 8.., the slot below

template <int W>
struct ImageLds {
    // per wave: the sets its token's walk has come to, and what the hash needs of them; while a byte's sets are told
    // apart, the table for that and the numbers of the states that stand for a set
    static constexpr int kSetWords = kImageSets * W > kImageSlots + 64 ? kImageSets * W : kImageSlots + 64;
    __align__(16) uint32_t sets[kImageWaves][kSetWords];
    uint32_t members[kImageWaves][kImageSets];  // how many, and the first and the last of them
    uint32_t state[256];                        // per byte: whether and where the two tables below have it
    uint32_t cursor, slots;
    // where the waves share out the tokens that every state walks for itself: which tokens, how many, of how many tokens
    // it is known whether they are one; per token the hash so far and the chunks done
    uint32_t alone[kImageWaves], alones, known, done[kImageWaves];
    unsigned long long hash[kImageWaves];
    uint8_t set_of[kImageBytes][256];           // [slot][start state]: number of its successor set
    uint8_t first_with[kImageBytes][kImageSets];  // [slot][set]: the first state that has it
};

// How many members a set has, the first and the last.
template <int W>
__device__ __forceinline__ void set_members(const uint32_t (&set)[W], uint32_t &count, uint32_t &first, uint32_t &last) {
    count = 0, first = 0, last = 0;
#pragma unroll
    for (int w = 0; w < W; ++w) count += __popc(set[w]);
#pragma unroll
    for (int w = W - 1; w >= 0; --w) first = set[w] ? 32u * w + (uint32_t)__ffs(set[w]) - 1u : first;
#pragma unroll
    for (int w = 0; w < W; ++w) last = set[w] ? 32u * w + 31u - (uint32_t)__clz(set[w]) : last;
}

template <int W>
__device__ __forceinline__ void add_row(uint32_t (&set)[W], const uint32_t *row) {
    if (W % 4 == 0) {  // rows are whole 16-byte units (the base is 16-byte aligned)
#pragma unroll
        for (int k = 0; k < W / 4; ++k) {
            const uint4 v = reinterpret_cast<const uint4 *>(row)[k];
            set[4 * k] |= v.x;
            set[4 * k + 1] |= v.y;
            set[4 * k + 2] |= v.z;
            set[4 * k + 3] |= v.w;
        }
    } else {
#pragma unroll
        for (int k = 0; k < W; ++k) set[k] |= row[k];
    }
}

template <int W>
__device__ __forceinline__ void store_set(uint32_t *row, const uint32_t (&set)[W]) {
    if (W % 4 == 0) {
#pragma unroll
        for (int k = 0; k < W / 4; ++k)
            reinterpret_cast<uint4 *>(row)[k] = make_uint4(set[4 * k], set[4 * k + 1], set[4 * k + 2], set[4 * k + 3]);
    } else {
#pragma unroll
        for (int w = 0; w < W; ++w) row[w] = set[w];
    }
}

// One byte: the union of the successor rows of the members.  One or two members, as a lexer's sets have, are found
// without going through the words.
template <int W>
__device__ __forceinline__ void set_step(uint32_t (&set)[W], const uint32_t *step, uint32_t last_word_mask) {
    uint32_t count, first, last;
    set_members<W>(set, count, first, last);
    uint32_t next[W];
#pragma unroll
    for (int w = 0; w < W; ++w) next[w] = 0;
    if (count) add_row<W>(next, step + first * W);
    if (count > 1) add_row<W>(next, step + last * W);
    if (count > 2) {
#pragma unroll
        for (int w = 0; w < W; ++w)
            for (uint32_t bits = set[w]; bits; bits &= bits - 1) add_row<W>(next, step + (w * 32 + __ffs(bits) - 1) * W);
    }
    next[W - 1] &= last_word_mask;  // a stray pad bit must not become a state number
#pragma unroll
    for (int w = 0; w < W; ++w) set[w] = next[w];
}

// The bytes of a token, 64 at a time in the lanes of the wave.
struct WaveBytes {
    const uint8_t *bytes;
    int64_t beg, end, chunk;
    uint32_t mine;
    __device__ WaveBytes(const uint8_t *tok_bytes, int64_t b0, int64_t b1) : bytes(tok_bytes), beg(b0), end(b1), chunk(b0) { load(); }
    __device__ void load() {
        const int64_t p = chunk + (threadIdx.x & 63);
        mine = p < end ? bytes[p] : 0u;
    }
    __device__ int at(int64_t p) {  // p does not decrease from call to call
        if (p >= chunk + 64) {
            chunk = p;
            load();
        }
        return (int)__builtin_amdgcn_readlane(mine, (int)(p - chunk));
    }
};

// A row's part of the hash: the terms of empty words are zero.
template <int W>
__device__ __forceinline__ uint64_t row_hash(const uint32_t (&set)[W], int q, uint64_t seed) {
    uint64_t h = 0;
#pragma unroll
    for (int w = 0; w < W; ++w) {
        if (set[w]) {
            const uint32_t e = 2u * (uint32_t)(q * W + w);  // 16-bit entries 2(qW+w), 2(qW+w)+1
            if (set[w] & 0xFFFFu) h += (splitmix64_at(seed, e) | 1ull) * (uint64_t)(set[w] & 0xFFFFu);
            if (set[w] >> 16) h += (splitmix64_at(seed, e + 1u) | 1ull) * (uint64_t)(set[w] >> 16);
        }
    }
    return h;
}
// The same for a set of one member y: its bit's place in the entry y / 16 of the row.
__device__ __forceinline__ uint64_t member_hash(uint32_t q, uint32_t W, uint32_t y, uint64_t seed) {
    return (splitmix64_at(seed, 2u * W * q + (y >> 4)) | 1ull) << (y & 15u);
}

__device__ __forceinline__ void lds_order() { __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "workgroup"); }

// Tells the successor sets of byte b apart, by the whole wave: numbers them by the first state that has them.  Returns
// the byte's state.
template <int W>
__device__ __forceinline__ uint32_t number_sets(const NfaArgs &a, ImageLds<W> &L, uint32_t *scratch, int b) {
    const int lane = threadIdx.x & 63;
    int slot = 0;
    if (lane == 0) slot = (int)atomicAdd(&L.slots, 1u);
    slot = __builtin_amdgcn_readfirstlane(slot);
    if (slot >= kImageBytes) return kImageMany;
    uint32_t *table = scratch;                                                // [kImageSlots]: hash above the state
    uint8_t *number = reinterpret_cast<uint8_t *>(scratch + kImageSlots);     // [256]
    for (int i = lane; i < kImageSlots; i += 64) table[i] = ~0u;
    lds_order();
    const uint32_t *step = a.nfa + (size_t)b * a.S * W;
    uint32_t n = 0;
    uint32_t ahead[W];  // the next states' rows, on their way while these are told apart
#pragma unroll
    for (int w = 0; w < W; ++w) ahead[w] = 0;
    if (lane < a.S) add_row<W>(ahead, step + (size_t)lane * W);
    for (int q0 = 0; q0 < a.S; q0 += 64) {
        const int q = q0 + lane;
        const bool in = q < a.S;
        uint32_t row[W];
#pragma unroll
        for (int w = 0; w < W; ++w) {
            row[w] = ahead[w];
            ahead[w] = 0;
        }
        if (q + 64 < a.S) add_row<W>(ahead, step + (size_t)(q + 64) * W);
        uint32_t h = 0;
#pragma unroll
        for (int w = 0; w < W; ++w) h = (h ^ row[w]) * 0x9E3779B1u + (h >> 15);
        h = (h ^ (h >> 13)) & 0x7FFFFFFFu;  // so that no entry looks like an empty slot
        int like = q;
        if (in) {
            uint32_t at = h % kImageSlots;
            for (int probe = 0; probe < kImageSlots; ++probe, at = (at + 1) % kImageSlots) {
                const uint32_t seen = atomicCAS(&table[at], ~0u, (h & ~0xFFu) | (uint32_t)q);
                if (seen == ~0u) break;
                if (((seen ^ h) >> 8) == 0u) {
                    uint32_t other[W], differ = 0;
#pragma unroll
                    for (int w = 0; w < W; ++w) other[w] = 0;
                    add_row<W>(other, step + (size_t)(seen & 0xFFu) * W);
#pragma unroll
                    for (int w = 0; w < W; ++w) differ |= other[w] ^ row[w];
                    if (!differ) {
                        like = (int)(seen & 0xFFu);
                        break;
                    }
                }
            }
        }
        const uint64_t fresh = __ballot(in && like == q);
        if (in && like == q) {
            const uint32_t k = n + (uint32_t)__popcll(fresh & ((1ull << lane) - 1ull));
            number[q] = (uint8_t)k;
            if (k < (uint32_t)kImageSets) L.first_with[slot][k] = (uint8_t)q;
        }
        n += (uint32_t)__popcll(fresh);
        lds_order();
        if (in) L.set_of[slot][q] = number[like];
    }
    lds_order();
    return n <= (uint32_t)kImageSets ? (n << 8) | (uint32_t)slot : kImageMany;
}

// Up to 256 states.  A workgroup of sixteen waves takes `per_group` consecutive tokens, a wave one at a time; which
// successor sets a byte has is worked out once per workgroup and first byte, by the wave that first needs it.
// 32,000 tokens x 256 states: 154 us with a thread per (token, start state), bound by instruction issue (75.6 M wave
// instructions), 90 us so; half of what is left is writing the rows (262 MB, 39-45 us).
//
// `split`: a token that every state walks for itself is shared out among the waves, 64 states each.  So where there is a
// wave per token or less (per_group <= 16), which would leave the others idle behind it: 8,000 tokens x 256 states
// without structure 95 us, 105 otherwise, and 1,060 against 1,280 with sets that grow.  With more tokens the waves are
// busy anyway, and a wave that walks all of a token's states finds their rows in its cache (32,000 tokens: 269 us split,
// 254 otherwise).  What that costs against a thread per pair, on sets that grow: 3.2 ms, 2.6 there; the tokens are dealt
// out beforehand and their work differs.  Without structure it is 254 against 329, on lexers 106 against 167.
template <int W>
__global__ __launch_bounds__(kImageThreads, 8) void nfa_image_kernel(NfaArgs a, int per_group, bool split) {
    __shared__ ImageLds<W> L;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    if (tid < 256) L.state[tid] = kImageUnknown;
    if (tid < kImageWaves) {
        L.done[tid] = 0;
        L.hash[tid] = 0;
    }
    if (tid == 0) {
        L.cursor = 0;
        L.slots = 0;
        L.alones = 0;
        L.known = 0;
    }
    __syncthreads();
    uint32_t *sets = L.sets[wave], *members = L.members[wave];
    const int group0 = (int)blockIdx.x * per_group, in_group = min(per_group, a.V - group0);
    const size_t matrix = (size_t)a.S * W;
    const int chunks = (a.S + 63) >> 6;
    for (;;) {
        // Keeps the wave together: without it the compiler joins the branch below with the one that ends the round
        // (lane 0 stores the hash), and the other lanes go round alone, reading a `taken` that is never theirs.
        __builtin_amdgcn_wave_barrier();
        int taken = 0;
        if (lane == 0) taken = (int)atomicAdd(&L.cursor, 1u);
        taken = __builtin_amdgcn_readfirstlane(taken);
        int item = taken, chunk = -1;
        if (taken >= in_group) {
            if (!split) break;
            // All tokens are taken.  What is left is those that every state walks for itself, once the waves that have
            // the last tokens have said which those are (they wait for nothing but a numbering).
            while (__builtin_amdgcn_readfirstlane(__hip_atomic_load(&L.known, __ATOMIC_RELAXED,
                                                                    __HIP_MEMORY_SCOPE_WORKGROUP)) < (uint32_t)in_group)
                __builtin_amdgcn_s_sleep(2);
            lds_order();
            const int alones = (int)__builtin_amdgcn_readfirstlane(L.alones), rest = taken - in_group;
            if (rest >= alones * chunks) break;
            item = (int)__builtin_amdgcn_readfirstlane(L.alone[rest / chunks]);
            chunk = rest % chunks;
        }
        const int t = group0 + item;
        const int64_t b0 = a.tok_off[t], b1 = a.tok_off[t + 1];
        uint32_t *out = a.rel + (size_t)t * matrix;
        uint64_t h = 0;
        uint32_t state = kImageMany;
        int b = 0;
        WaveBytes bytes(a.tok_bytes, b0, b1);
        if (chunk < 0 && b1 > b0) {
            b = bytes.at(b0);
            for (;;) {
                state = __hip_atomic_load(&L.state[b], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
                state = __builtin_amdgcn_readfirstlane(state);
                if (state == kImageUnknown) {
                    uint32_t was = 0;
                    if (lane == 0) was = atomicCAS(&L.state[b], kImageUnknown, kImageWorkedOut);
                    was = __builtin_amdgcn_readfirstlane(was);
                    if (was == kImageUnknown) {
                        state = number_sets<W>(a, L, sets, b);
                        if (lane == 0)
                            __hip_atomic_store(&L.state[b], state, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
                    }
                    continue;
                }
                if (state != kImageWorkedOut) break;
                __builtin_amdgcn_s_sleep(2);  // another wave is at it, and waits for nothing while it works
            }
            lds_order();
        }
        if (split && chunk < 0) {
            if (lane == 0) {
                if (state <= 0xFFu) L.alone[atomicAdd(&L.alones, 1u)] = (uint32_t)item;
                lds_order();
                atomicAdd(&L.known, 1u);
            }
            if (state <= 0xFFu) continue;
        }
        if (state > 0xFFu) {
            const int n = (int)(state >> 8), slot = (int)(state & 0xFFu);
            for (int j0 = 0; j0 < n; j0 += 64) {
                const int j = j0 + lane;
                uint32_t set[W];
#pragma unroll
                for (int w = 0; w < W; ++w) set[w] = 0;
                if (j < n) add_row<W>(set, a.nfa + b * matrix + (size_t)L.first_with[slot][j] * W);
                set[W - 1] &= a.last_word_mask;
                for (int64_t p = b0 + 1; p < b1; ++p) {
                    uint32_t any = 0;
#pragma unroll
                    for (int w = 0; w < W; ++w) any |= set[w];
                    if (__ballot(any != 0u) == 0ull) break;  // no state left anywhere: the rows stay empty
                    set_step<W>(set, a.nfa + (size_t)bytes.at(p) * matrix, a.last_word_mask);
                }
                if (j < n) {
                    uint32_t count, first, last;
                    set_members<W>(set, count, first, last);
                    members[j] = min(count, 3u) | (first << 8) | (last << 16);
#pragma unroll
                    for (int w = 0; w < W; ++w) sets[j * W + w] = set[w];
                }
                if (j0 + 64 < n) bytes = WaveBytes(a.tok_bytes, b0, b1);  // once more from the front
            }
            lds_order();
            const uint8_t *set_of = L.set_of[slot];
            // the rows, as one run of 16-byte units (or words) over the lanes
            if (W % 4 == 0) {
                constexpr int kPerRow = W / 4 > 0 ? W / 4 : 1;
                const int units = a.S * kPerRow;
                for (int x = lane; x < units; x += 64)
                    reinterpret_cast<uint4 *>(out)[x] =
                        reinterpret_cast<const uint4 *>(sets)[set_of[x / kPerRow] * kPerRow + x % kPerRow];
            } else {
                const int units = a.S * W;
                for (int x = lane; x < units; x += 64) out[x] = sets[set_of[x / W] * W + x % W];
            }
            if (a.hash) {
                for (int q = lane; q < a.S; q += 64) {
                    const uint32_t k = set_of[q], m = members[k], count = m & 0xFFu;
                    if (count == 0) continue;
                    if (count <= 2) {
                        h += member_hash((uint32_t)q, W, (m >> 8) & 0xFFu, a.seed);
                        if (count == 2) h += member_hash((uint32_t)q, W, m >> 16, a.seed);
                    } else {
                        uint32_t set[W];
#pragma unroll
                        for (int w = 0; w < W; ++w) set[w] = sets[k * W + w];
                        h += row_hash<W>(set, q, a.seed);
                    }
                }
            }
        } else {
            // the empty token (its relation is the identity), or a first byte that leaves many different sets: every
            // start state walks for itself
            for (int q0 = split ? 64 * chunk : 0, q1 = split ? q0 + 64 : a.S; q0 < q1; q0 += 64) {
                const int q = q0 + lane;
                uint32_t set[W];
#pragma unroll
                for (int w = 0; w < W; ++w) set[w] = (q < a.S && (q >> 5) == w) ? 1u << (q & 31) : 0u;
                WaveBytes from_front(a.tok_bytes, b0, b1);
                for (int64_t p = b0; p < b1; ++p) {
                    uint32_t any = 0;
#pragma unroll
                    for (int w = 0; w < W; ++w) any |= set[w];
                    if (__ballot(any != 0u) == 0ull) break;
                    set_step<W>(set, a.nfa + (size_t)from_front.at(p) * matrix, a.last_word_mask);
                }
                if (q >= a.S) continue;
                store_set<W>(out + (size_t)q * W, set);
                if (a.hash) h += row_hash<W>(set, q, a.seed);
            }
        }
        if (a.hash) {
#pragma unroll
            for (int off = 1; off < 64; off <<= 1) h += __shfl_xor(h, off, 64);
            if (chunk < 0) {
                if (lane == 0) a.hash[t] = h;
            } else if (lane == 0) {  // the last of the token's chunks to be done writes
                atomicAdd(&L.hash[item], (unsigned long long)h);
                lds_order();
                if ((int)atomicAdd(&L.done[item], 1u) + 1 == chunks) {
                    lds_order();
                    a.hash[t] = __hip_atomic_load(&L.hash[item], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
                }
            }
        }
        __builtin_amdgcn_wave_barrier();
    }
}

// A thread owns one (token, start state) pair.  (Two or four start states per thread, for more row reads in flight, made
// it slower: it is bound by instruction issue where it fills the chip, not by the latency of its reads.)
template <int W>
__global__ __launch_bounds__(kThreads) void nfa_walk_kernel(NfaArgs a, int threads_per_token) {
    __shared__ unsigned long long hash_sum[kThreads / 64];
    __shared__ uint8_t head_bytes[kThreads / 64][kStagedBytes];  // each token's first bytes
    const int slot = threadIdx.x / threads_per_token;
    const int q = threadIdx.x % threads_per_token;
    const int t = blockIdx.x * (kThreads / threads_per_token) + slot;
    if (threadIdx.x < kThreads / 64) hash_sum[threadIdx.x] = 0;
    int64_t b0 = 0, b1 = 0;
    if (t < a.V) {
        b0 = a.tok_off[t];
        b1 = a.tok_off[t + 1];
        if (q < kStagedBytes && b0 + q < b1) head_bytes[slot][q] = a.tok_bytes[b0 + q];
    }
    __syncthreads();
    uint64_t h = 0;
    if (t < a.V && q < a.S) {
        uint32_t set[W];
#pragma unroll
        for (int w = 0; w < W; ++w) set[w] = (q >> 5) == w ? 1u << (q & 31) : 0u;
        const size_t matrix = (size_t)a.S * W;
        for (int64_t p = b0; p < b1; ++p) {
            const int ch = p - b0 < kStagedBytes ? head_bytes[slot][p - b0] : a.tok_bytes[p];
            const uint32_t *step = a.nfa + ch * matrix;
            uint32_t next[W];
#pragma unroll
            for (int w = 0; w < W; ++w) next[w] = 0;
#pragma unroll
            for (int w = 0; w < W; ++w)
                for (uint32_t bits = set[w]; bits; bits &= bits - 1)
                    add_row<W>(next, step + (size_t)(w * 32 + __ffs(bits) - 1) * W);
            next[W - 1] &= a.last_word_mask;  // a stray pad bit must not become a state number
            uint32_t any = 0;
#pragma unroll
            for (int w = 0; w < W; ++w) {
                set[w] = next[w];
                any |= next[w];
            }
            if (!any) break;  // no state left: the row stays empty
        }
        store_set<W>(a.rel + ((size_t)t * a.S + q) * W, set);
        if (a.hash) h = row_hash<W>(set, q, a.seed);
    }
    if (a.hash) {
        if (h) atomicAdd(&hash_sum[slot], (unsigned long long)h);
        __syncthreads();
        if (q == 0 && t < a.V) a.hash[t] = hash_sum[slot];
    }
}

// More than 256 states: the sets no longer fit in registers.  A workgroup takes 256 start states
// of one token; a thread keeps its current and next set in LDS, word w of thread t at [w][t] (so
// the threads of a wave hit different banks), and per byte ORs the successor rows of the set's
// members into the next set.  The hash is accumulated per token with one atomic per workgroup
// (hash_out is cleared by a launch before).
__global__ __launch_bounds__(kThreads) void nfa_walk_lds_kernel(NfaArgs a, int W, int q_blocks) {
    extern __shared__ uint32_t sets[];  // [2][W][kThreads]
    __shared__ unsigned long long hash_sum;
    const int t = blockIdx.x / q_blocks;
    const int q = (blockIdx.x % q_blocks) * kThreads + threadIdx.x;
    uint32_t *cur = sets + threadIdx.x, *nxt = sets + (size_t)W * kThreads + threadIdx.x;
    if (threadIdx.x == 0) hash_sum = 0;
    __syncthreads();
    uint64_t h = 0;
    if (q < a.S) {
        for (int w = 0; w < W; ++w) cur[(size_t)w * kThreads] = (q >> 5) == w ? 1u << (q & 31) : 0u;
        const int64_t b0 = a.tok_off[t], b1 = a.tok_off[t + 1];
        const size_t matrix = (size_t)a.S * W;
        for (int64_t p = b0; p < b1; ++p) {
            const uint32_t *step = a.nfa + (size_t)a.tok_bytes[p] * matrix;
            for (int w = 0; w < W; ++w) nxt[(size_t)w * kThreads] = 0;
            for (int w = 0; w < W; ++w) {
                uint32_t bits = cur[(size_t)w * kThreads];
                while (bits) {
                    const int x = w * 32 + __ffs(bits) - 1;
                    bits &= bits - 1;
                    const uint32_t *row = step + (size_t)x * W;
                    for (int k = 0; k < W; ++k) nxt[(size_t)k * kThreads] |= row[k];
                }
            }
            nxt[(size_t)(W - 1) * kThreads] &= a.last_word_mask;  // a stray pad bit must not become a state number
            uint32_t any = 0;
            for (int w = 0; w < W; ++w) any |= nxt[(size_t)w * kThreads];
            uint32_t *tmp = cur;
            cur = nxt;
            nxt = tmp;
            if (!any) break;  // no state left: the row stays empty
        }
        uint32_t *out = a.rel + ((size_t)t * a.S + q) * W;
        for (int w = 0; w < W; ++w) {
            const uint32_t v = cur[(size_t)w * kThreads];
            out[w] = v;
            if (a.hash && v) {
                const uint32_t e = 2u * (uint32_t)(q * W + w);
                if (v & 0xFFFFu) h += (splitmix64_at(a.seed, e) | 1ull) * (uint64_t)(v & 0xFFFFu);
                if (v >> 16) h += (splitmix64_at(a.seed, e + 1u) | 1ull) * (uint64_t)(v >> 16);
            }
        }
    }
    if (a.hash) {
        if (h) atomicAdd(&hash_sum, (unsigned long long)h);
        __syncthreads();
        if (threadIdx.x == 0 && hash_sum)
            atomicAdd(reinterpret_cast<unsigned long long *>(a.hash + t), hash_sum);
    }
}

__global__ void clear_u64_kernel(uint64_t *p, int n) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) p[i] = 0;
}

template <int W>
int launch_nfa(const NfaArgs &a, int n_cu, hipStream_t stream) {
    constexpr bool kWalkOnly = W * 32 <= kWalkStates;
    if (kWalkOnly || (int64_t)a.V * a.S <= kWalkPairs) {
        int threads_per_token = 64;  // whole waves, a power of two so that a workgroup holds whole tokens
        while (threads_per_token < a.S) threads_per_token *= 2;
        hipLaunchKernelGGL(nfa_walk_kernel<W>, dim3((unsigned)ceil_div(a.V, kThreads / threads_per_token)), dim3(kThreads),
                           0, stream, a, threads_per_token);
        return check_launch();
    }
    if constexpr (!kWalkOnly) {
        // two workgroups per compute unit (their LDS is what there is), the tokens spread evenly
        const int64_t groups = std::min<int64_t>(2 * n_cu, ceil_div(a.V, kImageWaves));
        const int per_group = (int)std::min<int64_t>(kImageGroup, ceil_div(a.V, groups));
        hipLaunchKernelGGL(nfa_image_kernel<W>, dim3((unsigned)ceil_div(a.V, per_group)), dim3(kImageThreads), 0, stream, a,
                           per_group, per_group <= kImageWaves);
    }
    return check_launch();
}

}  // namespace
}  // namespace cfgzip

using namespace cfgzip;

extern "C" int cfgzip_nfa_signatures(const uint8_t *tok_bytes, const int64_t *tok_off, int32_t V,
                                     const int32_t *nfa, int32_t S, int32_t *rel_out,
                                     uint64_t *hash_out, uint64_t hash_seed, void *stream_) {
    if (!tok_off || !nfa || !rel_out) return CFGZIP_E_INVALID;
    if (V <= 0 || S <= 0 || S > kMaxNfaStates) return CFGZIP_E_INVALID;
    if (!aligned_to(tok_off, 8) || !aligned_to(nfa, 16) || !aligned_to(rel_out, 16) ||
        !aligned_to(hash_out, 8))
        return CFGZIP_E_INVALID;
    NfaArgs a{};
    a.tok_bytes = tok_bytes;
    a.tok_off = tok_off;
    a.nfa = reinterpret_cast<const uint32_t *>(nfa);
    a.rel = reinterpret_cast<uint32_t *>(rel_out);
    a.hash = hash_out;
    a.seed = hash_seed;
    a.V = V;
    a.S = S;
    a.last_word_mask = (S & 31) ? (1u << (S & 31)) - 1u : 0xFFFFFFFFu;
    hipStream_t stream = static_cast<hipStream_t>(stream_);
    if (S > kMaxRegisterStates) {
        const int W = (S + 31) / 32, q_blocks = (S + kThreads - 1) / kThreads;
        if ((int64_t)V * q_blocks > 0x7FFFFFFF) return CFGZIP_E_INVALID;
        if (hash_out) {
            hipLaunchKernelGGL(clear_u64_kernel, dim3((unsigned)ceil_div(V, kThreads)), dim3(kThreads), 0,
                               stream, hash_out, V);
            CFGZIP_TRY(check_launch());
        }
        const size_t dyn = (size_t)2 * W * kThreads * sizeof(uint32_t);
        if (dyn > 48 * 1024)
            CFGZIP_TRY(check_hip(hipFuncSetAttribute(reinterpret_cast<const void *>(nfa_walk_lds_kernel),
                                                     hipFuncAttributeMaxDynamicSharedMemorySize, (int)dyn)));
        hipLaunchKernelGGL(nfa_walk_lds_kernel, dim3((unsigned)(V * q_blocks)), dim3(kThreads), dyn, stream,
                           a, W, q_blocks);
        return check_launch();
    }
    int dev = 0, n_cu = 256;
    CFGZIP_TRY(check_hip(hipGetDevice(&dev)));
    CFGZIP_TRY(check_hip(hipDeviceGetAttribute(&n_cu, hipDeviceAttributeMultiprocessorCount, dev)));
    if (n_cu <= 0) n_cu = 256;
    switch ((S + 31) / 32) {
        case 1: return launch_nfa<1>(a, n_cu, stream);
        case 2: return launch_nfa<2>(a, n_cu, stream);
        case 3: return launch_nfa<3>(a, n_cu, stream);
        case 4: return launch_nfa<4>(a, n_cu, stream);
        case 5: return launch_nfa<5>(a, n_cu, stream);
        case 6: return launch_nfa<6>(a, n_cu, stream);
        case 7: return launch_nfa<7>(a, n_cu, stream);
        default: return launch_nfa<8>(a, n_cu, stream);
    }
}
