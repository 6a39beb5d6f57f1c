// What the passes over the displacement sets share: the grammar and its tables as the kernels see them, the
// per-record hash, and the mark of a token that overflows.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace cfgzip {
namespace {

constexpr int kStatusOk = 0;
constexpr int kStatusOverflow = 1;
constexpr int kStatusBadGrammar = 2;

struct GrammarHeader {
    int32_t invalid;      // set by the index kernel when the productions break a stated rule
    // two lists of tokens: those that the shared walk hands on, or with more than 255 symbols all, and then those that the
    // pass over them hands on
    int32_t retry_count[2];
    int32_t retry_next[2];  // next entry of each list to be taken
    int32_t pad[59];
};

struct Grammar {
    const uint16_t *head;
    const uint8_t *byte;
    const int32_t *body_off;  // [P + 1]: the body of production i is body[body_off[i] .. body_off[i+1])
    const uint16_t *body;
    int P, N, W;              // W = words per bit row over the symbols
    int body_total;           // body symbols the caller says there are (the offsets are checked against it)
};

__device__ __forceinline__ int body_len(const Grammar &g, int i) { return g.body_off[i + 1] - g.body_off[i]; }

// A production in one word: up to four body symbols (12 bits each), the head (12 bits), the length of the body
// (4 bits; kLongBody: more than four symbols, all of them in the symbol array).
constexpr uint32_t kLongBody = 15;
__device__ __forceinline__ uint32_t packed_symbol(unsigned long long p, int k) { return (uint32_t)(p >> (12 * k)) & 0xFFFu; }
__device__ __forceinline__ uint32_t packed_head(unsigned long long p) { return (uint32_t)(p >> 48) & 0xFFFu; }
__device__ __forceinline__ uint32_t packed_length(unsigned long long p) { return (uint32_t)(p >> 60); }
__device__ __forceinline__ unsigned long long pack_production(const Grammar &g, int i, int off, int len) {
    unsigned long long p = (unsigned long long)g.head[i] << 48;
    if (len > 4) return p | ((unsigned long long)kLongBody << 60);
    for (int k = 0; k < len; ++k) p |= (unsigned long long)g.body[off + k] << (12 * k);
    return p | ((unsigned long long)len << 60);
}

struct DisplacementArgs {
    Grammar g;
    GrammarHeader *hdr;
    const int32_t *byte_off;
    const int32_t *pair_first;
    const uint4 *prod_short;
    const unsigned long long *prod_packed;  // [P]
    const uint8_t *byte_like;  // [256]: the first byte with the same productions
    const uint32_t *adj;
    const uint8_t *tok_bytes;
    const int64_t *tok_off;
    uint16_t *rows;
    uint64_t *hash;
    int32_t *status;
    int32_t *retry_list[2];
    uint64_t seed;
    int V, row_len;
};

// 64-bit mix of a record's entries ni, no, queue, stack (FNV-1a style pass, SplitMix64 finaliser)
struct RecordMix {
    uint64_t h;
    __device__ explicit RecordMix(uint64_t seed) : h(seed ^ 0x9E3779B97F4A7C15ull) {}
    __device__ void add(uint32_t x) {  // times 0x100000001B3
        h ^= x;
        h = h * 0x1B3ull + (h << 40);
    }
    __device__ uint64_t done() const {
        uint64_t z = h;
        z ^= z >> 30;
        z *= 0xBF58476D1CE4E5B9ull;
        z ^= z >> 27;
        z *= 0x94D049BB133111EBull;
        z ^= z >> 31;
        return z;
    }
};

// the hash of a token that overflows: a function of its id, so that it shares a class with no other
__device__ inline uint64_t overflow_hash(uint64_t seed, int t) {
    RecordMix mix(seed);
    mix.add(0xFFFFu);
    mix.add((uint32_t)t & 0xFFFFu);
    mix.add((uint32_t)t >> 16);
    return mix.done();
}

}  // namespace
}  // namespace cfgzip
