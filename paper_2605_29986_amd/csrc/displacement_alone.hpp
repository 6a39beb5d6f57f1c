// The passes behind the shared walk: one wave owns one token and carries its set of configurations through the bytes in
// two LDS buffers.
//
// A configuration of Algorithm 1 is a record (input queue, output stack, symbol consumed last), and the wave advances the
// set of its live configurations one byte at a time:
//   - a configuration with a non-empty output stack pops the top symbol A and pushes the body
//     of every production A -> a beta whose terminal is the byte read;
//   - one with an empty output stack backtracks: every production A -> a beta with that
//     terminal, whose head A is stack-adjacent to the symbol consumed last (any head at the
//     very first byte), appends A to the input queue and starts the output stack with beta.
// Successors are appended to a second LDS buffer through one LDS counter; duplicates are
// dropped while the survivors are packed back into the first.  What is left after the last byte, without the third
// component, is the displacement; it is written as a fixed-length row in a canonical order
// together with an order-free 64-bit hash, so that equal sets give equal rows and the class
// builder can group tokens by comparing rows.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "displacement_common.hpp"

namespace cfgzip {
namespace {

constexpr int kRowChunk = 256;                 // row entries staged in LDS at a time
constexpr int kMaxByteSymbols = 255;           // up to here a symbol (and "none") fits a byte

// caps of the second pass (over what the shared walk hands on) and of the third (over what the second could not
// finish), which are the interface's
// The second pass's queue and stack: what a token needs there sets how many waves a compute unit holds.  8-bit symbols: 24
// (eleven waves), up to which tokens of as many bytes stay out of the third pass, which takes four at a time.  16 / 20 / 24, calls
// on 32,000 tokens that share no sets, us: of 8 bytes 197 / 199 / 200, of 12 357 / 389 / 421, of 18 1,514 / 535 / 594, of 24 2,318 /
// 2,475 / 833.
template <typename Sym>
constexpr int kLists1 = sizeof(Sym) == 1 ? 24 : 12;
constexpr int kFrontier1 = 128;
constexpr int kIn2 = 32, kOut2 = 32, kFrontier2 = 256;
// the third pass keeps the current byte's productions and the relation in LDS when they fit
constexpr int kStageCap = 128;      // productions of one terminal
constexpr int kStageBodyCap = 512;  // body symbols of those productions together
constexpr int kAdjLdsWords = 512;   // N * W(N) words: N <= 128

// A record in LDS: ni, no, MAX_IN queue entries, MAX_OUT stack entries (top first), the symbol
// consumed last, zero padding up to an odd number of 32-bit words (lanes that read one record
// each then hit different banks).  Grammars with at most kMaxByteSymbols symbols use byte
// entries: half the LDS per token, twice the waves per compute unit.
template <typename Sym, int MAX_IN, int MAX_OUT>
struct Rec {
    static constexpr int kLen = 2 + MAX_IN + MAX_OUT;
    static constexpr int kStackAt = 2 + MAX_IN;
    static constexpr int kPrevAt = kLen;  // "none" before anything was consumed
    static constexpr int kWords = (((kLen + 1) * (int)sizeof(Sym) + 3) / 4) | 1;
    static constexpr int kStride = kWords * 4 / (int)sizeof(Sym);
    static constexpr int kOrderWords = (kLen * (int)sizeof(Sym) + 3) / 4;
    static constexpr int kBits = 8 * (int)sizeof(Sym);
    static constexpr int kNone = (1 << kBits) - 1;
};

// What the wave has written to LDS comes before what it reads next (no other wave has a part in it).
__device__ __forceinline__ void wave_order() {
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "workgroup");
    __builtin_amdgcn_wave_barrier();
}

template <typename R>
__device__ inline bool records_equal(const uint32_t *a, const uint32_t *b) {
    for (int k = 0; k < R::kWords; ++k)
        if (a[k] != b[k]) return false;
    return true;
}

// Canonical order: by (ni, no), then the queue, then the stack.  With equal ni and no the
// padding of two records sits at the same entries, so this is the ascending order of the padded
// entries: in the first word that differs, the lowest entry that differs decides (entry e of a
// word sits at bits e * kBits and up).  Called once the symbol consumed last has been cleared,
// so the words beyond the last entry are equal.
template <typename R>
__device__ inline bool record_less(const uint32_t *a, const uint32_t *b) {
    for (int k = 0; k < R::kOrderWords; ++k) {
        const uint32_t x = a[k], y = b[k];
        if (x != y) {
            const int shift = (__ffs(x ^ y) - 1) & ~(R::kBits - 1);
            const uint32_t mask = (uint32_t)R::kNone;
            return ((x >> shift) & mask) < ((y >> shift) & mask);
        }
    }
    return false;
}

// Drops every record of src[0..m) that equals an earlier one and packs the rest into dst;
// returns how many are left.  Called by the whole wave; m <= FRONTIER.  A 16-bit fingerprint of
// every record goes to `fp` first: a lane then scans the fingerprints before its own without
// branching (independent LDS reads) and compares whole records only where one matches.
// `empty_list` receives the positions (in dst) of the records whose stack is empty, `n_empty`
// how many there are: the next byte's backtrack visits only those.
template <typename Sym, typename R, int FRONTIER>
__device__ int drop_duplicates(const Sym (*src)[R::kStride], Sym (*dst)[R::kStride], int m, int lane,
                               uint16_t *fp, uint8_t *empty_list, int &n_empty) {
    for (int i = lane; i < m; i += 64) {
        const uint32_t *w = reinterpret_cast<const uint32_t *>(src[i]);
        uint32_t h = 0;
#pragma unroll
        for (int k = 0; k < R::kWords; ++k) h = h * 0x9E3779B1u + w[k];
        fp[i] = (uint16_t)((h >> 16) ^ h);
    }
    wave_order();
    int kept = 0;
    n_empty = 0;
    for (int base = 0; base < FRONTIER; base += 64) {
        if (base >= m) break;  // the same for every lane
        const int i = base + lane;
        bool keep = i < m;
        if (keep) {
            const uint32_t mine_fp = fp[i];
            bool candidate = false;
            const int last = min(m, base + 64) - 1;  // the same bound for every lane: no divergence
#pragma unroll 4
            for (int j = 0; j < last; ++j) candidate |= (j < i) & (fp[j] == mine_fp);
            if (candidate) {
                const uint32_t *mine = reinterpret_cast<const uint32_t *>(src[i]);
                for (int j = 0; j < i; ++j)
                    if (fp[j] == mine_fp &&
                        records_equal<R>(mine, reinterpret_cast<const uint32_t *>(src[j]))) {
                        keep = false;
                        break;
                    }
            }
        }
        const uint64_t mask = __ballot(keep);
        const bool empty = keep && src[i][1] == 0;
        const uint64_t empty_mask = __ballot(empty);
        const uint64_t below = (1ull << lane) - 1ull;
        if (keep) {
            const int pos = kept + __popcll(mask & below);
            const uint32_t *s = reinterpret_cast<const uint32_t *>(src[i]);
            uint32_t *d = reinterpret_cast<uint32_t *>(dst[pos]);
            for (int k = 0; k < R::kWords; ++k) d[k] = s[k];
            if (empty) empty_list[n_empty + __popcll(empty_mask & below)] = (uint8_t)pos;
        }
        kept += __popcll(mask);
        n_empty += __popcll(empty_mask);
    }
    return kept;
}

// LDS of one workgroup (one wave)
template <typename Sym, typename R, int FRONTIER, bool STAGE>
struct TokenLds {
    __align__(8) Sym buf[2][FRONTIER][R::kStride];
    __align__(8) uint16_t row[kRowChunk];
    int n_emit, crossed, total_len;
    unsigned long long hash_sum;
    uint16_t fingerprint[FRONTIER];
    uint8_t empty_list[FRONTIER];  // positions of the live configurations with an empty stack
    // STAGE only: the productions lo .. hi-1 of the byte being read (heads, body offsets
    // relative to the first, body symbols), and the relation
    uint16_t sp_body[STAGE ? kStageBodyCap : 1];
    uint16_t sp_off[STAGE ? kStageCap + 1 : 1];
    uint16_t sp_head[STAGE ? kStageCap : 1];
    uint32_t adj[STAGE ? kAdjLdsWords : 1];
};

// The displacement of token t under the caps MAX_IN, MAX_OUT, FRONTIER, by the whole wave.
// Returns whether it crosses one of them (the same for every lane); it then still gets the overflow row, which a later
// pass under wider caps overwrites if it gets through.
template <typename Sym, int MAX_IN, int MAX_OUT, int FRONTIER, bool STAGE>
__device__ bool token_displacement(const DisplacementArgs &a, int t,
                                   TokenLds<Sym, Rec<Sym, MAX_IN, MAX_OUT>, FRONTIER, STAGE> &L,
                                   bool adj_in_lds) {
    using R = Rec<Sym, MAX_IN, MAX_OUT>;
    constexpr int kStride = R::kStride;
    constexpr int kNone = R::kNone;
    static_assert(FRONTIER % 64 == 0 && FRONTIER <= 256, "whole waves of records; positions fit a byte");
    constexpr int kPerLane = FRONTIER / 64;
    const int lane = threadIdx.x & 63;
    const Grammar &g = a.g;
    const int64_t b0 = a.tok_off[t], b1 = a.tok_off[t + 1];

    // the start configuration: nothing consumed, nothing pushed
    for (int k = lane; k < kStride; k += 64) L.buf[0][0][k] = (Sym)(k == R::kPrevAt ? kNone : 0);
    if (lane == 0) {
        L.crossed = 0;
        L.empty_list[0] = 0;
    }
    int n = 1, n_empty = 1;
    bool caps_crossed = false;
    wave_order();

    Sym(*src)[kStride] = L.buf[0];  // the live set is always handed back to buf[0]
    Sym(*dst)[kStride] = L.buf[1];
    for (int64_t p = b0; p < b1 && n > 0; ++p) {
        const int ch = a.tok_bytes[p];
        const int lo = a.byte_off[ch], hi = a.byte_off[ch + 1];
        if (lane == 0) L.n_emit = 0;
        const int body_lo = hi > lo ? g.body_off[lo] : 0;
        const bool staged = STAGE && hi - lo <= kStageCap &&
                            (hi > lo ? g.body_off[hi] - body_lo : 0) <= kStageBodyCap;  // the same for every lane
        if (staged) {
            for (int i = lo + lane; i < hi; i += 64) L.sp_head[i - lo] = g.head[i];
            for (int i = lo + lane; i <= hi; i += 64) L.sp_off[i - lo] = (uint16_t)(g.body_off[i] - body_lo);
            const int symbols = hi > lo ? g.body_off[hi] - body_lo : 0;
            for (int x = lane; x < symbols; x += 64) L.sp_body[x] = g.body[body_lo + x];
        }
        wave_order();
        auto head_of = [&](int i) -> int { return staged ? L.sp_head[i - lo] : g.head[i]; };
        // a production's body: staged symbols in LDS, or the packed record (its first four symbols,
        // length and offset in one 16-byte load) with the symbol array behind it for longer bodies
        auto body_of = [&](int i) -> uint4 {
            if (staged) return make_uint4(0, 0, (uint32_t)(L.sp_off[i - lo + 1] - L.sp_off[i - lo]), L.sp_off[i - lo]);
            return a.prod_short[i];
        };
        auto body_sym = [&](const uint4 &b, int k) -> int {
            if (staged) return L.sp_body[b.w + k];
            if (k < 4) return (int)(((k < 2 ? b.x : b.y) >> (16 * (k & 1))) & 0xFFFFu);
            return g.body[b.w + k];
        };

        // pops: a lane per configuration (few productions per (terminal, head))
        for (int c = lane; c < n; c += 64) {
            const Sym *rec = src[c];
            const int no = rec[1];
            if (no == 0) continue;
            const int top = rec[R::kStackAt];
            const int first = a.pair_first[(size_t)ch * g.N + top] - 1;
            if (first < 0) continue;
            for (int i = first; i < hi && head_of(i) == top; ++i) {
                const uint4 body = body_of(i);
                const int len = (int)body.z;
                const int slot = atomicAdd(&L.n_emit, 1);
                if (no - 1 + len > MAX_OUT) {
                    L.crossed = 1;
                } else if (slot < FRONTIER) {
                    // the old record, then the stack rewritten: the body on top of what was below
                    Sym *o = dst[slot];
                    const uint32_t *rw = reinterpret_cast<const uint32_t *>(rec);
                    uint32_t *ow = reinterpret_cast<uint32_t *>(o);
                    for (int k = 0; k < R::kWords; ++k) ow[k] = rw[k];
                    const int new_no = no - 1 + len;
                    for (int k = 0; k < new_no; ++k)
                        o[R::kStackAt + k] = k < len ? (Sym)body_sym(body, k) : rec[R::kStackAt + k - len + 1];
                    if (len == 0) o[R::kStackAt + new_no] = 0;  // the stack got shorter by one
                    o[1] = (Sym)new_no;
                    o[R::kPrevAt] = (Sym)top;
                }
            }
        }
        // stack backtracks: the wave per configuration with an empty stack (every production of
        // the terminal)
        for (int e = 0; e < n_empty; ++e) {
            const Sym *rec = src[L.empty_list[e]];
            const int ni = rec[0];
            const int prev = rec[R::kPrevAt];
            for (int i = lo + lane; i < hi; i += 64) {
                const int A = head_of(i);
                if (prev != kNone) {
                    const size_t w = (size_t)A * g.W + (prev >> 5);
                    const uint32_t bits = (STAGE && adj_in_lds) ? L.adj[w] : a.adj[w];
                    if (!((bits >> (prev & 31)) & 1u)) continue;
                }
                const uint4 body = body_of(i);
                const int len = (int)body.z;
                const int slot = atomicAdd(&L.n_emit, 1);
                if (ni + 1 > MAX_IN || len > MAX_OUT) {
                    L.crossed = 1;
                } else if (slot < FRONTIER) {
                    // the old record (its stack is empty) with A appended to the queue, the body
                    // as the new stack
                    Sym *o = dst[slot];
                    const uint32_t *rw = reinterpret_cast<const uint32_t *>(rec);
                    uint32_t *ow = reinterpret_cast<uint32_t *>(o);
                    for (int k = 0; k < R::kWords; ++k) ow[k] = rw[k];
                    o[0] = (Sym)(ni + 1);
                    o[1] = (Sym)len;
                    o[2 + ni] = (Sym)A;
                    for (int k = 0; k < len; ++k) o[R::kStackAt + k] = (Sym)body_sym(body, k);
                    o[R::kPrevAt] = (Sym)A;
                }
            }
        }
        wave_order();
        const int m = L.n_emit;
        if (m > FRONTIER || L.crossed) {
            caps_crossed = true;
            break;
        }
        // back into the buffer just read
        n = drop_duplicates<Sym, R, FRONTIER>(dst, src, m, lane, L.fingerprint, L.empty_list, n_empty);
        wave_order();
    }

    int start[kPerLane];  // where this lane's records begin in the row
    bool overflow = caps_crossed;
    int total = 1;
    if (!caps_crossed) {
        // the displacement forgets the symbol consumed last
        for (int c = lane; c < n; c += 64) src[c][R::kPrevAt] = 0;
        if (lane == 0) {
            L.total_len = 1;
            L.hash_sum = 0;
        }
        wave_order();
        n = drop_duplicates<Sym, R, FRONTIER>(src, dst, n, lane, L.fingerprint, L.empty_list, n_empty);
        wave_order();
        // canonical order by counting: a record starts behind all smaller ones
#pragma unroll
        for (int u = 0; u < kPerLane; ++u) {
            const int c = lane + 64 * u;
            start[u] = 1;
            if (c < n) {
                const uint32_t *mine = reinterpret_cast<const uint32_t *>(dst[c]);
                for (int j = 0; j < n; ++j) {
                    const Sym *r = dst[j];
                    if (j != c && record_less<R>(reinterpret_cast<const uint32_t *>(r), mine))
                        start[u] += 2 + r[0] + r[1];
                }
                atomicAdd(&L.total_len, 2 + dst[c][0] + dst[c][1]);
            }
        }
        wave_order();
        total = L.total_len;
        if (total > a.row_len) overflow = true;
    }

    if (overflow) {
        if (lane == 0) {
            a.hash[t] = overflow_hash(a.seed, t);
            if (a.status) a.status[t] = kStatusOverflow;
        }
    } else {
        uint64_t h = 0;
#pragma unroll
        for (int u = 0; u < kPerLane; ++u) {
            const int c = lane + 64 * u;
            if (c < n) {
                const Sym *r = dst[c];
                RecordMix mix(a.seed);
                mix.add(r[0]);
                mix.add(r[1]);
                for (int k = 0; k < r[0]; ++k) mix.add(r[2 + k]);
                for (int k = 0; k < r[1]; ++k) mix.add(r[R::kStackAt + k]);
                h += mix.done();
            }
        }
        if (h) atomicAdd(&L.hash_sum, (unsigned long long)h);
    }

    // the row, kRowChunk entries at a time through LDS; chunks behind the data are plain zeros
    uint16_t *out_row = a.rows + (size_t)t * a.row_len;
    const int used = overflow ? 3 : total;
    for (int base = 0; base < a.row_len; base += kRowChunk) {
        uint2 *out = reinterpret_cast<uint2 *>(out_row + base);
        if (base >= used) {  // the same for every lane
            out[lane] = make_uint2(0, 0);
            continue;
        }
        reinterpret_cast<uint2 *>(L.row)[lane] = make_uint2(0, 0);
        wave_order();
        if (overflow) {
            if (lane == 0) {
                L.row[0] = 0xFFFF;
                L.row[1] = (uint16_t)(t & 0xFFFF);
                L.row[2] = (uint16_t)((uint32_t)t >> 16);
            }
        } else {
            if (lane == 0 && base == 0) L.row[0] = (uint16_t)n;
#pragma unroll
            for (int u = 0; u < kPerLane; ++u) {
                const int c = lane + 64 * u;
                if (c >= n) continue;
                const Sym *r = dst[c];
                const int ni = r[0], no = r[1];
                const int first = start[u] - base;  // position of the record's first entry in this chunk
                if (first >= kRowChunk || first + 2 + ni + no <= 0) continue;
                for (int e = max(0, -first); e < 2 + ni + no && first + e < kRowChunk; ++e) {
                    const int v = e < 2 ? r[e] : (e < 2 + ni ? r[e] : r[R::kStackAt + e - 2 - ni]);
                    L.row[first + e] = (uint16_t)v;
                }
            }
        }
        wave_order();
        out[lane] = reinterpret_cast<const uint2 *>(L.row)[lane];
    }
    wave_order();
    if (!overflow && lane == 0) {
        a.hash[t] = L.hash_sum;
        if (a.status) a.status[t] = kStatusOk;
    }
    wave_order();  // the wave's next token starts from settled LDS
    return caps_crossed;
}

}  // namespace
}  // namespace cfgzip
