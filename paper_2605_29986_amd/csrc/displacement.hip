// Displacement sets of tokens over a context-free grammar in Greibach normal form (paper
// Section 3.2.1, Algorithm 1) and the stack-adjacency relation that prunes the stack
// backtrack (Section 3.2.2, Appendix C).
//
// The tables of a small grammar come out of one launch, those of a large one out of several.  The displacements
// then take three passes, most of the time only the first of which has anything to do:
//   1. displacement_shared.hpp: all tokens, by a walk over configuration sets that a workgroup's tokens share;
//   2. displacement_alone.hpp: the tokens whose sets did not fit there, one wave each, under small caps (little LDS, many
//      waves per compute unit);
//   3. what crosses those, again one wave each, under the caps that the interface states.
// The second and the third are one launch.  With more than 255 symbols there is no shared walk, and the two passes behind it
// are launches of their own over all tokens.
//
// Everything is bounded: queue, stack, number of successors per byte and row length each have
// a cap.  A token that crosses the interface's caps, or whose set does not fit the row,
// gets a row and hash of its own (its class is a singleton, which costs compression and never
// correctness).

#include <algorithm>

#include "common.hpp"
#include "displacement_common.hpp"
#include "displacement_alone.hpp"
#include "displacement_shared.hpp"

namespace cfgzip {
namespace {

constexpr int kMaxRowLen = 4096;
constexpr int kMaxSymbols = 4096;

struct GrammarWorkspace {
    GrammarHeader *hdr;
    int32_t *byte_off;  // [257]: productions with terminal b are byte_off[b] .. byte_off[b+1]-1
    uint32_t *unary;    // [W]: symbols with a production without body
    uint32_t *reach[2]; // [N][W]: reachability over "right-most body symbol" edges
    uint32_t *adj;      // [N][W]: bit Y of row Z <=> (Y, Z) stack-adjacent
    int32_t *pair_first;  // [256][N]: 1 + index of the first production with (terminal, head), 0 = none
    uint8_t *byte_like;   // [256]: the first byte with the same productions
    unsigned long long *prod_packed;  // [P]: the production in one word
    uint4 *prod_short;    // [P]: first four body symbols (16 bits each), body length, body offset: one load per production
    int32_t *retry_list[2];  // [V] each: ids of the tokens handed on
    size_t clear_words; // words from hdr to the end that start at zero
    size_t bytes;
};

GrammarWorkspace carve_grammar_ws(void *ws, int N, int V, int P) {
    GrammarWorkspace g{};
    const size_t W = (size_t)ceil_div(N, 32);
    size_t off = 0;
    auto take = [&](size_t bytes) {
        char *p = static_cast<char *>(ws) + off;
        off += (bytes + 255) / 256 * 256;
        return p;
    };
    g.hdr = reinterpret_cast<GrammarHeader *>(take(sizeof(GrammarHeader)));
    g.byte_off = reinterpret_cast<int32_t *>(take(257 * sizeof(int32_t)));
    g.unary = reinterpret_cast<uint32_t *>(take(W * 4));
    g.reach[0] = reinterpret_cast<uint32_t *>(take((size_t)N * W * 4));
    g.adj = reinterpret_cast<uint32_t *>(take((size_t)N * W * 4));
    g.pair_first = reinterpret_cast<int32_t *>(take((size_t)256 * N * 4));
    g.clear_words = off / 4;
    g.reach[1] = reinterpret_cast<uint32_t *>(take((size_t)N * W * 4));  // fully written
    g.byte_like = reinterpret_cast<uint8_t *>(take(256));  // fully written for a valid grammar
    g.prod_packed = reinterpret_cast<unsigned long long *>(take((size_t)P * 8));  // fully written for a valid grammar
    g.prod_short = reinterpret_cast<uint4 *>(take((size_t)P * sizeof(uint4)));  // fully written for a valid grammar
    g.retry_list[0] = reinterpret_cast<int32_t *>(take((size_t)V * 4));
    g.retry_list[1] = reinterpret_cast<int32_t *>(take((size_t)V * 4));
    g.bytes = off;
    return g;
}

__global__ void clear_words_kernel(uint32_t *p, size_t n) {
    for (size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x; i < n;
         i += (size_t)gridDim.x * blockDim.x)
        p[i] = 0;
}

// (byte, head, body) of production i strictly below that of production j, bodies compared
// symbol by symbol, a proper prefix first.  Both bodies lie inside the body array.
__device__ bool production_less(const Grammar &g, int i, int j) {
    if (g.byte[i] != g.byte[j]) return g.byte[i] < g.byte[j];
    if (g.head[i] != g.head[j]) return g.head[i] < g.head[j];
    const int li = body_len(g, i), lj = body_len(g, j);
    const uint16_t *bi = g.body + g.body_off[i], *bj = g.body + g.body_off[j];
    for (int k = 0; k < min(li, lj); ++k)
        if (bi[k] != bj[k]) return bi[k] < bj[k];
    return li < lj;
}

// Whether production i keeps the rules, as far as it and the one before it show; its body's place comes back.
__device__ bool production_valid(const Grammar &g, int i, int &off, int &end) {
    off = g.body_off[i];
    end = g.body_off[i + 1];
    bool ok = g.head[i] < g.N && off >= 0 && end >= off && end <= g.body_total;
    if (ok && i == 0) ok = off == 0;
    if (ok && i == g.P - 1) ok = end == g.body_total;
    if (ok && i > 0) {  // the body before this one must be in bounds before it is compared
        const int poff = g.body_off[i - 1];
        ok = poff >= 0 && poff <= off;
    }
    if (ok)
        for (int k = off; k < end; ++k) ok = ok && g.body[k] < g.N;
    if (ok && i > 0) ok = production_less(g, i - 1, i);
    return ok;
}

// A production as the displacement kernels read it.
__device__ unsigned long long write_records(const Grammar &g, const GrammarWorkspace &w, int i, int off, int len) {
    uint32_t sym[4] = {0, 0, 0, 0};
    for (int k = 0; k < min(len, 4); ++k) sym[k] = g.body[off + k];
    w.prod_short[i] = make_uint4(sym[0] | (sym[1] << 16), sym[2] | (sym[3] << 16), (uint32_t)len, (uint32_t)off);
    const unsigned long long packed = pack_production(g, i, off, len);
    w.prod_packed[i] = packed;
    return packed;
}

// One thread per production and per symbol: checks the rules the other kernels rely on
// (body offsets ascending from 0 to the stated total, symbols < N, strictly ascending order of
// the productions), finds where each terminal's productions start, marks unary symbols and
// seeds the reachability matrix with the identity and the edges head -> right-most body symbol
// (Appendix C's graph).
__global__ void grammar_index_kernel(Grammar g, GrammarWorkspace w) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i < g.N) atomicOr(&w.reach[0][(size_t)i * g.W + (i >> 5)], 1u << (i & 31));
    if (i >= g.P) return;
    int off, end;
    const bool ok = production_valid(g, i, off, end);
    const int len = end - off;
    if (!ok) {
        w.hdr->invalid = 1;
        return;
    }
    const int b = g.byte[i];
    const int first = i == 0 ? 0 : g.byte[i - 1] + 1;
    for (int x = first; x <= b; ++x) w.byte_off[x] = i;  // empty when the bytes are equal
    if (i == g.P - 1)
        for (int x = b + 1; x <= 256; ++x) w.byte_off[x] = g.P;
    const int A = g.head[i];
    if (i == 0 || g.byte[i - 1] != b || g.head[i - 1] != A) w.pair_first[(size_t)b * g.N + A] = i + 1;
    write_records(g, w, i, off, len);
    if (len == 0) {
        atomicOr(&w.unary[A >> 5], 1u << (A & 31));
    } else {
        const int last = g.body[end - 1];
        atomicOr(&w.reach[0][(size_t)A * g.W + (last >> 5)], 1u << (last & 31));
    }
}

// Bytes with the same productions (heads and bodies) lead every set of configurations to the same set: byte_like[b]
// is the first of them.  By one workgroup of at least 256 threads; a hash of all productions of a byte picks the
// candidate, which a table in LDS gives, and the productions decide.  byte_off: first production of every byte (and P),
// packed(i): production i in one word, both readable by everybody.
struct LikeLds {
    uint32_t hash[256];
    uint32_t slot[512], first[512];  // a hash (never 0), the first byte that has it
};
template <typename Packed>
__device__ __forceinline__ void find_like_bytes(const Grammar &g, const GrammarWorkspace &w, const int32_t *byte_off, LikeLds &L,
                                                const Packed &packed) {
    const int tid = threadIdx.x;
    if (tid < 256) L.hash[tid] = (uint32_t)(byte_off[tid + 1] - byte_off[tid]);
    for (int i = tid; i < 512; i += blockDim.x) {
        L.slot[i] = 0;
        L.first[i] = 256;
    }
    __syncthreads();
    for (int i = tid; i < g.P; i += blockDim.x) {
        const unsigned long long p = packed(i);  // of a long body only that it is one: the comparison tells them apart
        const uint32_t h = ((uint32_t)p ^ ((uint32_t)(p >> 32) * 0x85EBCA6Bu)) * 0x9E3779B1u;
        const int b = g.byte[i];
        atomicAdd(&L.hash[b], (h ^ (h >> 15)) * (2u * (uint32_t)(i - byte_off[b]) + 1u));
    }
    __syncthreads();
    const uint32_t mine = tid < 256 ? L.hash[tid] | 1u : 0u;
    uint32_t at = (mine * 0x9E3779B1u) >> 23;
    if (tid < 256) {
        for (;; at = (at + 1) & 511u) {  // (at most half full)
            uint32_t seen = *(volatile uint32_t *)&L.slot[at];  // most bytes have no productions: look before the atomics
            if (seen == 0u) seen = atomicCAS(&L.slot[at], 0u, mine);
            if (seen == 0u || seen == mine) break;
        }
        if (*(volatile uint32_t *)&L.first[at] > (uint32_t)tid) atomicMin(&L.first[at], (uint32_t)tid);
    }
    __syncthreads();
    if (tid >= 256) return;
    int like = (int)L.first[at];  // the first byte with the same hash, itself at the latest
    if (like != tid) {
        const int lo = byte_off[tid], n = byte_off[tid + 1] - lo, other = byte_off[like];
        bool same = byte_off[like + 1] - other == n;
        bool any_long = false;
        if (same)
#pragma unroll 4
            for (int i = 0; i < n; ++i) {  // to the end: reads that wait for nothing
                const unsigned long long p = packed(lo + i);
                same = same & (p == packed(other + i));
                any_long = any_long | (packed_length(p) == kLongBody);
            }
        for (int i = 0; any_long && same && i < n; ++i) {
            const int len = body_len(g, lo + i);
            if (len <= 4) continue;
            same = body_len(g, other + i) == len;
            for (int k = 0; same && k < len; ++k) same = g.body[g.body_off[lo + i] + k] == g.body[g.body_off[other + i] + k];
        }
        if (!same) like = tid;
    }
    w.byte_like[tid] = (uint8_t)like;
}

__global__ __launch_bounds__(1024) void byte_like_kernel(Grammar g, GrammarWorkspace w) {
    __shared__ LikeLds lds;
    if (w.hdr->invalid) return;  // the same for every thread
    find_like_bytes(g, w, w.byte_off, lds, [&](int i) { return w.prod_packed[i]; });
}

// All tables of a small grammar in one launch, by one workgroup with the grammar and the two matrices in LDS (eleven
// launches otherwise, each a few us of waiting for the one before).  What there is to wait for is one read of the grammar
// and then a chain of LDS accesses: read from memory as they were needed, production after body after the production
// before it, the bytes without productions filled in and like bytes found one by one, 480 productions over 27 symbols took
// 16.4 us and 786 over 25 19.0; 11.1 and 10.9 so, of which the launch is 4.5.
constexpr int kSmallSymbols = 128;
constexpr int kSmallWords = kSmallSymbols / 32;
constexpr int kSmallProductions = 4096;
constexpr int kSmallBodies = 16384;  // body symbols of all productions kept in LDS; if there are more they stay in memory
template <bool BODIES>
__global__ __launch_bounds__(1024) void grammar_tables_kernel(Grammar from, GrammarWorkspace w) {
    __shared__ uint32_t reach[2][kSmallSymbols * kSmallWords];
    __shared__ uint32_t adj[kSmallSymbols * kSmallWords];
    __shared__ uint32_t unary[kSmallWords];
    __shared__ unsigned long long packed[kSmallProductions];
    __shared__ int32_t byte_off[257], body_off[kSmallProductions + 1];
    __shared__ LikeLds lds;
    __shared__ uint16_t head[kSmallProductions];
    __shared__ uint8_t byte[kSmallProductions];
    __shared__ uint16_t body[BODIES ? kSmallBodies : 1];
    __shared__ int invalid;
    Grammar g = from;
    const int tid = threadIdx.x, threads = blockDim.x, words = g.N * g.W;
    {
        // a thread's first of each are asked for together
        const int last = g.P - 1, most = g.body_total - 1;
        const uint16_t first_head = from.head[min(tid, last)];
        const uint8_t first_byte = from.byte[min(tid, last)];
        const int32_t first_off = from.body_off[min(tid, last + 1)];
        const uint16_t first_symbol = BODIES && most >= 0 ? from.body[min(tid, most)] : (uint16_t)0;
        for (int i = tid + threads; i < g.P; i += threads) {
            head[i] = from.head[i];
            byte[i] = from.byte[i];
        }
        for (int i = tid + threads; i <= g.P; i += threads) body_off[i] = from.body_off[i];
        if (BODIES)
            for (int i = tid + threads; i < g.body_total; i += threads) body[i] = from.body[i];
        if (tid < g.P) {
            head[tid] = first_head;
            byte[tid] = first_byte;
        }
        if (tid <= g.P) body_off[tid] = first_off;
        if (BODIES && tid < g.body_total) body[tid] = first_symbol;
    }
    g.head = head;
    g.byte = byte;
    g.body_off = body_off;
    if (BODIES) g.body = body;
    for (int i = tid; i < words; i += threads) {
        const int X = i / g.W, word = i - X * g.W;
        reach[0][i] = (X >> 5) == word ? 1u << (X & 31) : 0u;
        adj[i] = 0;
    }
    if (tid < kSmallWords) unary[tid] = 0;
    if (tid == 0) invalid = 0;
    for (int i = tid; i < 256 * g.N; i += threads) w.pair_first[i] = 0;
    for (int i = tid; i < (int)(sizeof(GrammarHeader) / 4); i += threads) reinterpret_cast<int32_t *>(w.hdr)[i] = 0;
    __syncthreads();
    for (int i = tid; i < g.P; i += threads) {
        int off, end;
        if (!production_valid(g, i, off, end)) {
            invalid = 1;
            continue;
        }
        const int b = byte[i], A = head[i];
        if (i == 0 || byte[i - 1] != b || head[i - 1] != A) w.pair_first[(size_t)b * g.N + A] = i + 1;
        packed[i] = write_records(g, w, i, off, end - off);
        if (off == end) {
            atomicOr(&unary[A >> 5], 1u << (A & 31));
        } else {
            const int last = g.body[end - 1];
            atomicOr(&reach[0][A * g.W + (last >> 5)], 1u << (last & 31));
        }
    }
    if (tid < 257) {  // the first production whose byte is not below `tid` (one by one the last thread had 130 to fill in)
        int lo = 0;
        for (int count = g.P; count > 0;) {
            const int half = count >> 1;
            const bool right = (int)byte[lo + half] < tid;
            lo = right ? lo + half + 1 : lo;
            count = right ? count - half - 1 : half;
        }
        byte_off[tid] = lo;
    }
    __syncthreads();
    if (invalid) {  // the same for every thread
        if (tid == 0) w.hdr->invalid = 1;
        for (int i = tid; i < words; i += threads) w.adj[i] = 0;
        return;
    }
    // closure by doubling: every row holds its own symbol, so ceil(log2 N) rounds reach every path.  A wave per row, a
    // lane per pair of symbols of the row: what they reach is ORed together by register moves.
    int cur = 0;
    for (int span = 1; span < g.N; span <<= 1, cur ^= 1) {
        for (int X = tid >> 6; X < g.N; X += threads >> 6) {
            uint32_t acc[kSmallWords];
#pragma unroll
            for (int word = 0; word < kSmallWords; ++word) acc[word] = 0;
#pragma unroll
            for (int h = 0; h < kSmallSymbols / 64; ++h) {
                const int Y = (tid & 63) + 64 * h;
                if (Y < g.N && ((reach[cur][X * g.W + (Y >> 5)] >> (Y & 31)) & 1u))
                    for (int word = 0; word < kSmallWords; ++word)
                        if (word < g.W) acc[word] |= reach[cur][Y * g.W + word];
            }
#pragma unroll
            for (int word = 0; word < kSmallWords; ++word)
                if (word < g.W) {  // the same for every lane
                    const uint32_t all = wave_or32(acc[word]);
                    if ((tid & 63) == 0) reach[cur ^ 1][X * g.W + word] = all;
                }
        }
        __syncthreads();
    }
    // Appendix C over the neighbouring pairs of every body
    for (int i = tid; i < g.P; i += threads)
        for (int p = body_off[i]; p + 1 < body_off[i + 1]; ++p) {
            const int Bn = g.body[p], Z = g.body[p + 1];
            for (int word = 0; word < g.W; ++word) {
                const uint32_t bits = reach[cur][Bn * g.W + word] & unary[word];
                if (bits) atomicOr(&adj[Z * g.W + word], bits);
            }
        }
    if (tid < 257) w.byte_off[tid] = byte_off[tid];
    find_like_bytes(g, w, byte_off, lds, [&](int i) { return packed[i]; });
    __syncthreads();
    for (int i = tid; i < words; i += threads) w.adj[i] = adj[i];
}

// One doubling step of the transitive closure: out[X] = union of in[Y] over Y in in[X].  Every
// row holds its own symbol, so rows only grow; ceil(log2 N) steps reach every path.
__global__ __launch_bounds__(64) void closure_round_kernel(const uint32_t *__restrict__ in,
                                                           uint32_t *__restrict__ out, int N,
                                                           int W) {
    const int X = blockIdx.x, lane = threadIdx.x;
    uint32_t acc0 = 0, acc1 = 0;
    for (int w = 0; w < W; ++w) {
        uint32_t bits = in[(size_t)X * W + w];
        while (bits) {
            const int Y = w * 32 + __ffs(bits) - 1;
            bits &= bits - 1;
            if (Y < N) {
                if (lane < W) acc0 |= in[(size_t)Y * W + lane];
                if (lane + 64 < W) acc1 |= in[(size_t)Y * W + lane + 64];
            }
        }
    }
    if (lane < W) out[(size_t)X * W + lane] = acc0;
    if (lane + 64 < W) out[(size_t)X * W + lane + 64] = acc1;
}

// Appendix C: for a production A -> a B_1 .. B_n Z beta (n >= 1), every unary symbol reachable
// from B_n is consumed right before Z.  One thread per (production, word); it goes through the
// neighbouring pairs of the body.
__global__ void adjacency_kernel(Grammar g, GrammarWorkspace w, const uint32_t *__restrict__ reach) {
    const int64_t idx = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    const int word = (int)(idx % g.W);
    const int64_t i = idx / g.W;
    if (i >= g.P || w.hdr->invalid) return;
    const int off = g.body_off[i], end = g.body_off[i + 1];
    for (int p = off; p + 1 < end; ++p) {
        const int Bn = g.body[p], Z = g.body[p + 1];
        const uint32_t bits = reach[(size_t)Bn * g.W + word] & w.unary[word];
        if (bits) atomicOr(&w.adj[(size_t)Z * g.W + word], bits);
    }
}

__global__ void copy_words_kernel(const uint32_t *__restrict__ src, int32_t *__restrict__ dst,
                                  size_t n) {
    for (size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x; i < n;
         i += (size_t)gridDim.x * blockDim.x)
        dst[i] = (int32_t)src[i];
}

// `like_bytes`: whether byte_like is wanted too (8 us of a large grammar's tables: 144 -> 152 us with 3,944 productions
// over 135 symbols); only the shared walk reads it.
int enqueue_grammar_tables(const Grammar &g, const GrammarWorkspace &w, bool like_bytes, hipStream_t stream) {
    if (g.N <= kSmallSymbols && g.P <= kSmallProductions) {
        if (g.body_total <= kSmallBodies) hipLaunchKernelGGL(grammar_tables_kernel<true>, dim3(1), dim3(1024), 0, stream, g, w);
        else hipLaunchKernelGGL(grammar_tables_kernel<false>, dim3(1), dim3(1024), 0, stream, g, w);
        return check_launch();
    }
    hipLaunchKernelGGL(clear_words_kernel, dim3((unsigned)std::min<int64_t>(1024, ceil_div((int64_t)w.clear_words, 256))),
                       dim3(256), 0, stream, reinterpret_cast<uint32_t *>(w.hdr), w.clear_words);
    CFGZIP_TRY(check_launch());
    hipLaunchKernelGGL(grammar_index_kernel, dim3((unsigned)ceil_div(std::max(g.P, g.N), 256)),
                       dim3(256), 0, stream, g, w);
    CFGZIP_TRY(check_launch());
    int rounds = 0;
    while ((1 << rounds) < g.N) ++rounds;
    int cur = 0;
    for (int r = 0; r < rounds; ++r, cur ^= 1) {
        hipLaunchKernelGGL(closure_round_kernel, dim3(g.N), dim3(64), 0, stream, w.reach[cur],
                           w.reach[cur ^ 1], g.N, g.W);
        CFGZIP_TRY(check_launch());
    }
    const int64_t items = (int64_t)g.P * g.W;
    if (like_bytes) {
        hipLaunchKernelGGL(byte_like_kernel, dim3(1), dim3(1024), 0, stream, g, w);
        CFGZIP_TRY(check_launch());
    }
    hipLaunchKernelGGL(adjacency_kernel, dim3((unsigned)ceil_div(items, 256)), dim3(256), 0, stream,
                       g, w, w.reach[cur]);
    return check_launch();
}

// ---- what the shared walk hands on ---------------------------------------------------------

// What the passes behind the shared walk hold, as many waves as there is LDS for.
constexpr int kAloneThreads = 1024;
struct AloneLds {
    using First = TokenLds<uint8_t, Rec<uint8_t, kLists1<uint8_t>, kLists1<uint8_t>>, kFrontier1, false>;
    using Last = TokenLds<uint8_t, Rec<uint8_t, kIn2, kOut2>, kFrontier2, true>;
    static constexpr int kRoom = 160 * 1024 - 16, kWaves = kAloneThreads / 64;
    static constexpr int kFirst = kRoom / (int)sizeof(First) < kWaves ? kRoom / (int)sizeof(First) : kWaves;
    static constexpr int kLast = kRoom / (int)sizeof(Last) < kWaves ? kRoom / (int)sizeof(Last) : kWaves;
    __align__(16) uint32_t next[2];  // of the workgroup's two lists
    uint32_t left;                   // entries of the second
    union {
        First first[kFirst];
        Last last[kLast];
    };
};
static_assert(sizeof(AloneLds) <= 160 * 1024 && AloneLds::kFirst >= 11 && AloneLds::kLast >= 4, "");

// The tokens that the shared walk has no room for: a wave each, under small caps, and those that cross them once more under
// the interface's.  They are on one list for all workgroups: workgroup b takes entries b, b + grid, ...  Where such tokens lie
// together in a vocabulary the workgroups of the walk that had them would otherwise be the only ones that work: 128,256 tokens
// over the JSON grammar of which the last 8,000 (of 12 bytes) share no sets 1,430 us a call, 389 so; 120,556 of which the last
// 300 (of 28 bytes, most of which take the wide caps) 7,400 and 550.  What it costs is a launch that usually has nothing to
// do: 2 us of 50 with 2,000 tokens over the statement grammar, 2 to 3 of 105 to 125 with 32,000 and 128,256 over the JSON
// grammar; and where all workgroups have such tokens, they are not taken while others still walk: 32,000 tokens over the
// statement grammar five and eight times over 677 and 1,028 us, each by its own workgroup 595 and 845.  (A workgroup that keeps
// its own up to twice the average: 600 and 850, but who leaves its own to all then waits behind those who do not, random
// grammars up to 1.7 times as long.  Lists offered by each workgroup to those that are through with their walk save the
// launch, but these are gone by then, or all at one cursor: 1,620 us, 10,900, and 32,000 tokens that share no sets 7,140 where
// it is 420.)
__global__ __launch_bounds__(kAloneThreads) void displacement_alone_kernel(DisplacementArgs a) {
    __shared__ AloneLds A;
    const int count = min(a.hdr->retry_count[0], a.V), grid = (int)gridDim.x, block = (int)blockIdx.x;
    if (block >= count) return;
    const int mine = (count - 1 - block) / grid + 1;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    if (threadIdx.x == 0) A.next[0] = A.next[1] = A.left = 0;
    __syncthreads();
    // the next entry of the workgroup's list `which`, -1 behind its end
    auto take = [&](int which, int n) -> int {
        int i = 0;
        if (lane == 0) i = (int)atomicAdd(&A.next[which], 1u);
        i = __builtin_amdgcn_readfirstlane(i);
        if (i >= n) return -1;
        const int32_t *entry = a.retry_list[which] + block + (int64_t)i * grid;  // (of the second: another wave of the workgroup wrote it)
        return __builtin_amdgcn_readfirstlane(__hip_atomic_load(entry, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP));
    };
    if (wave < AloneLds::kFirst)
        for (int t; (t = take(0, mine)) >= 0;) {
            const bool crosses = token_displacement<uint8_t, kLists1<uint8_t>, kLists1<uint8_t>, kFrontier1, false>(a, t, A.first[wave], false);
            if (crosses && lane == 0) a.retry_list[1][block + (int64_t)atomicAdd(&A.left, 1u) * grid] = t;
            wave_order();
        }
    __syncthreads();
    const int left = (int)__builtin_amdgcn_readfirstlane(A.left);
    if (wave >= AloneLds::kLast || wave >= left) return;
    AloneLds::Last &lds = A.last[wave];
    const bool adj_in_lds = a.g.N * a.g.W <= kAdjLdsWords;
    if (adj_in_lds)
        for (int i = lane; i < a.g.N * a.g.W; i += 64) lds.adj[i] = a.adj[i];
    for (int t; (t = take(1, left)) >= 0;) {
        token_displacement<uint8_t, kIn2, kOut2, kFrontier2, true>(a, t, lds, adj_in_lds);
        wave_order();
    }
}

// ---- more than 255 symbols ----------------------------------------------------------------

// Entries of a long list that a workgroup of the second pass takes at a time.  The atomics on the list's one cursor are
// served one after the other, 14 ns each, which is more than a short token's share of the chip: 32,000 entries over 500
// symbols 3.45 ms in fours (3.73 one by one, 4.49 dealt out beforehand).  The few long tokens of the third pass are taken
// one by one.
constexpr int kRetryChunk = 4;

// Persistent workgroups of one wave take retry list LIST entry by entry; what they cannot finish goes to list HAND_ON
// (none if negative)
template <typename Sym, int MAX_IN, int MAX_OUT, int FRONTIER, int LIST, int HAND_ON, bool STAGE>
__global__ __launch_bounds__(64) void displacement_retry_kernel(DisplacementArgs a) {
    __shared__ TokenLds<Sym, Rec<Sym, MAX_IN, MAX_OUT>, FRONTIER, STAGE> lds;
    __shared__ int next_item;
    const int count = min(a.hdr->retry_count[LIST], a.V);
    if (count == 0) return;
    const bool adj_in_lds = STAGE && a.g.N * a.g.W <= kAdjLdsWords;
    if (adj_in_lds)
        for (int i = threadIdx.x; i < a.g.N * a.g.W; i += 64) lds.adj[i] = a.adj[i];
    const int chunk = HAND_ON < 0 ? 1 : min(max(count / (int)gridDim.x, 1), kRetryChunk);
    for (;;) {
        if (threadIdx.x == 0) next_item = atomicAdd(&a.hdr->retry_next[LIST], chunk);
        __syncthreads();
        const int first = next_item;
        __syncthreads();
        if (first >= count) break;  // the same for every lane
        for (int i = first; i < min(first + chunk, count); ++i) {
            const int t = a.retry_list[LIST][i];
            const bool crosses = token_displacement<Sym, MAX_IN, MAX_OUT, FRONTIER, STAGE>(a, t, lds, adj_in_lds);
            if (HAND_ON >= 0 && crosses && threadIdx.x == 0)
                a.retry_list[HAND_ON < 0 ? 0 : HAND_ON][atomicAdd(&a.hdr->retry_count[HAND_ON < 0 ? 0 : HAND_ON], 1)] = t;
        }
    }
}

template <typename Sym, int MAX_IN, int MAX_OUT, int FRONTIER, int LIST, int HAND_ON, bool STAGE>
int launch_retry(const DisplacementArgs &a, int n_cu, hipStream_t stream) {
    // as many one-wave workgroups as the LDS of all compute units holds at once
    const size_t lds = sizeof(TokenLds<Sym, Rec<Sym, MAX_IN, MAX_OUT>, FRONTIER, STAGE>);
    const int64_t per_cu = std::min<int64_t>(32, (160 * 1024) / lds);
    hipLaunchKernelGGL((displacement_retry_kernel<Sym, MAX_IN, MAX_OUT, FRONTIER, LIST, HAND_ON, STAGE>),
                       dim3((unsigned)std::min<int64_t>(a.V, n_cu * std::max<int64_t>(1, per_cu))), dim3(64), 0, stream, a);
    return check_launch();
}

// Every token onto the first list; with a grammar that breaks the rules, every token's outputs instead.
__global__ void hand_all_kernel(DisplacementArgs a) {
    const int step = gridDim.x * blockDim.x, first = blockIdx.x * blockDim.x + threadIdx.x;
    if (!a.hdr->invalid) {
        for (int t = first; t < a.V; t += step) a.retry_list[0][t] = t;
        if (first == 0) a.hdr->retry_count[0] = a.V;
        return;
    }
    for (int t = first; t < a.V; t += step) {
        a.hash[t] = 0;
        if (a.status) a.status[t] = kStatusBadGrammar;
    }
    const size_t units = (size_t)a.V * a.row_len / 4;
    for (size_t u = first; u < units; u += step) reinterpret_cast<uint2 *>(a.rows)[u] = make_uint2(0, 0);
}

int launch_displacements(const DisplacementArgs &a, int n_cu, hipStream_t stream) {
    if (a.g.N <= kMaxByteSymbols) {
        static_assert(kShMaxSymbols == kMaxByteSymbols, "the shared walk takes every grammar whose symbols fit a byte");
        // a workgroup of sixteen waves per compute unit, the tokens spread evenly
        const int64_t groups = std::min<int64_t>(n_cu, ceil_div(a.V, kShWaves));
        const int per_group = (int)ceil_div(a.V, groups);
        const unsigned grid = (unsigned)ceil_div(a.V, per_group);
        if (aligned_to(a.rows, 16))
            hipLaunchKernelGGL(displacement_shared_kernel<true>, dim3(grid), dim3(kShThreads), 0, stream, a, per_group);
        else
            hipLaunchKernelGGL(displacement_shared_kernel<false>, dim3(grid), dim3(kShThreads), 0, stream, a, per_group);
        CFGZIP_TRY(check_launch());
        hipLaunchKernelGGL(displacement_alone_kernel, dim3((unsigned)std::min<int64_t>(n_cu, a.V)), dim3(kAloneThreads), 0, stream, a);
        return check_launch();
    }
    // more symbols than a shared cell holds: every token is taken alone
    using Sym = uint16_t;
    hipLaunchKernelGGL(hand_all_kernel, dim3((unsigned)std::min<int64_t>(1024, ceil_div(a.V, 256))), dim3(256), 0, stream, a);
    CFGZIP_TRY(check_launch());
    CFGZIP_TRY((launch_retry<Sym, kLists1<Sym>, kLists1<Sym>, kFrontier1, 0, 1, false>(a, n_cu, stream)));
    return launch_retry<Sym, kIn2, kOut2, kFrontier2, 1, -1, true>(a, n_cu, stream);
}

int check_grammar_args(const uint16_t *prod_head, const uint8_t *prod_byte, const int32_t *prod_body_off,
                       const uint16_t *prod_body, int32_t body_total, int32_t P, int32_t N) {
    if (!prod_head || !prod_byte || !prod_body_off) return CFGZIP_E_INVALID;
    if (P <= 0 || N <= 0 || N > kMaxSymbols || body_total < 0) return CFGZIP_E_INVALID;
    if (body_total > 0 && !prod_body) return CFGZIP_E_INVALID;
    if (!aligned_to(prod_head, 2) || !aligned_to(prod_body_off, 4) || !aligned_to(prod_body, 2))
        return CFGZIP_E_INVALID;
    return CFGZIP_OK;
}

}  // namespace
}  // namespace cfgzip

using namespace cfgzip;

extern "C" size_t cfgzip_displacements_workspace_bytes(int32_t V, int32_t N, int32_t P) {
    if (V < 0 || N <= 0 || N > kMaxSymbols || P <= 0) return 0;
    return carve_grammar_ws(nullptr, N, V, P).bytes;
}

extern "C" int cfgzip_stack_adjacency(const uint16_t *prod_head, const uint8_t *prod_byte,
                                      const int32_t *prod_body_off, const uint16_t *prod_body,
                                      int32_t body_total, int32_t P, int32_t N, int32_t *adj_out,
                                      int32_t *invalid_out, void *ws, size_t ws_bytes, void *stream_) {
    CFGZIP_TRY(check_grammar_args(prod_head, prod_byte, prod_body_off, prod_body, body_total, P, N));
    if (!adj_out || !aligned_to(adj_out, 4) || !aligned_to(invalid_out, 4)) return CFGZIP_E_INVALID;
    if (!ws || !aligned_to(ws, 256)) return CFGZIP_E_WORKSPACE;
    GrammarWorkspace w = carve_grammar_ws(ws, N, 0, P);
    if (ws_bytes < w.bytes) return CFGZIP_E_WORKSPACE;
    hipStream_t stream = static_cast<hipStream_t>(stream_);
    Grammar g{prod_head, prod_byte, prod_body_off, prod_body, P, N, (int)ceil_div(N, 32), body_total};
    CFGZIP_TRY(enqueue_grammar_tables(g, w, false, stream));
    const size_t words = (size_t)N * g.W;
    hipLaunchKernelGGL(copy_words_kernel, dim3((unsigned)std::min<int64_t>(1024, ceil_div((int64_t)words, 256))),
                       dim3(256), 0, stream, w.adj, adj_out, words);
    CFGZIP_TRY(check_launch());
    if (invalid_out) {
        hipLaunchKernelGGL(copy_words_kernel, dim3(1), dim3(64), 0, stream,
                           reinterpret_cast<const uint32_t *>(&w.hdr->invalid), invalid_out,
                           (size_t)1);
        CFGZIP_TRY(check_launch());
    }
    return CFGZIP_OK;
}

extern "C" int cfgzip_displacements(const uint8_t *tok_bytes, const int64_t *tok_off, int32_t V,
                                    const uint16_t *prod_head, const uint8_t *prod_byte,
                                    const int32_t *prod_body_off, const uint16_t *prod_body,
                                    int32_t body_total, int32_t P, int32_t N, uint16_t *rows_out,
                                    int32_t row_len, uint64_t *hash_out, int32_t *status_out,
                                    uint64_t hash_seed, void *ws, size_t ws_bytes, void *stream_) {
    CFGZIP_TRY(check_grammar_args(prod_head, prod_byte, prod_body_off, prod_body, body_total, P, N));
    if (!tok_off || !rows_out || !hash_out || V <= 0) return CFGZIP_E_INVALID;
    if (row_len < kRowChunk || row_len > kMaxRowLen || row_len % kRowChunk) return CFGZIP_E_INVALID;
    if (!aligned_to(tok_off, 8) || !aligned_to(rows_out, 8) || !aligned_to(hash_out, 8) ||
        !aligned_to(status_out, 4))
        return CFGZIP_E_INVALID;
    if (!ws || !aligned_to(ws, 256)) return CFGZIP_E_WORKSPACE;
    GrammarWorkspace w = carve_grammar_ws(ws, N, V, P);
    if (ws_bytes < w.bytes) return CFGZIP_E_WORKSPACE;
    hipStream_t stream = static_cast<hipStream_t>(stream_);
    Grammar g{prod_head, prod_byte, prod_body_off, prod_body, P, N, (int)ceil_div(N, 32), body_total};
    CFGZIP_TRY(enqueue_grammar_tables(g, w, N <= kMaxByteSymbols, stream));
    DisplacementArgs a{};
    a.g = g;
    a.hdr = w.hdr;
    a.byte_off = w.byte_off;
    a.pair_first = w.pair_first;
    a.prod_short = w.prod_short;
    a.byte_like = w.byte_like;
    a.prod_packed = w.prod_packed;
    a.adj = w.adj;
    a.tok_bytes = tok_bytes;
    a.tok_off = tok_off;
    a.rows = rows_out;
    a.hash = hash_out;
    a.status = status_out;
    a.retry_list[0] = w.retry_list[0];
    a.retry_list[1] = w.retry_list[1];
    a.seed = hash_seed;
    a.V = V;
    a.row_len = row_len;
    int n_cu = 256;
    {
        int dev = 0;
        CFGZIP_TRY(check_hip(hipGetDevice(&dev)));
        CFGZIP_TRY(check_hip(hipDeviceGetAttribute(&n_cu, hipDeviceAttributeMultiprocessorCount, dev)));
        if (n_cu <= 0) n_cu = 256;
    }
    return launch_displacements(a, n_cu, stream);
}
