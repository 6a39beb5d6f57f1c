// Device-side pieces of cfgzip_build_classes that both ways of grouping share: the counters the
// host reads, and the exact comparison of two tokens' signatures from each source.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "walk_device.hpp"

namespace cfgzip {
namespace {

struct Counters {
    int32_t unresolved;
    int32_t num_classes;
    int32_t store_state;  // of the walk store handed in: 0 usable, 1 not this call's, 2 overflowed
    int32_t other_rows;   // links between tokens of different image rows, listed for the kernel after
    int32_t no_room;      // a bucket of the hash table was too small for its classes
    int32_t pad[3];
};
constexpr int kStoreForeign = 1, kStoreOverflowed = 2;

// ---------------------------------------------------------------- comparing two tokens' signatures

__device__ __forceinline__ uint64_t hash_part(uint64_t key) { return key >> 8; }

// What the comparisons read when the walk vectors of cfgzip_signatures are at hand.
struct StoreSource {
    Tables T;
    WalkStoreView store;
    int32_t V, S;
};

// 0 if the store holds this call's vectors, `stride` entries per token, else why not.
__device__ __forceinline__ int walk_store_state(const StoreSource &s, uint32_t &stride) {
    const WalkStore hdr = *s.store.header;
    stride = hdr.stride;
    if (hdr.magic != kWalkStoreMagic || hdr.V != s.V || hdr.S != s.S ||
        (hdr.stride != walk_store_stride(s.S, kWalkStoreMaxStride) &&
         hdr.stride != walk_store_stride(s.S, kWalkStoreSmallStride)))
        return kStoreForeign;
    return hdr.overflow ? kStoreOverflowed : 0;
}

// Image row of a token as the store has it (256: the empty token, whose signature is the
// identity and whose vector is not kept).
__device__ __forceinline__ uint32_t store_row(const StoreSource &s, int32_t tok) {
    return min(walk_row_of(s.store.wrow[tok]), 256u);
}

// Two tokens with the same image row < 256: idx[row] is onto, so their signatures are
// equal iff their walk vectors are.  One thread, 16 bytes at a time (the padding behind a
// vector is zero on both sides).
__device__ __forceinline__ bool store_same_row_differ(const StoreSource &s, uint32_t stride, int32_t ta, int32_t tb) {
    const uint4 *wa = reinterpret_cast<const uint4 *>(s.store.wvec + (size_t)ta * stride);
    const uint4 *wb = reinterpret_cast<const uint4 *>(s.store.wvec + (size_t)tb * stride);
    const uint32_t n16 = min(walk_units_of(s.store.wrow[ta]), stride / 8u);  // the same for both: one row
    bool diff = false;
    constexpr int kAhead = 4;  // independent 16-byte loads in flight per side
    for (uint32_t k0 = 0; k0 < n16; k0 += kAhead) {
        uint4 x[kAhead], y[kAhead];
#pragma unroll
        for (int u = 0; u < kAhead; ++u) {
            const uint32_t k = min(k0 + u, n16 - 1);  // repeats the last one past the end
            x[u] = wa[k];
            y[u] = wb[k];
        }
#pragma unroll
        for (int u = 0; u < kAhead; ++u)
            diff |= (x[u].x != y[u].x) | (x[u].y != y[u].y) | (x[u].z != y[u].z) | (x[u].w != y[u].w);
    }
    return diff;
}

// Two tokens with different image rows (neighbours at the border between two first bytes inside
// a segment, or an empty token): sig[q] = w[idx[row][q]] has to be compared for every q; the
// empty token's signature is sig[q] = q.  One wave; both vectors are staged in the wave's LDS
// buffers la, lb (kWalkStoreMaxStride entries each).  Returns whether any entry differs
// (wave-uniform).  `part` of `parts`: the wave looks only at every parts-th stretch of 512 states,
// starting with stretch `part` (several waves then share one pair; S >= 8 only).
__device__ __forceinline__ bool store_other_row_differ(const StoreSource &s, uint32_t stride, int32_t ta, int32_t tb,
                                                       uint32_t ra, uint32_t rb, uint16_t *la,
                                                       uint16_t *lb, int part = 0, int parts = 1) {
    const int lane = threadIdx.x & 63;
    const int S = s.S;
    const bool ida = ra == 256u, idb = rb == 256u;
    if (ida && idb) return false;
    if (part * 512 >= S) return false;  // nothing of this pair falls to this wave
    // positions in a kept vector are below the row's image size, which is at most the stride in a
    // store that has not overflowed; the bound keeps a corrupt index inside the staged vector
    const uint32_t na = stride, nb = stride;
    const uint16_t *ia = s.T.idx + (size_t)ra * S, *ib = s.T.idx + (size_t)rb * S;
    // 16 bytes of each index row per lane and step (the identity row is not read); the first are asked for together
    // with the vectors
    constexpr int kAhead = 2;
    const bool vec = S >= 8;
    u32x4_any xa[kAhead], xb[kAhead];
    auto fetch = [&](int q0) {
#pragma unroll
        for (int u = 0; u < kAhead; ++u) {
            const int q = min(q0 + 512 * parts * u, S - 8);  // the last eight where fewer are left
            xa[u] = xb[u] = u32x4_any{0u, 0u, 0u, 0u};
            if (!ida) xa[u] = *reinterpret_cast<const u32x4_any *>(ia + q);
            if (!idb) xb[u] = *reinterpret_cast<const u32x4_any *>(ib + q);
        }
    };
    const int first = lane * 8 + 512 * part;
    if (vec) fetch(first);
    {
        // lanes 0..31 copy vector a, lanes 32..63 vector b, 16 bytes each and round
        const bool second = lane >= 32;
        const uint16_t *src = s.store.wvec + (size_t)(second ? tb : ta) * stride;
        if (!(second ? idb : ida))
            for (uint32_t u = lane & 31; u * 8 < stride; u += 32)
                reinterpret_cast<uint4 *>(second ? lb : la)[u] = reinterpret_cast<const uint4 *>(src)[u];
    }
    // the staged vectors are read below as 16-bit entries by other lanes of this wave
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    bool d = false;
    auto entry_a = [&](uint32_t q, uint32_t j) -> uint32_t { return ida ? q : (j < na ? la[j] : 0xFFFFu); };
    auto entry_b = [&](uint32_t q, uint32_t j) -> uint32_t { return idb ? q : (j < nb ? lb[j] : 0xFFFFu); };
    if (vec) {
        for (int q0 = first; q0 < S; q0 += 512 * parts * kAhead) {
            if (q0 != first) fetch(q0);
#pragma unroll
            for (int u = 0; u < kAhead; ++u) {
                if (q0 + 512 * parts * u >= S) continue;
                const int q = min(q0 + 512 * parts * u, S - 8);
                const uint32_t ja[8] = {xa[u].x & 0xFFFFu, xa[u].x >> 16, xa[u].y & 0xFFFFu, xa[u].y >> 16,
                                        xa[u].z & 0xFFFFu, xa[u].z >> 16, xa[u].w & 0xFFFFu, xa[u].w >> 16};
                const uint32_t jb[8] = {xb[u].x & 0xFFFFu, xb[u].x >> 16, xb[u].y & 0xFFFFu, xb[u].y >> 16,
                                        xb[u].z & 0xFFFFu, xb[u].z >> 16, xb[u].w & 0xFFFFu, xb[u].w >> 16};
#pragma unroll
                for (int e = 0; e < 8; ++e) d |= entry_a(q + e, ja[e]) != entry_b(q + e, jb[e]);
            }
        }
    } else {
        for (int q = lane; q < S; q += 64)
            d |= entry_a(q, ida ? 0u : (uint32_t)ia[q]) != entry_b(q, idb ? 0u : (uint32_t)ib[q]);
    }
    const bool any = __ballot(d) != 0ull;
    __builtin_amdgcn_wave_barrier();  // the next pair restages la, lb
    return any;
}

// Stored signature rows of two tokens, one wave.
__device__ __forceinline__ bool rows_differ(const uint16_t *__restrict__ sig, int S, bool vec,
                                            int32_t ta, int32_t tb) {
    const int lane = threadIdx.x & 63;
    const uint16_t *a = sig + (size_t)ta * S;
    const uint16_t *b = sig + (size_t)tb * S;
    bool diff = false;
    if (vec) {
        const uint4 *a4 = reinterpret_cast<const uint4 *>(a);
        const uint4 *b4 = reinterpret_cast<const uint4 *>(b);
        for (int j = lane; j < S / 8; j += 64) {
            const uint4 x = a4[j], y = b4[j];
            diff |= (x.x != y.x) | (x.y != y.y) | (x.z != y.z) | (x.w != y.w);
        }
    } else {
        for (int j = lane; j < S; j += 64) diff |= a[j] != b[j];
    }
    return __ballot(diff) != 0ull;
}

}  // namespace
}  // namespace cfgzip
