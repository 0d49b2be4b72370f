// Parent events (see parent.hip): what the kernels over the parent array and
// the map scan share.
#pragma once
#include "internal.h"
#include "maps.h"

namespace ltl4c {

// bound of an own event: the parent-array entries ordered before it, and
// whether none of its parent's entries is before it, or none is after it
constexpr uint32_t kPeIndex = (1u << 30) - 1u, kPeNoneBefore = 1u << 30, kPeNoneAfter = 1u << 31;

// (prefix, trace index) of a sorted word; the parent array is in this order
__device__ __forceinline__ uint64_t pe_prefix(const ParentArgs& a, uint64_t w) {
    return (w >> a.prefix_shift) & a.prefix_mask;
}
__device__ __forceinline__ uint64_t pe_key(const ParentArgs& a, uint64_t w) {
    return (pe_prefix(a, w) << a.ibits) | ((w >> a.cbits) & a.index_mask);
}

// Maps in memory take 4 bits per state: state q's image is nibble q.
template <int MW>
__device__ __forceinline__ BMap<MW> pe_unpack(const uint2& v) {
    BMap<MW> r;
#pragma unroll
    for (int i = 0; i < MW; ++i) {
        uint32_t x = ((i < 2 ? v.x : v.y) >> (16 * (i & 1))) & 0xFFFFu;
        x = (x | (x << 8)) & 0x00FF00FFu;
        r.d[i] = (x | (x << 4)) & 0x0F0F0F0Fu;
    }
    return r;
}
__device__ __forceinline__ uint32_t pe_pack4(uint32_t x) {       // nibbles at bits 0, 8, 16, 24
    x = (x | (x >> 4)) & 0x00FF00FFu;
    return (x | (x >> 8)) & 0xFFFFu;
}
__device__ __forceinline__ uint2 pe_pack(const BMap<4>& m) {
    return make_uint2(pe_pack4(m.d[0]) | (pe_pack4(m.d[1]) << 16), pe_pack4(m.d[2]) | (pe_pack4(m.d[3]) << 16));
}

// Composition of the class maps of parent-array entries [l, r), in order, for
// property p (cm: its class maps).  Up to kPeShortGap entries: their words are
// loaded together; longer ranges walk the segment tree, whose level-L node q
// composes the entries [q 2^L, (q + 1) 2^L).
template <int MW>
__device__ __forceinline__ BMap<MW> pe_range(const ParentArgs& a, const uint32_t (*cm)[MW], const uint64_t* par,
                                             uint32_t p, uint32_t l, uint32_t r) {
    if (r - l <= (uint32_t)kPeShortGap) {
        uint32_t c[kPeShortGap];
#pragma unroll
        for (int j = 0; j < kPeShortGap; ++j) c[j] = l < r ? (uint32_t)par[min(l + (uint32_t)j, r - 1u)] & a.class_mask : 0u;
        BMap<MW> m = bm_identity<MW>();
#pragma unroll
        for (int j = 0; j < kPeShortGap; ++j)
            if (l + (uint32_t)j < r) m = bm_compose<MW>(bm_load<MW>(cm[c[j]]), m);
        return m;
    }
    auto node = [&](uint32_t L, uint32_t q) {
        if (L == 0) return bm_load<MW>(cm[(uint32_t)par[q] & a.class_mask]);
        return pe_unpack<MW>(a.tree[a.tree_off[L] + (uint64_t)p * a.tree_cnt[L] + q]);
    };
    BMap<MW> left = bm_identity<MW>(), right = bm_identity<MW>();
    uint32_t L = 0;
    while (l < r) {
        if (l & 1u) left = bm_compose<MW>(node(L, l++), left);
        if (r & 1u) right = bm_compose<MW>(right, node(L, --r));
        l >>= 1;
        r >>= 1;
        ++L;
    }
    return bm_compose<MW>(right, left);
}

}  // namespace ltl4c
