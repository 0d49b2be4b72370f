// Parent events: events that carry the keys of every quantifier level but the
// innermost one join the cluster u^D of every instance D under their parent,
// at their place in trace order (the proxy-cache case study of Section 5,
// where per-video cache events bear on every request of the video).
//
// After the radix sort the own events (full value vectors, kind bit 0) come
// first, sorted by (key, trace index), and the parent events (kind bit 1) after
// them, sorted by (parent prefix, trace index): the "parent array" P.  The map
// scan (mapscan.hip) runs over the own events; what it needs to merge the
// parent events in is prepared here:
//   * the bound of every own event: the number of entries of P ordered before
//     it by (prefix, trace index).  An instance's own events split its
//     parent's run of P at their bounds into gaps;
//   * for every entry of P and property, the state from q0 through its
//     parent's run up to and with the entry (what an instance whose first own
//     event follows it starts from) and the map of the run's rest from the
//     entry on (what an instance whose last own event precedes it ends with),
//     so that the two gaps every instance has cost one look-up each;
//   * a segment tree over P of composed class maps (level L node q composes
//     the entries [q 2^L, (q+1) 2^L)), built eight levels per launch in LDS,
//     for the gaps inside an instance.
#include "parent.h"

namespace ltl4c {

namespace {

// first index in [lo, hi) of `key_at` whose key is not below `target` (hi if none)
template <typename K>
__device__ __forceinline__ uint32_t lower_bound(K key_at, uint32_t lo, uint32_t hi, uint64_t target) {
    while (lo < hi) {
        const uint32_t mid = (lo + hi) >> 1;
        if (key_at(mid) < target) lo = mid + 1;
        else hi = mid;
    }
    return lo;
}

// the same by a whole wave over the parent array: 64 probes a round trip
__device__ __forceinline__ uint32_t wave_lower_bound(const ParentArgs& a, const uint64_t* par, uint32_t k,
                                                     uint64_t target) {
    const uint32_t lane = threadIdx.x & 63u;
    uint32_t lo = 0, hi = k;
    while (lo < hi) {
        const uint32_t step = (hi - lo + 63u) / 64u;
        const uint64_t at = (uint64_t)lo + (uint64_t)(lane + 1u) * step - 1u;    // the last of this lane's part
        const uint32_t n = (uint32_t)__popcll(__ballot(at < hi && pe_key(a, par[at < hi ? at : hi - 1u]) < target));
        lo += n * step;                            // parts [0, n) are below; the bound is in part n
        hi = min(hi, lo + step - 1u);
    }
    return lo;
}

__device__ __forceinline__ void load_class_maps(const ParentArgs& a, uint32_t p, uint32_t (*s_cm)[4]) {
    if (threadIdx.x < 64) s_cm[threadIdx.x >> 2][threadIdx.x & 3] = a.plan->prop[p].bmap[threadIdx.x >> 2][threadIdx.x & 3];
    __syncthreads();
}

}  // namespace

// Levels L0+1 .. L0+nlev of the segment tree of property blockIdx.y, from
// level L0: each block takes 256 level-L0 nodes and halves them in LDS.  A
// missing right child counts as the identity.
__global__ __launch_bounds__(256) void k_pe_tree(ParentArgs a, uint32_t L0, uint32_t nlev) {
    __shared__ uint4 s[256];
    __shared__ uint32_t s_cm[16][4];
    const uint32_t p = blockIdx.y;
    load_class_maps(a, p, s_cm);
    const uint32_t k = *a.n_par;
    const uint64_t* par = a.words + *a.n_own;
    const uint64_t cnt0 = ((uint64_t)k + (1ull << L0) - 1) >> L0;
    const uint32_t t = threadIdx.x;
    auto put = [&](uint32_t i, const BMap<4>& m) { s[i] = make_uint4(m.d[0], m.d[1], m.d[2], m.d[3]); };
    auto get = [&](uint32_t i) {
        const uint4 v = s[i];
        return BMap<4>{{v.x, v.y, v.z, v.w}};
    };
    for (uint64_t b = blockIdx.x; b * 256 < cnt0; b += gridDim.x) {
        const uint64_t q = b * 256 + t;
        BMap<4> m = bm_identity<4>();
        if (q < cnt0)
            m = L0 == 0 ? bm_load<4>(s_cm[(uint32_t)par[q] & a.class_mask])
                        : pe_unpack<4>(a.tree[a.tree_off[L0] + (uint64_t)p * a.tree_cnt[L0] + q]);
        for (uint32_t l = 1; l <= nlev; ++l) {
            if (t < (256u >> (l - 1))) put(t, m);
            __syncthreads();
            if (t < (256u >> l)) {
                m = bm_compose<4>(get(2 * t + 1), get(2 * t));
                const uint32_t L = L0 + l;
                const uint64_t node = b * (256u >> l) + t;
                if (node < (((uint64_t)k + (1ull << L) - 1) >> L))
                    a.tree[a.tree_off[L] + (uint64_t)p * a.tree_cnt[L] + node] = pe_pack(m);
            }
            __syncthreads();
        }
    }
}

// Per entry of the parent array and property (blockIdx.y): the state from q0
// through its run up to and with it, and the map of the run from it on.
__global__ __launch_bounds__(256) void k_pe_affix(ParentArgs a) {
    __shared__ uint32_t s_cm[16][4];
    const uint32_t p = blockIdx.y;
    load_class_maps(a, p, s_cm);
    const uint32_t k = *a.n_par, q0 = a.plan->prop[p].q0;
    const uint64_t* par = a.words + *a.n_own;
    for (uint32_t e = blockIdx.x * blockDim.x + threadIdx.x; e < k; e += gridDim.x * blockDim.x) {
        const uint64_t pf = pe_prefix(a, par[e]);
        auto prefix_at = [&](uint32_t i) { return pe_prefix(a, par[i]); };
        // the run's ends, by doubling steps away from e
        uint32_t lo = e, step = 1;               // entries [lo, e] are of the run
        while (lo >= step && prefix_at(lo - step) == pf) lo -= step, step <<= 1;
        const uint32_t rs = lower_bound(prefix_at, lo >= step ? lo - step + 1u : 0u, lo, pf);
        uint32_t hi = e;                         // entries [e, hi] are of the run
        step = 1;
        while (step < k - hi && prefix_at(hi + step) == pf) hi += step, step <<= 1;
        const uint32_t re = lower_bound(prefix_at, hi + 1u, step < k - hi ? hi + step : k, pf + 1u);
        a.pre[(uint64_t)p * a.cap + e] = (uint8_t)bm_at<4>(pe_range<4>(a, s_cm, par, p, rs, e + 1u), q0);
        a.suf[(uint64_t)p * a.cap + e] = pe_pack(pe_range<4>(a, s_cm, par, p, e, re));
    }
}

// The bound of every own event.  A block's 4,096 own events are of few
// consecutive parents, so it first finds the part of the parent array that
// belongs to them (64-way searches by two waves) and, when that part is short
// (it nearly always is), copies its keys to LDS.  Each thread then finds its
// parents' runs and searches for its 16 events together, so that the steps of
// one search hide those of the others: 47.5 us for 10M events (1.5M: 16.7 us).
// With one search per event and property inside a scan of its own, dependent
// memory trips in a row, the two passes over 10M events and two properties took
// 66 + 301 us (1.5M: 34 + 197 us) besides the map scan.
constexpr uint32_t kPeStage = 2048;
template <bool STAGED>
__device__ __forceinline__ void pe_bounds_run(const ParentArgs& a, const uint64_t* s_key, const uint64_t* part,
                                              uint32_t b0, uint32_t m, uint64_t my0, uint32_t cnt) {
    auto key_at = [&](uint32_t i) { return STAGED ? s_key[i] : pe_key(a, part[i]); };
    uint64_t w[kPeItems];
    const uint4* src = reinterpret_cast<const uint4*>(a.words + (cnt ? my0 : 0));   // (padded past the last word)
#pragma unroll
    for (int q = 0; q < kPeItems / 2; ++q) {
        const uint4 v = src[q];
        w[2 * q] = (uint64_t)v.x | ((uint64_t)v.y << 32);
        w[2 * q + 1] = (uint64_t)v.z | ((uint64_t)v.w << 32);
    }
    uint32_t change = 0;                           // events whose prefix differs from the one before
#pragma unroll
    for (int j = 0; j < kPeItems; ++j) {
        w[j] = pe_key(a, w[j]);
        if ((uint32_t)j < cnt && (j == 0 || w[j] >> a.ibits != w[j - 1] >> a.ibits)) change |= 1u << j;
    }
    uint32_t lo[kPeItems], hi[kPeItems];
#pragma unroll
    for (int j = 0; j < kPeItems; ++j) lo[j] = hi[j] = 0;
    uint32_t re = 0;
    for (uint32_t rest = change; rest != 0u; rest &= rest - 1u) {
        const uint32_t j0 = (uint32_t)__ffs(rest) - 1u;
        const uint64_t pf = pe_prefix(a, a.words[my0 + j0]);
        const uint32_t rs = lower_bound(key_at, re, m, pf << a.ibits);
        re = lower_bound(key_at, rs, m, (pf + 1u) << a.ibits);
#pragma unroll
        for (int j = 0; j < kPeItems; ++j)
            if ((uint32_t)j >= j0) {               // (later prefixes overwrite their events)
                lo[j] = rs;
                hi[j] = re;
            }
    }
    bool more = true;
    while (more) {
        more = false;
#pragma unroll
        for (int j = 0; j < kPeItems; ++j) {
            if (lo[j] >= hi[j]) continue;
            const uint32_t mid = (lo[j] + hi[j]) >> 1;
            if (key_at(mid) < w[j]) lo[j] = mid + 1;
            else hi[j] = mid;
            more = more || lo[j] < hi[j];
        }
    }
    uint32_t out[kPeItems];
#pragma unroll
    for (int j = 0; j < kPeItems; ++j) {
        const uint64_t pf = w[j] >> a.ibits;
        const uint32_t g = lo[j];
        out[j] = b0 + g;
        if (g == 0 || key_at(g - 1u) >> a.ibits != pf) out[j] |= kPeNoneBefore;
        if (g >= m || key_at(g) >> a.ibits != pf) out[j] |= kPeNoneAfter;
    }
    if (cnt == kPeItems) {
        uint4* dst = reinterpret_cast<uint4*>(a.bound + my0);
#pragma unroll
        for (int q = 0; q < kPeItems / 4; ++q) dst[q] = make_uint4(out[4 * q], out[4 * q + 1], out[4 * q + 2], out[4 * q + 3]);
    } else {
#pragma unroll
        for (int j = 0; j < kPeItems; ++j)
            if ((uint32_t)j < cnt) a.bound[my0 + j] = out[j];
    }
}

__global__ __launch_bounds__(kPeThreads) void k_pe_bounds(ParentArgs a) {
    __shared__ uint64_t s_key[kPeStage];
    __shared__ uint32_t s_part[2];
    const uint32_t n_own = *a.n_own, k = *a.n_par;
    const uint64_t* par = a.words + n_own;
    const uint64_t base = (uint64_t)blockIdx.x * kPeTile;
    if (base >= n_own) return;
    const uint32_t tid = threadIdx.x, wave = tid >> 6;
    if (wave < 2) {
        const uint64_t at = wave == 0 ? base : min<uint64_t>(base + kPeTile, n_own) - 1u;
        const uint32_t b = wave_lower_bound(a, par, k, (pe_prefix(a, a.words[at]) + wave) << a.ibits);
        if ((tid & 63u) == 0) s_part[wave] = b;
    }
    __syncthreads();
    // (own events in order give s_part[1] >= b0; m bounds every read below, so it
    // does not rest on that)
    const uint32_t b0 = s_part[0], m = max(s_part[1], b0) - b0;
    const uint64_t my0 = base + (uint64_t)tid * kPeItems;
    const uint32_t cnt = my0 < n_own ? (uint32_t)min<uint64_t>(kPeItems, n_own - my0) : 0u;
    if (m <= kPeStage) {
        for (uint32_t i = tid; i < m; i += kPeThreads) s_key[i] = pe_key(a, par[b0 + i]);
        __syncthreads();
        if (cnt) pe_bounds_run<true>(a, s_key, par + b0, b0, m, my0, cnt);
    } else if (cnt) {
        pe_bounds_run<false>(a, s_key, par + b0, b0, m, my0, cnt);
    }
}

hipError_t launch_parent_tree(const ParentArgs& a, uint32_t level0, uint32_t nlev, uint64_t max_nodes0,
                              hipStream_t s) {
    const uint64_t want = (max_nodes0 + 255) / 256;
    const uint32_t blocks = (uint32_t)(want < 1024 ? (want ? want : 1) : 1024);
    hipLaunchKernelGGL(k_pe_tree, dim3(blocks, a.n_props), dim3(256), 0, s, a, level0, nlev);
    return hipGetLastError();
}

hipError_t launch_parent_affix(const ParentArgs& a, uint64_t max_entries, hipStream_t s) {
    const uint64_t want = (max_entries + 255) / 256;
    hipLaunchKernelGGL(k_pe_affix, dim3((uint32_t)(want < 1024 ? (want ? want : 1) : 1024), a.n_props), dim3(256), 0, s, a);
    return hipGetLastError();
}

hipError_t launch_parent_bounds(const ParentArgs& a, uint64_t max_own, hipStream_t s) {
    const uint64_t tiles = (max_own + kPeTile - 1) / kPeTile;
    hipLaunchKernelGGL(k_pe_bounds, dim3((uint32_t)(tiles ? tiles : 1)), dim3(kPeThreads), 0, s, a);
    return hipGetLastError();
}

}  // namespace ltl4c
