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
//     for the gaps inside an instance and for runs that reach over a block.
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

// the same by a whole wave over entries [lo, hi) of the parent array: 64 probes a round trip
__device__ __forceinline__ uint32_t wave_lower_bound(const ParentArgs& a, const uint64_t* par, uint32_t lo, uint32_t hi,
                                                     uint64_t target) {
    const uint32_t lane = threadIdx.x & 63u;
    while (lo < hi) {
        const uint32_t step = (hi - lo + 63u) / 64u;
        const uint64_t at = (uint64_t)lo + (uint64_t)(lane + 1u) * step - 1u;    // the last of this lane's part
        const uint32_t n = (uint32_t)__popcll(__ballot(at < hi && pe_key(a, par[at < hi ? at : hi - 1u]) < target));
        lo += n * step;                            // parts [0, n) are below; the bound is in part n
        hi = min(hi, lo + step - 1u);
    }
    return lo;
}

// pe_range by a whole wave, one round trip: the nodes that cover [l, r), at most
// two of a level, one per lane in the order of their entries (lanes 0..31 the
// left ones upwards, 32..63 the right ones downwards), composed by a scan.
__device__ __forceinline__ BMap<4> wave_range(const ParentArgs& a, const uint32_t (*cm)[4], const uint64_t* par,
                                              uint32_t p, uint32_t l, uint32_t r) {
    const uint32_t lane = threadIdx.x & 63u, L = lane < 32u ? lane : 63u - lane;
    const uint64_t lo = ((uint64_t)l + (1ull << L) - 1ull) >> L, hi = (uint64_t)r >> L;   // whole nodes of level L
    const uint64_t node = lane < 32u ? lo : hi - 1u;
    BMap<4> m = bm_identity<4>();
    if (lo < hi && ((lane < 32u ? lo : hi) & 1u))
        m = L == 0 ? bm_load<4>(cm[(uint32_t)par[node] & a.class_mask])
                   : pe_unpack<4>(a.tree[a.tree_off[L] + (uint64_t)p * a.tree_cnt[L] + node]);
    return bm_bcast<4>(bm_wave_incl_scan<4>(m), 63);
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
    if (*a.n_own == 0) return;                     // no instance to merge them into
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
// through its run up to and with it, and the map of the run from it on.  Both
// are scans over the entries, forwards with the state restarted at a run's
// first entry and backwards with the map restarted at its last: a thread takes
// 8 consecutive entries, the block joins its threads, and where a run reaches
// over the block's edge one wave finds its end and composes that part of it
// from the segment tree.  Each entry so costs a few compositions however long
// its run is.  With two tree walks per entry instead, 2M entries of one parent
// and 16 properties took 3,055 us, 230 us so.
constexpr int kAffixItems = 8;
constexpr uint32_t kAffixTile = 256 * kAffixItems;
__global__ __launch_bounds__(256) void k_pe_affix(ParentArgs a) {
    __shared__ uint32_t s_cm[16][4];
    __shared__ uint32_t s_fwd[4][4], s_bwd[4][4], s_end[4];   // per wave: map forwards; map up to its first run end, if any
    __shared__ uint32_t s_before, s_after[4];
    const uint32_t p = blockIdx.y;
    const uint32_t k = *a.n_par, n_own = *a.n_own, q0 = a.plan->prop[p].q0;
    if (n_own == 0) return;                      // no instance to merge them into
    load_class_maps(a, p, s_cm);
    const uint64_t* par = a.words + n_own;
    const uint32_t tid = threadIdx.x, lane = tid & 63u, w = tid >> 6;
    for (uint64_t base = (uint64_t)blockIdx.x * kAffixTile; base < k; base += (uint64_t)gridDim.x * kAffixTile) {
        const uint64_t my0 = base + tid * kAffixItems;
        const uint32_t cnt = my0 >= k ? 0u : min(k - (uint32_t)my0, (uint32_t)kAffixItems);
        // (unconditional loads of clamped entries: all in flight together)
        uint64_t pf[kAffixItems + 2];            // the prefix before, the run's, and the one after
        uint32_t cls = 0;
#pragma unroll
        for (int j = 0; j < kAffixItems + 2; ++j) {
            const uint64_t at = my0 + j > 0 ? my0 + j - 1u : 0u;
            const uint64_t x = par[at < k ? at : k - 1u];
            pf[j] = pe_prefix(a, x);
            if (j > 0 && j <= kAffixItems) cls |= ((uint32_t)x & a.class_mask) << (4 * (j - 1));
        }
        uint32_t heads = 0, ends = 0;
#pragma unroll
        for (int j = 0; j < kAffixItems; ++j) {
            heads |= (uint32_t)(my0 + j == 0 || pf[j] != pf[j + 1]) << j;
            ends |= (uint32_t)(my0 + j + 1 == k || pf[j + 1] != pf[j + 2]) << j;
        }
        auto map_of = [&](int j) { return bm_load<4>(s_cm[(cls >> (4 * j)) & 15u]); };
        BMap<4> f = bm_identity<4>(), b = bm_identity<4>();
        uint32_t ended = 0;
#pragma unroll
        for (int j = 0; j < kAffixItems; ++j) {
            if ((uint32_t)j >= cnt) continue;
            const BMap<4> c = map_of(j);
            f = bm_compose<4>(c, ((heads >> j) & 1u) ? bm_const<4>(q0) : f);
            if (!ended) b = bm_compose<4>(c, b);
            ended |= (ends >> j) & 1u;
        }
        f = bm_wave_incl_scan<4>(f);
        const BMap<4> fx = bm_wave_shr1<4>(f);   // of the lanes before
#pragma unroll
        for (int off = 1; off < 64; off <<= 1) { // of this lane and those after it, up to a run end
            const BMap<4> later = bm_shfl_down<4>(b, off);
            const uint32_t e = __shfl_down(ended, off, 64);
            if (lane + off < 64u && !ended) {
                b = bm_compose<4>(later, b);
                ended = e;
            }
        }
        BMap<4> bx = bm_shfl_down<4>(b, 1);      // of the lanes after alone
        uint32_t ex = __shfl_down(ended, 1, 64);
        if (lane == 63u) {
            bx = bm_identity<4>();
            ex = 0;
        }
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            if (lane == 63u) s_fwd[w][i] = f.d[i];
            if (lane == 0u) s_bwd[w][i] = b.d[i];
        }
        if (lane == 0u) s_end[w] = ended;
        if (w == 0) {                            // the run that reaches into the tile
            const uint64_t first = __shfl(pf[1], 0, 64);
            uint32_t s = q0;
            if (!(__shfl(heads, 0, 64) & 1u)) {
                const uint32_t rs = wave_lower_bound(a, par, 0u, (uint32_t)base, first << a.ibits);
                s = bm_at<4>(wave_range(a, s_cm, par, p, rs, (uint32_t)base), q0);
            }
            if (lane == 0u) s_before = s;
        } else if (w == 3) {                     // the run that reaches out of it
            BMap<4> m = bm_identity<4>();
            const uint32_t next = min((uint32_t)base + kAffixTile, k);
            const uint64_t last = pe_prefix(a, par[next - 1u]);
            if (next < k && pe_prefix(a, par[next]) == last) {
                const uint32_t re = wave_lower_bound(a, par, next, k, (last + 1u) << a.ibits);
                m = wave_range(a, s_cm, par, p, next, re);
            }
#pragma unroll
            for (int i = 0; i < 4; ++i)
                if (lane == 0u) s_after[i] = m.d[i];
        }
        __syncthreads();
        uint32_t s = s_before;
        for (uint32_t i = 0; i < w; ++i) s = bm_at<4>(bm_load<4>(s_fwd[i]), s);
        s = bm_at<4>(fx, s);
        for (uint32_t i = w + 1; i < 4 && !ex; ++i) {
            bx = bm_compose<4>(bm_load<4>(s_bwd[i]), bx);
            ex = s_end[i];
        }
        if (!ex) bx = bm_compose<4>(bm_load<4>(s_after), bx);
        uint32_t out[2] = {0, 0};
#pragma unroll
        for (int j = 0; j < kAffixItems; ++j) {
            s = bm_at<4>(map_of(j), ((heads >> j) & 1u) ? q0 : s);
            out[j >> 2] |= s << (8 * (j & 3));
        }
        uint8_t* pre = a.pre + (uint64_t)p * a.cap + my0;
        if (cnt == kAffixItems) __builtin_memcpy(pre, out, 8);
        else
            for (uint32_t j = 0; j < cnt; ++j) pre[j] = (uint8_t)(out[j >> 2] >> (8 * (j & 3)));
        uint2* suf = a.suf + (uint64_t)p * a.cap + my0;
#pragma unroll
        for (int j = kAffixItems - 1; j >= 0; --j) {
            if ((uint32_t)j >= cnt) continue;
            const BMap<4> c = map_of(j);
            bx = ((ends >> j) & 1u) ? c : bm_compose<4>(bx, c);
            suf[j] = pe_pack(bx);
        }
        __syncthreads();                         // every thread has read the block's totals
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
        const uint32_t b = wave_lower_bound(a, par, 0u, k, (pe_prefix(a, a.words[at]) + wave) << a.ibits);
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
    const uint64_t want = (max_entries + kAffixTile - 1) / kAffixTile;
    hipLaunchKernelGGL(k_pe_affix, dim3((uint32_t)(want < 1024 ? (want ? want : 1) : 1024), a.n_props), dim3(256), 0, s, a);
    return hipGetLastError();
}

hipError_t launch_parent_bounds(const ParentArgs& a, uint64_t max_own, hipStream_t s) {
    const uint64_t tiles = (max_own + kPeTile - 1) / kPeTile;
    hipLaunchKernelGGL(k_pe_bounds, dim3((uint32_t)(tiles ? tiles : 1)), dim3(kPeThreads), 0, s, a);
    return hipGetLastError();
}

}  // namespace ltl4c
