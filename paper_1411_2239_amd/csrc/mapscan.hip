// The segmented transition-map scan (Def. 6: the state of every instance
// after its cluster, composed as maps so that a cluster may spread over any
// number of lanes and tiles), in three steps without look-back:
//   reduce  per tile of 4,096 or 8,192 sorted words: every thread composes the
//           maps of its 16 or 32 consecutive words (a head restarts from q0),
//           the block scans the threads in order; the tile's map per property
//           and its head counts per level go to `agg`, every thread's
//           exclusive prefix within the tile to `trec`;
//   spine   exclusive prefixes of the tile records in tile order, in a few
//           launches of their own, or, where every block can read the records
//           before it (kOwnTiles), by the blocks of the down sweep themselves;
//   down    per tile: every thread starts from its prefix (tile prefix, then
//           its own), steps its states word by word and writes instance
//           verdicts, parents, numbering and nodes (and, on request, the
//           verdict timeline; a one-level tree's verdicts are counted here).
// Words are read as 16 or 32 consecutive 64-bit words per thread with 16-byte
// loads (no LDS staging).  The first reduce writes one descriptor byte per word
// (class, head and level-head flags); the down sweep and the launches of
// further property groups read those instead of the words.  No tile waits on
// another, so several tiles share a CU.
#include <type_traits>

#include "parent.h"

namespace ltl4c {

namespace {

constexpr uint32_t kAll = 0xFFFFFFFFu;

// Words of a tile record in memory: four counts and the maps, in whole 16-byte
// parts (the arrays are sized for kMsRec).
template <int PMAX, int MW>
constexpr uint32_t ms_rec() {
    static_assert(4 + PMAX * MW <= kMsRec, "record fits the arrays");
    return (4 + PMAX * MW + 3) / 4 * 4;
}

// PE kernels merge parent events in (parent.hip prepares what they read).
struct NoParent {};
template <bool PE>
using PeParam = std::conditional_t<PE, ParentArgs, NoParent>;

// Flags and classes of a thread's run of words: `cnt` valid words (a prefix of
// the run), head (a new instance), level-m heads (a new level-m node), classes
// packed 4 bits per word.
// SYM kernels (classes of at most 3 bits) keep a symbol instead: the class with
// the head flag in bit 3, so that "restart, then step" is one table entry.
struct Run {
    uint32_t cnt, m_head, m_lvl[kMaxLevels];
    uint64_t cls[2];
};

// (selects rather than indexing, so that runs never leave registers)
__device__ __forceinline__ uint32_t run_class(const Run& r, int j) {
    return (uint32_t)((j < 16 ? r.cls[0] : r.cls[1]) >> (4 * (j & 15))) & 15u;
}

__device__ __forceinline__ uint32_t valid_mask(uint32_t cnt) { return cnt >= 32 ? kAll : (1u << cnt) - 1u; }

template <int ITEMS, bool SYM>
__device__ __forceinline__ Run run_from_words(const ScanArgs& a, uint64_t my0, uint32_t n) {
    // Loads are unconditional, so that all of them are in flight together:
    // the word buffers have room for a whole run past the last valid word.
    // A thread without valid words reads the first run instead (in bounds).
    Run r{};
    r.cnt = my0 < n ? (uint32_t)min<uint64_t>(ITEMS, n - my0) : 0u;
    const uint64_t ld0 = r.cnt ? my0 : 0;
    const uint64_t prev0 = a.words[ld0 > 0 ? ld0 - 1 : 0];
    uint64_t wv[ITEMS];
    const uint4* p = reinterpret_cast<const uint4*>(a.words + ld0);
#pragma unroll
    for (int k = 0; k < ITEMS / 2; ++k) {
        const uint4 v = p[k];
        wv[2 * k] = ((uint64_t)v.y << 32) | v.x;
        wv[2 * k + 1] = ((uint64_t)v.w << 32) | v.z;
    }
    const uint64_t hlim = 1ull << a.cbits;
    uint64_t llim[kMaxLevels];
#pragma unroll
    for (int m = 1; m < kMaxLevels; ++m) llim[m] = (uint32_t)m < a.n_levels ? 1ull << a.prefix_shift[m] : ~0ull;
    uint64_t prev = prev0;
#pragma unroll
    for (int j = 0; j < ITEMS; ++j) {
        const uint64_t x = wv[j];
        const bool valid = (uint32_t)j < r.cnt;
        const bool first = my0 + j == 0;
        const uint64_t d = prev ^ x;
        prev = x;
        const uint32_t head = (uint32_t)(valid && (first || d >= hlim));
        r.m_head |= head << j;
#pragma unroll
        for (int m = 1; m < kMaxLevels; ++m)
            if ((uint32_t)m < a.n_levels) r.m_lvl[m] |= (uint32_t)(valid && (first || d >= llim[m])) << j;
        const uint64_t cj = (uint64_t)(((uint32_t)x & a.class_mask) | (SYM ? head << 3 : 0u)) << (4 * (j & 15));
        if (j < 16) r.cls[0] |= cj;
        else r.cls[1] |= cj;
    }
    return r;
}

template <bool SYM>
__device__ __forceinline__ uint32_t desc_byte(const Run& r, int j) {
    uint32_t b = run_class(r, j) & (SYM ? 7u : 15u);
    b |= ((r.m_head >> j) & 1u) << 4;
#pragma unroll
    for (int m = 1; m < kMaxLevels; ++m) b |= ((r.m_lvl[m] >> j) & 1u) << (4 + m);
    return b;
}

template <int ITEMS, bool SYM>
__device__ __forceinline__ void store_desc(const ScanArgs& a, uint64_t my0, const Run& r) {
    if (r.cnt == ITEMS) {
        uint32_t d[ITEMS / 4];
#pragma unroll
        for (int i = 0; i < ITEMS / 4; ++i) d[i] = 0;
#pragma unroll
        for (int j = 0; j < ITEMS; ++j) d[j >> 2] |= desc_byte<SYM>(r, j) << (8 * (j & 3));
        uint4* q = reinterpret_cast<uint4*>(a.desc + my0);
#pragma unroll
        for (int i = 0; i < ITEMS / 16; ++i) q[i] = make_uint4(d[4 * i], d[4 * i + 1], d[4 * i + 2], d[4 * i + 3]);
    } else {
        for (uint32_t j = 0; j < r.cnt; ++j) a.desc[my0 + j] = (uint8_t)desc_byte<SYM>(r, (int)j);
    }
}

// Four words' descriptor bytes (one dword) at once: the low nibbles packed
// into 16 bits (the classes), the high nibbles as a transposed 4 x 4 bit
// matrix, so that nibble f holds flag f (head, level-1..3 head) of the four
// words.
__device__ __forceinline__ uint32_t pack_nibbles(uint32_t x) {   // nibbles at bits 0, 8, 16, 24
    x = (x | (x >> 4)) & 0x00FF00FFu;
    return (x | (x >> 8)) & 0xFFFFu;
}
__device__ __forceinline__ uint32_t transpose4x4(uint32_t y) {   // bit 4k + f -> bit 4f + k
    uint32_t t = ((y >> 3) ^ y) & 0x0A0Au;
    y ^= t ^ (t << 3);
    t = ((y >> 6) ^ y) & 0x00CCu;
    return y ^ t ^ (t << 6);
}

template <int ITEMS, bool SYM>
__device__ __forceinline__ Run run_from_desc(const ScanArgs& a, uint64_t my0, uint32_t n) {
    // (the descriptor buffer has room for a whole run past the last word)
    Run r{};
    r.cnt = my0 < n ? (uint32_t)min<uint64_t>(ITEMS, n - my0) : 0u;
    const uint4* q = reinterpret_cast<const uint4*>(a.desc + (r.cnt ? my0 : 0));
#pragma unroll
    for (int i = 0; i < ITEMS / 16; ++i) {
        const uint4 v = q[i];
        uint32_t d[4] = {v.x, v.y, v.z, v.w};
        if (r.cnt < ITEMS) {
            // the bytes of words past the end read as 0
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                const uint32_t s0 = 16u * i + 4u * k;
                d[k] = s0 >= r.cnt ? 0u : s0 + 4u > r.cnt ? d[k] & ((1u << (8u * (r.cnt - s0))) - 1u) : d[k];
            }
        }
        uint64_t c = 0;
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            c |= (uint64_t)pack_nibbles(SYM ? (d[k] & 0x07070707u) | ((d[k] >> 1) & 0x08080808u) : d[k] & 0x0F0F0F0Fu) << (16 * k);
            const uint32_t f = transpose4x4(pack_nibbles((d[k] >> 4) & 0x0F0F0F0Fu));
            const int at = 16 * i + 4 * k;
            r.m_head |= (f & 15u) << at;
#pragma unroll
            for (int m = 1; m < kMaxLevels; ++m) r.m_lvl[m] |= ((f >> (4 * m)) & 15u) << at;
        }
        r.cls[i] = c;
    }
    return r;
}

// The composed map of a run per property: a head restarts the monitor at
// `start` (only the last head's start shows in the result).  FULL: every word of the run is valid (all threads but the trace's last).
template <int PMAX, int MW, int ITEMS, bool FULL>
__device__ __forceinline__ void run_maps_t(const Run& r, uint32_t P, const uint32_t (*s_cm)[16][MW],
                                           const uint32_t* start_q, BMap<MW>* f) {
    const uint32_t valid = FULL ? kAll : valid_mask(r.cnt);
#pragma unroll
    for (int p = 0; p < PMAX; ++p) {
        f[p] = bm_identity<MW>();
        if (p > 0 && p >= (int)P) continue;    // (a launch has at least one property)
        const BMap<MW> start = bm_const<MW>(start_q[p]);
#pragma unroll
        for (int j = 0; j < ITEMS; ++j) {
            const BMap<MW> cm = bm_load<MW>(s_cm[p][run_class(r, j)]);
            const BMap<MW> g = bm_compose<MW>(cm, ((r.m_head >> j) & 1u) ? start : f[p]);
            if (FULL || ((valid >> j) & 1u)) f[p] = g;
        }
    }
}
template <int PMAX, int MW, int ITEMS>
__device__ __forceinline__ void run_maps(const Run& r, uint32_t P, const uint32_t (*s_cm)[16][MW], const uint32_t* start_q,
                                         BMap<MW>* f) {
    // (four 16-state maps keep the one path: the second copy costs them registers)
    if (PMAX * MW <= 8 && r.cnt == ITEMS) run_maps_t<PMAX, MW, ITEMS, true>(r, P, s_cm, start_q, f);
    else run_maps_t<PMAX, MW, ITEMS, false>(r, P, s_cm, start_q, f);
}

// SYM: the map of every symbol (head flag << 3 | class: a head is the constant
// map of q0's successor), and of every pair of symbols, first one in the low
// nibble; one pair per thread of the block.
template <int MW>
__device__ __forceinline__ BMap<MW> sym_map(const uint32_t (*cm)[MW], uint32_t q0, uint32_t sym) {
    const BMap<MW> c = bm_load<MW>(cm[sym & 7u]);
    return (sym & 8u) ? bm_const<MW>(bm_at<MW>(c, q0)) : c;
}
template <int PMAX, int MW>
__device__ __forceinline__ void build_pairs(uint32_t P, const uint32_t (*s_cm)[16][MW], const uint32_t* s_q0,
                                            uint32_t (*s_pair)[256][MW]) {
    static_assert(kMsThreads == 256, "one pair per thread");
    const uint32_t i = threadIdx.x;
#pragma unroll
    for (int p = 0; p < PMAX; ++p) {
        if (p > 0 && p >= (int)P) continue;
        const BMap<MW> m = bm_compose<MW>(sym_map<MW>(s_cm[p], s_q0[p], i >> 4), sym_map<MW>(s_cm[p], s_q0[p], i & 15u));
#pragma unroll
        for (int k = 0; k < MW; ++k) s_pair[p][i][k] = m.d[k];
    }
}
// A full run's maps by pairs: half the compositions and half the table reads of
// run_maps, and no selects.  The reduce of many or large maps is bound by its
// vector instructions: 592M events, launches of four 16-state, four 16-state
// and eight 8-state maps 3400 + 2906 + 1280 us by single words, 2240 + 1723 +
// 740 us by pairs (with maps of 4 bits per state in the thread records, and the
// wave totals scanned over their few lanes only).  One or two 8-state maps are
// bound by memory and keep the single words (10M words 22.6 us, 4.4 TB/s).
template <int PMAX, int MW, int ITEMS>
__device__ __forceinline__ void run_maps_pairs(const Run& r, uint32_t P, const uint32_t (*s_pair)[256][MW], BMap<MW>* f) {
#pragma unroll
    for (int p = 0; p < PMAX; ++p) {
        f[p] = bm_identity<MW>();
        if (p > 0 && p >= (int)P) continue;
#pragma unroll
        for (int k = 0; k < ITEMS / 2; ++k) {
            const BMap<MW> m = bm_load<MW>(s_pair[p][(uint32_t)(r.cls[k >> 3] >> (8 * (k & 7))) & 255u]);
            f[p] = k ? bm_compose<MW>(m, f[p]) : m;
        }
    }
}

// Maps in the thread records: 4 bits per state.
template <int MW>
__device__ __forceinline__ void store_map4(uint32_t* row0, uint64_t row, const BMap<MW>& m) {
#pragma unroll
    for (int k = 0; k < MW / 2; ++k) row0[k * row] = pack_nibbles(m.d[2 * k]) | (pack_nibbles(m.d[2 * k + 1]) << 16);
}

// The bounds of a run's own events, and the events whose gap to the event
// before them (of the same instance) holds parent entries.
struct Bounds {
    uint32_t g[16];
    uint32_t gaps;
};
__device__ __forceinline__ Bounds load_bounds(const ParentArgs& q, uint64_t my0, const Run& r) {
    Bounds b;
    const uint64_t at = r.cnt ? my0 : 0;         // unconditional loads; the array is followed by others
    const uint4* src = reinterpret_cast<const uint4*>(q.bound + at);
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        const uint4 v = src[k];
        b.g[4 * k] = v.x;
        b.g[4 * k + 1] = v.y;
        b.g[4 * k + 2] = v.z;
        b.g[4 * k + 3] = v.w;
    }
    const uint32_t before = q.bound[at ? at - 1 : 0];
    b.gaps = 0;
#pragma unroll
    for (int j = 0; j < 16; ++j)
        b.gaps |= (uint32_t)((b.g[j] & kPeIndex) > ((j ? b.g[j - 1] : before) & kPeIndex)) << j;
    b.gaps &= valid_mask(r.cnt) & ~r.m_head;
    return b;
}
// property p's state before an instance's first own event with bound g (the
// load is unconditional, so that those of a run are in flight together)
__device__ __forceinline__ uint32_t pe_start(const ParentArgs& q, uint32_t p, uint32_t g, uint32_t q0) {
    const uint32_t i = g & kPeIndex;
    const uint32_t s = q.pre[p * q.cap + (i ? min<uint64_t>(i - 1u, q.cap - 1u) : 0u)];
    return (g & kPeNoneBefore) ? q0 : s;
}

// The class maps of the launch's properties, one table word per thread
// (PMAX * 16 * MW <= 256 = the block), plus q0 and the packed labels: read
// into registers first (the loads overlap the block's data loads), stored to
// LDS afterwards.
struct TableRegs {
    uint32_t cm, q0, lab0, lab1;
};

// prop_idx[p] for a thread-dependent p, by selects over kernel-argument
// scalars (indexing the argument array would be a vector load)
template <int PMAX>
__device__ __forceinline__ uint32_t prop_index(const ScanArgs& a, uint32_t p) {
    uint32_t r = a.prop_idx[0];
#pragma unroll
    for (int q = 1; q < PMAX; ++q)
        if (p == (uint32_t)q) r = a.prop_idx[q];
    return r;
}

template <int PMAX, int MW>
__device__ __forceinline__ TableRegs read_tables(const ScanArgs& a) {
    static_assert(PMAX * 16 * MW <= kMsThreads, "one table word per thread");
    TableRegs t{0, 0, 0, 0};
    const uint32_t P = a.n_props, i = threadIdx.x;
    if (i < P * 16 * MW) {
        const uint32_t p = i / (16 * MW), c = (i / MW) % 16, k = i % MW;
        t.cm = a.plan->prop[prop_index<PMAX>(a, p)].bmap[c][k];
    }
    if (i < P) {
        const PropDev& pd = a.plan->prop[prop_index<PMAX>(a, i)];
        t.q0 = pd.q0;
        t.lab0 = pd.blabel[0];
        t.lab1 = pd.blabel[1];
    }
    return t;
}

template <int PMAX, int MW>
__device__ __forceinline__ void store_tables(const ScanArgs& a, const TableRegs& t, uint32_t (*s_cm)[16][MW],
                                             uint32_t* s_q0, uint32_t (*s_lab)[2]) {
    const uint32_t P = a.n_props, i = threadIdx.x;
    if (i < P * 16 * MW) s_cm[i / (16 * MW)][(i / MW) % 16][i % MW] = t.cm;
    if (i < P) {
        s_q0[i] = t.q0;
        if (s_lab) {
            s_lab[i][0] = t.lab0;
            s_lab[i][1] = t.lab1;
        }
    }
}

// Block-wide ordered scan of one map per property and four counts per
// thread: on return `excl` and `cexcl` hold this thread's exclusive prefix
// within the block, `tot` / `ctot` (valid in every thread) the block's total.
// With PACK, the counts of a tile (below 2^16) travel two to a word, and the
// second word only when there are more than two levels.  The wave totals are
// scanned once, by wave 0 (row WAVES of s_wm / s_wc receives the block total),
// so no thread composes more than log2(WAVES) of them.
template <int PMAX, int MW, int THREADS, bool PACK = false>
__device__ __forceinline__ void block_scan(uint32_t P, const BMap<MW>* f, const uint32_t* cnt, BMap<MW>* excl,
                                           uint32_t* cexcl, BMap<MW>* tot, uint32_t* ctot,
                                           uint32_t (*s_wm)[THREADS / 64 + 1][MW], uint32_t (*s_wc)[THREADS / 64 + 1],
                                           uint32_t levels = 4) {
    constexpr int WAVES = THREADS / 64;
    constexpr int NC = PACK ? 2 : 4;
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    uint32_t c[4];
    if (PACK) {
        c[0] = cnt[0] | (cnt[1] << 16);
        c[1] = cnt[2] | (cnt[3] << 16);
    } else {
        c[0] = cnt[0], c[1] = cnt[1], c[2] = cnt[2], c[3] = cnt[3];
    }
#pragma unroll
    for (int p = 0; p < PMAX; ++p) {
        BMap<MW> v = f[p];
        if (p < (int)P) v = bm_wave_incl_scan<MW>(v);
        excl[p] = bm_wave_shr1<MW>(v);
        if (lane == 63)
#pragma unroll
            for (int k = 0; k < MW; ++k) s_wm[p][w][k] = v.d[k];
    }
#pragma unroll
    for (int k = 0; k < NC; ++k) {
        uint32_t x = c[k];
        if ((uint32_t)k * (4 / NC) < levels) x = wave_incl_sum(x);    // counts of absent levels stay zero
        cexcl[k] = x - c[k];
        if (lane == 63) s_wc[k][w] = x;
    }
    __syncthreads();
    if (w == 0) {
        // wave 0: exclusive scan of the wave totals, in place; the block total
        // goes to row WAVES
#pragma unroll
        for (int p = 0; p < PMAX; ++p) {
            if (p >= (int)P) continue;
            BMap<MW> v = lane < WAVES ? bm_load<MW>(s_wm[p][lane]) : bm_identity<MW>();
            v = bm_row_incl_scan<MW, WAVES>(v);
            const BMap<MW> ex = bm_wave_shr1<MW>(v);
            if (lane < WAVES) {
#pragma unroll
                for (int k = 0; k < MW; ++k) s_wm[p][lane][k] = ex.d[k];
            }
            if (lane == WAVES - 1)
#pragma unroll
                for (int k = 0; k < MW; ++k) s_wm[p][WAVES][k] = v.d[k];
        }
#pragma unroll
        for (int k = 0; k < NC; ++k) {
            const uint32_t c0 = lane < WAVES ? s_wc[k][lane] : 0u;
            const uint32_t x = row_incl_sum<WAVES>(c0);
            if (lane < WAVES) s_wc[k][lane] = x - c0;
            if (lane == WAVES - 1) s_wc[k][WAVES] = x;
        }
    }
    __syncthreads();
#pragma unroll
    for (int p = 0; p < PMAX; ++p) {
        if (p >= (int)P) {
            tot[p] = bm_identity<MW>();
            continue;
        }
        excl[p] = bm_compose<MW>(excl[p], bm_load<MW>(s_wm[p][w]));
        tot[p] = bm_load<MW>(s_wm[p][WAVES]);
    }
#pragma unroll
    for (int k = 0; k < NC; ++k) {
        cexcl[k] += s_wc[k][w];
        ctot[k] = s_wc[k][WAVES];
    }
    if (PACK) {
#pragma unroll
        for (int k = 1; k >= 0; --k) {
            cexcl[2 * k + 1] = cexcl[k] >> 16;
            cexcl[2 * k] = cexcl[k] & 0xFFFFu;
            ctot[2 * k + 1] = ctot[k] >> 16;
            ctot[2 * k] = ctot[k] & 0xFFFFu;
        }
    }
}

}  // namespace

template <int PMAX, int MW, int ITEMS, bool PE, bool SYM>
__global__ __launch_bounds__(kMsThreads) void k_ms_reduce(ScanArgs a, PeParam<PE> q) {
    constexpr uint32_t TILE = kMsThreads * ITEMS;
    __shared__ uint32_t s_pair[SYM ? PMAX : 1][SYM ? 256 : 1][MW];
    __shared__ uint32_t s_cm[PMAX][16][MW];
    __shared__ uint32_t s_q0[PMAX];
    __shared__ uint32_t s_wm[PMAX][kMsThreads / 64 + 1][MW];
    __shared__ uint32_t s_wc[4][kMsThreads / 64 + 1];
    const uint32_t n = a.n_dev ? *a.n_dev : a.n;
    const uint64_t base = (uint64_t)blockIdx.x * TILE;
    if (base >= n) return;                       // the whole block: no word of this tile
    const uint64_t my0 = base + (uint64_t)threadIdx.x * ITEMS;
    Run r = a.read_desc ? run_from_desc<ITEMS, SYM>(a, my0, n) : run_from_words<ITEMS, SYM>(a, my0, n);
    const TableRegs tr = read_tables<PMAX, MW>(a);
    store_tables<PMAX, MW>(a, tr, s_cm, s_q0, nullptr);
    if (!a.read_desc && a.desc && r.cnt) store_desc<ITEMS, SYM>(a, my0, r);
    __syncthreads();
    if constexpr (SYM) {
        build_pairs<PMAX, MW>(a.n_props, s_cm, s_q0, s_pair);
        __syncthreads();
    }
    BMap<MW> f[PMAX], excl[PMAX], tot[PMAX];
    if constexpr (PE) {
        const Bounds bd = load_bounds(q, my0, r);
        const uint32_t last = r.m_head ? 31u - (uint32_t)__clz(r.m_head) : 0u;
        const uint32_t from = r.m_head ? ~((2u << last) - 1u) : kAll;          // what follows the last head
        const uint32_t gl = q.bound[r.m_head ? my0 + last : 0];
        uint32_t start_q[PMAX];
#pragma unroll
        for (int p = 0; p < PMAX; ++p)
            start_q[p] = p < (int)a.n_props ? pe_start(q, prop_index<PMAX>(a, p), gl, s_q0[p]) : 0u;
        if ((bd.gaps & from) == 0) {
            run_maps<PMAX, MW, ITEMS>(r, a.n_props, s_cm, start_q, f);
        } else {
            // parent entries inside an instance: word by word, their range's map first
            const uint64_t* par = q.words + *q.n_own;
#pragma unroll
            for (int p = 0; p < PMAX; ++p) f[p] = r.m_head ? bm_const<MW>(start_q[p]) : bm_identity<MW>();
#pragma unroll 1
            for (uint32_t j = last; j < r.cnt; ++j) {
                const bool gap = (bd.gaps >> j) & 1u;
                const uint32_t hi = q.bound[my0 + j] & kPeIndex, lo = gap ? q.bound[my0 + j - 1] & kPeIndex : hi;
#pragma unroll
                for (int p = 0; p < PMAX; ++p) {
                    if (p >= (int)a.n_props) continue;
                    if (gap) f[p] = bm_compose<MW>(pe_range<MW>(q, s_cm[p], par, prop_index<PMAX>(a, p), lo, hi), f[p]);
                    f[p] = bm_compose<MW>(bm_load<MW>(s_cm[p][run_class(r, (int)j)]), f[p]);
                }
            }
        }
    } else if constexpr (SYM) {
        if (r.cnt == ITEMS) {
            run_maps_pairs<PMAX, MW, ITEMS>(r, a.n_props, s_pair, f);
        } else {
#pragma unroll
            for (int p = 0; p < PMAX; ++p) {
                f[p] = bm_identity<MW>();
                if (p > 0 && p >= (int)a.n_props) continue;
#pragma unroll 1
                for (uint32_t j = 0; j < r.cnt; ++j)
                    f[p] = bm_compose<MW>(sym_map<MW>(s_cm[p], s_q0[p], run_class(r, (int)j)), f[p]);
            }
        }
    } else {
        run_maps<PMAX, MW, ITEMS>(r, a.n_props, s_cm, s_q0, f);
    }
    uint32_t cnt[4], cexcl[4], ctot[4];
    cnt[0] = __popc(r.m_head);
#pragma unroll
    for (int m = 1; m < 4; ++m) cnt[m] = __popc(r.m_lvl[m]);
    block_scan<PMAX, MW, kMsThreads, true>(a.n_props, f, cnt, excl, cexcl, tot, ctot, s_wm, s_wc, a.n_levels);
    // this thread's exclusive prefix within the tile, for the down sweep
    // (rows of consecutive threads: coalesced)
    const uint64_t row = (uint64_t)a.tiles * kMsThreads, at = (uint64_t)blockIdx.x * kMsThreads + threadIdx.x;
    a.trec[at] = cexcl[0] | (cexcl[1] << 16);
    if (a.n_levels > 2) a.trec[row + at] = cexcl[2] | (cexcl[3] << 16);
#pragma unroll
    for (int p = 0; p < PMAX; ++p)
        if (p < (int)a.n_props) store_map4<MW>(a.trec + (2 + MW / 2 * p) * row + at, row, excl[p]);
    if (threadIdx.x < ms_rec<PMAX, MW>()) {
        const uint32_t k = threadIdx.x;
        uint32_t v = 0;
        if (k < 4) {
            v = ctot[k];
        } else {
            const uint32_t p = (k - 4) / MW, d = (k - 4) % MW;
#pragma unroll
            for (int q = 0; q < PMAX; ++q)
#pragma unroll
                for (int e = 0; e < MW; ++e)
                    if ((uint32_t)q == p && (uint32_t)e == d) v = tot[q].d[e];
        }
        a.agg[(uint64_t)blockIdx.x * ms_rec<PMAX, MW>() + k] = v;
    }
}

// Exclusive prefixes of the tile records (maps composed in tile order, head
// counts summed).  Records go in passes of kSpineThreads x (up to 4) records:
// each thread loads its chunk's records at once (16-byte loads, all in flight
// together), composes them, the block scans the thread totals, and the running
// prefix carries from pass to pass.  MODE 0: one block over all tiles (one
// pass up to 16M words).  Above a few passes the work is spread: MODE 1, block
// b composes the tiles of chunk b (a.spine_chunk tiles) into a chunk record;
// MODE 2, one block scans the chunk records; MODE 3, block b writes the tile
// prefixes of chunk b, starting from the chunk's prefix.
constexpr int kSpineThreads = kMsSpineThreads;

template <int NW>
__host__ __device__ constexpr int spine_chunk_items() { return NW <= 8 ? 4 : NW <= 12 ? 2 : 1; }

template <int PMAX, int MW, int ITEMS, int MODE>
__global__ __launch_bounds__(kSpineThreads) void k_ms_spine(ScanArgs a) {
    constexpr uint32_t TILE = kMsThreads * ITEMS;
    constexpr int NW = 4 + PMAX * MW;            // record words in use
    constexpr int kSpineChunk = spine_chunk_items<NW>();    // records held in registers
    constexpr int NQ = (NW + 3) / 4;             // 16-byte parts of a record
    __shared__ uint32_t s_wm[PMAX][kSpineThreads / 64 + 1][MW];
    __shared__ uint32_t s_wc[4][kSpineThreads / 64 + 1];
    __shared__ uint32_t s_carry[NW];
    const uint32_t n = a.n_dev ? *a.n_dev : a.n;
    const uint32_t tiles = (n + TILE - 1) / TILE;
    const uint32_t P = a.n_props;
    const uint32_t nchunks = MODE == 0 ? 1u : (tiles + a.spine_chunk - 1) / a.spine_chunk;
    uint32_t r0 = 0, r1 = tiles;                 // the records this block scans
    const uint32_t* in = a.agg;
    uint32_t* out = a.prefix;
    if (MODE == 1 || MODE == 3) {
        r0 = blockIdx.x * a.spine_chunk;
        r1 = min(tiles, r0 + a.spine_chunk);
        if (r0 >= r1) return;
    } else if (MODE == 2) {
        r1 = nchunks;
        in = a.chunk_agg;
        out = a.chunk_pre;
    }
    if (threadIdx.x < NW) {
        uint32_t v = threadIdx.x < 4 ? 0u : bm_identity<MW>().d[(threadIdx.x - 4) % MW];
        if (MODE == 3) v = a.chunk_pre[(uint64_t)blockIdx.x * ms_rec<PMAX, MW>() + threadIdx.x];
        s_carry[threadIdx.x] = v;
    }
    __syncthreads();
    for (uint32_t pass0 = r0; pass0 < r1; pass0 += kSpineThreads * kSpineChunk) {
        const uint32_t t0 = pass0 + threadIdx.x * kSpineChunk;
        const uint32_t cnt = t0 < r1 ? min<uint32_t>(kSpineChunk, r1 - t0) : 0u;
        // unconditional loads of clamped records: all of them in flight together
        uint32_t rec[kSpineChunk][NQ * 4];
#pragma unroll
        for (int i = 0; i < kSpineChunk; ++i) {
            const uint32_t t = min(t0 + (uint32_t)i, r1 - 1u);
            const uint4* src = reinterpret_cast<const uint4*>(in + (uint64_t)t * ms_rec<PMAX, MW>());
#pragma unroll
            for (int q = 0; q < NQ; ++q) {
                const uint4 v = src[q];
                rec[i][4 * q] = v.x;
                rec[i][4 * q + 1] = v.y;
                rec[i][4 * q + 2] = v.z;
                rec[i][4 * q + 3] = v.w;
            }
        }
        BMap<MW> f[PMAX], excl[PMAX], tot[PMAX];
        uint32_t c[4] = {0, 0, 0, 0}, cexcl[4], ctot[4];
#pragma unroll
        for (int p = 0; p < PMAX; ++p) f[p] = bm_identity<MW>();
#pragma unroll
        for (int i = 0; i < kSpineChunk; ++i) {
            const bool inr = (uint32_t)i < cnt;
#pragma unroll
            for (int p = 0; p < PMAX; ++p)
                if (p < (int)P && inr) f[p] = bm_compose<MW>(bm_load<MW>(&rec[i][4 + MW * p]), f[p]);
#pragma unroll
            for (int k = 0; k < 4; ++k) c[k] += inr ? rec[i][k] : 0u;
        }
        block_scan<PMAX, MW, kSpineThreads>(P, f, c, excl, cexcl, tot, ctot, s_wm, s_wc);
        if (MODE != 1) {
            // this thread's prefix: the carry from earlier passes, then the block's
            BMap<MW> acc[PMAX];
            uint32_t cc[4];
#pragma unroll
            for (int k = 0; k < 4; ++k) cc[k] = s_carry[k] + cexcl[k];
#pragma unroll
            for (int p = 0; p < PMAX; ++p) acc[p] = bm_compose<MW>(excl[p], bm_load<MW>(&s_carry[4 + MW * p]));
#pragma unroll
            for (int i = 0; i < kSpineChunk; ++i) {
                if ((uint32_t)i >= cnt) continue;
                uint32_t* o = out + (uint64_t)(t0 + i) * ms_rec<PMAX, MW>();
#pragma unroll
                for (int k = 0; k < 4; ++k) {
                    o[k] = cc[k];
                    cc[k] += rec[i][k];
                }
#pragma unroll
                for (int p = 0; p < PMAX; ++p) {
                    if (p >= (int)P) continue;
#pragma unroll
                    for (int k = 0; k < MW; ++k) o[4 + MW * p + k] = acc[p].d[k];
                    acc[p] = bm_compose<MW>(bm_load<MW>(&rec[i][4 + MW * p]), acc[p]);
                }
            }
        }
        __syncthreads();                         // every thread has read the carry
        if (threadIdx.x == 0) {
#pragma unroll
            for (int k = 0; k < 4; ++k) s_carry[k] += ctot[k];
#pragma unroll
            for (int p = 0; p < PMAX; ++p) {
                const BMap<MW> nc = bm_compose<MW>(tot[p], bm_load<MW>(&s_carry[4 + MW * p]));
#pragma unroll
                for (int k = 0; k < MW; ++k) s_carry[4 + MW * p + k] = nc.d[k];
            }
        }
        __syncthreads();
    }
    // the chunk's record: its composition (the carry started at the identity)
    if (MODE == 1 && threadIdx.x < NW) a.chunk_agg[(uint64_t)blockIdx.x * ms_rec<PMAX, MW>() + threadIdx.x] = s_carry[threadIdx.x];
}

// Before a tile: its state per property (the tile maps before it composed, at
// state 0: the first of them begins with a head, so the composition is
// constant) and its head counts, from the records of all tiles before it.  Each
// thread composes a contiguous share, the waves scan theirs in lane order and
// leave their totals in s_wm / s_wc; the caller adds those up after a barrier.
template <int PMAX, int MW>
__device__ __forceinline__ void compose_before(const ScanArgs& a, uint32_t P, uint32_t (*s_wm)[kMsThreads / 64][MW],
                                               uint32_t (*s_wc)[kMsThreads / 64]) {
    constexpr int NW = 4 + PMAX * MW, NQ = (NW + 3) / 4, kBatch = spine_chunk_items<NW>();
    const uint32_t b = blockIdx.x, share = (b + kMsThreads - 1) / kMsThreads;
    const uint32_t t0 = min(b, threadIdx.x * share), t1 = min(b, t0 + share);
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    BMap<MW> f[PMAX];
    uint32_t c[4] = {0, 0, 0, 0};
#pragma unroll
    for (int p = 0; p < PMAX; ++p) f[p] = bm_identity<MW>();
    for (uint32_t t = t0; t < t1; t += kBatch) {
        uint32_t rec[kBatch][NQ * 4];
#pragma unroll
        for (int i = 0; i < kBatch; ++i) {      // unconditional loads of clamped records, all in flight together
            const uint4* src = reinterpret_cast<const uint4*>(a.agg + (uint64_t)min(t + (uint32_t)i, t1 - 1u) * ms_rec<PMAX, MW>());
#pragma unroll
            for (int q = 0; q < NQ; ++q) {
                const uint4 v = src[q];
                rec[i][4 * q] = v.x;
                rec[i][4 * q + 1] = v.y;
                rec[i][4 * q + 2] = v.z;
                rec[i][4 * q + 3] = v.w;
            }
        }
#pragma unroll
        for (int i = 0; i < kBatch; ++i) {
            const bool in = t + (uint32_t)i < t1;
#pragma unroll
            for (int p = 0; p < PMAX; ++p)
                if (p < (int)P && in) f[p] = bm_compose<MW>(bm_load<MW>(&rec[i][4 + MW * p]), f[p]);
#pragma unroll
            for (int k = 0; k < 4; ++k) c[k] += in ? rec[i][k] : 0u;
        }
    }
#pragma unroll
    for (int p = 0; p < PMAX; ++p) {
        if (p >= (int)P) continue;
        const BMap<MW> v = bm_wave_incl_scan<MW>(f[p]);
        if (lane == 63)
#pragma unroll
            for (int k = 0; k < MW; ++k) s_wm[p][w][k] = v.d[k];
    }
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        const uint32_t x = (uint32_t)k < a.n_levels ? wave_incl_sum(c[k]) : 0u;
        if (lane == 63) s_wc[k][w] = x;
    }
}

// TL: the instantiation that also walks the verdict timeline (its registers
// stay out of the plain sweep's occupancy)
// OWN: the instantiation whose blocks compose what comes before them (again,
// its registers cost the others blocks per CU: batch down sweeps 616 -> 668 us).
template <int PMAX, int MW, int ITEMS, bool TL, bool PE, bool SYM, bool OWN>
__global__ __launch_bounds__(kMsThreads) void k_ms_down(ScanArgs a, PeParam<PE> q) {
    __shared__ uint8_t s_next[SYM ? PMAX : 1][SYM ? 256 : 1];    // successor of state (low nibble) by symbol (high)
    constexpr uint32_t TILE = kMsThreads * ITEMS;
    constexpr bool kParents = PMAX <= 4;         // LDS room to stage parent ids
    constexpr uint32_t kIvStride = TILE + 1;
    __shared__ uint32_t s_cm[PMAX][16][MW];
    __shared__ uint32_t s_q0[PMAX], s_lab[PMAX][2];
    __shared__ uint32_t s_red[2][kMsThreads / 64];
    // staging: verdict bytes [P][tile + 1], then 16-bit parent offsets [tile + 1];
    // with keys asked for, the last word of every instance too (dynamic, so
    // that calls without keys keep the blocks per CU)
    extern __shared__ uint16_t s_pos[];
    __shared__ uint32_t s_stage[(PMAX * kIvStride + 3) / 4 + (kParents ? (kIvStride + 1) / 2 : 0)];
    const uint32_t n = a.n_dev ? *a.n_dev : a.n;
    const uint64_t base = (uint64_t)blockIdx.x * TILE;
    if (base >= n) return;
    const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
    const uint32_t P = a.n_props, L = a.n_levels;
    const bool structure = kParents && a.structure != 0;
    const uint64_t my0 = base + (uint64_t)tid * ITEMS;
    // every load first, so that they are all in flight together: tables,
    // this thread's prefix within the tile (reduce), the tile's (spine), the
    // descriptors and the one after them
    const uint64_t row = (uint64_t)a.tiles * kMsThreads, at = (uint64_t)blockIdx.x * kMsThreads + tid;
    const uint32_t c01 = a.trec[at], c23 = a.n_levels > 2 ? a.trec[row + at] : 0u;
    uint32_t tex[PMAX][MW / 2];
#pragma unroll
    for (int p = 0; p < PMAX; ++p)
#pragma unroll
        for (int k = 0; k < MW / 2; ++k) tex[p][k] = a.trec[(2 + MW / 2 * p + k) * row + at];
    // Few instances end in the tile (about as many as begin): their states are
    // found one by one afterwards, each from the last head of its thread's run,
    // instead of stepping every word of every thread.  592M events of 16
    // properties, some 256 words per instance: down sweeps of 893 + 884 + 1683 us
    // stepping every word, 616 + 607 + 837 us so.
    constexpr bool kList = !TL && !PE;
    constexpr uint32_t kSparse = 256;
    __shared__ uint16_t s_end[kList ? kSparse + 1 : 1];
    __shared__ uint32_t s_hd[kList ? kMsThreads : 1], s_cur[kList ? kMsThreads : 1];
    __shared__ uint64_t s_cls[kList ? ITEMS / 16 : 1][kList ? kMsThreads : 1];
    const bool sparse = kList && a.agg[(uint64_t)blockIdx.x * ms_rec<PMAX, MW>()] < kSparse;
    // what comes before the tile: from the spine, or composed here
    __shared__ uint32_t s_wm[OWN ? PMAX : 1][kMsThreads / 64][MW];
    __shared__ uint32_t s_wc[OWN ? 4 : 1][kMsThreads / 64];
    uint32_t tcnt[4] = {0, 0, 0, 0}, pmap[PMAX];
    if constexpr (!OWN) {
        const uint32_t* pre = a.prefix + (uint64_t)blockIdx.x * ms_rec<PMAX, MW>();
#pragma unroll
        for (int k = 0; k < 4; ++k) tcnt[k] = pre[k];
#pragma unroll
        for (int p = 0; p < PMAX; ++p) pmap[p] = pre[4 + MW * p];     // (state 0's image: the map is constant)
    }
    const uint32_t next_desc = a.desc[(my0 < n ? my0 : 0) + ITEMS];
    const Run r = run_from_desc<ITEMS, SYM>(a, my0, n);
    const TableRegs tr = read_tables<PMAX, MW>(a);
    // an instance ends where the next word is absent or a head
    const bool next_head = my0 + ITEMS < n ? ((next_desc >> 4) & 1u) != 0 : true;
    store_tables<PMAX, MW>(a, tr, s_cm, s_q0, s_lab);
    if constexpr (OWN) compose_before<PMAX, MW>(a, P, s_wm, s_wc);
    __syncthreads();
    if constexpr (OWN) {
#pragma unroll
        for (int p = 0; p < PMAX; ++p) {
            pmap[p] = 0;
            if (p >= (int)P) continue;
#pragma unroll
            for (int i = 0; i < kMsThreads / 64; ++i) pmap[p] = bm_at<MW>(bm_load<MW>(s_wm[p][i]), pmap[p]);
        }
#pragma unroll
        for (int k = 0; k < 4; ++k)
#pragma unroll
            for (int i = 0; i < kMsThreads / 64; ++i) tcnt[k] += s_wc[k][i];
    }
    if constexpr (SYM) {
#pragma unroll
        for (int p = 0; p < PMAX; ++p)
            if (p < (int)P) s_next[p][tid] = (uint8_t)bm_at<MW>(sym_map<MW>(s_cm[p], s_q0[p], (uint32_t)tid >> 4), (uint32_t)tid & (4u * MW - 1u));
        __syncthreads();
    }
    uint32_t cexcl[4] = {c01 & 0xFFFFu, c01 >> 16, c23 & 0xFFFFu, c23 >> 16};
    uint32_t cur[PMAX];
#pragma unroll
    for (int p = 0; p < PMAX; ++p) {
        cur[p] = 0;
        // (both halves shifted before the choice, kept apart: no indexed register array)
        const uint32_t s0 = pmap[p] & 15u;
        uint32_t t0 = tex[p][0] >> (4u * (s0 & 7u)), t1 = tex[p][MW / 2 - 1] >> (4u * (s0 & 7u));
        asm("" : "+v"(t0), "+v"(t1));
        if (p < (int)P) cur[p] = (MW > 2 && s0 >= 8u ? t1 : t0) & 15u;
    }
    const bool timeline = TL && (a.inst_conc || a.event_pack);
    uint32_t cur0[PMAX];
#pragma unroll
    for (int p = 0; p < PMAX; ++p) cur0[p] = cur[p];
    const uint32_t valid = valid_mask(r.cnt);
    const uint32_t m_end = r.cnt ? valid & ((r.m_head >> 1) | ((next_head ? 1u : 0u) << (r.cnt - 1u))) : 0u;
    uint8_t* s_iv = reinterpret_cast<uint8_t*>(s_stage);
    uint16_t* s_par = reinterpret_cast<uint16_t*>(s_stage + (PMAX * kIvStride + 3) / 4);
    const uint32_t id_base = tcnt[0];
    const uint32_t m_par = L >= 4 ? r.m_lvl[3] : L == 3 ? r.m_lvl[2] : r.m_lvl[1];
    // parents are level-(L-1) nodes: id = the tile's count before it + a local offset
    const uint32_t lpar = L >= 4 ? 3u : L == 3 ? 2u : 1u;
    const uint32_t par_tile = tcnt[lpar] - 1u, par_local = cexcl[lpar];
    uint32_t my_lo = 0xFFFFFFFFu, my_hi = 0u, err = 0;
    if (sparse) {
        uint32_t packed = 0;
#pragma unroll
        for (int p = 0; p < PMAX; ++p) packed |= cur[p] << (4 * p);
        s_cur[tid] = packed;
#pragma unroll
        for (int h = 0; h < ITEMS / 16; ++h) s_cls[kList ? h : 0][kList ? tid : 0] = r.cls[h];
        s_hd[tid] = r.m_head;
    }
    // First every word's state, without branches (the class maps' LDS reads
    // do not wait on the instance bookkeeping): 4 bits per word and property.
    uint64_t st[PMAX][ITEMS / 16];
#pragma unroll
    for (int p = 0; p < PMAX; ++p)
#pragma unroll
        for (int h = 0; h < ITEMS / 16; ++h) st[p][h] = 0;
    if constexpr (PE) {
        const Bounds bd = load_bounds(q, my0, r);
        if (bd.gaps != 0) {
            // parent entries inside an instance: word by word
            const uint64_t* par = q.words + *q.n_own;
#pragma unroll 1
            for (uint32_t j = 0; j < r.cnt; ++j) {
                const bool hd = (r.m_head >> j) & 1u, gap = (bd.gaps >> j) & 1u;
                const uint32_t g = q.bound[my0 + j], hi = g & kPeIndex, lo = gap ? q.bound[my0 + j - 1] & kPeIndex : hi;
#pragma unroll
                for (int p = 0; p < PMAX; ++p) {
                    if (p >= (int)P) continue;
                    const uint32_t pi = prop_index<PMAX>(a, p);
                    if (hd) cur[p] = pe_start(q, pi, g, s_q0[p]);
                    else if (gap) cur[p] = bm_at<MW>(pe_range<MW>(q, s_cm[p], par, pi, lo, hi), cur[p]);
                    cur[p] = bm_at<MW>(bm_load<MW>(s_cm[p][run_class(r, (int)j)]), cur[p]);
                    st[p][0] |= (uint64_t)cur[p] << (4 * j);
                }
            }
        } else {
#pragma clang loop unroll(full)
            for (int p = 0; p < PMAX; ++p) {
                if (p >= (int)P) continue;
                const uint32_t pi = prop_index<PMAX>(a, p);
                uint32_t start[16];
#pragma clang loop unroll(full)
                for (int j = 0; j < 16; ++j) start[j] = pe_start(q, pi, bd.g[j], s_q0[p]);
#pragma clang loop unroll(full)
                for (int j = 0; j < 16; ++j) {
                    cur[p] = bm_at<MW>(bm_load<MW>(s_cm[p][run_class(r, j)]), ((r.m_head >> j) & 1u) ? start[j] : cur[p]);
                    st[p][0] |= (uint64_t)cur[p] << (4 * j);
                }
            }
        }
    }
    if (!PE && !sparse)
#pragma clang loop unroll(full)
    for (int j = 0; j < ITEMS; ++j) {
        const uint32_t c = run_class(r, j);
        const bool hd = (r.m_head >> j) & 1u;
#pragma clang loop unroll(full)
        for (int p = 0; p < PMAX; ++p) {    // (a launch has at least one property)
            if (p > 0 && p >= (int)P) continue;
            if constexpr (SYM) cur[p] = s_next[p][(c << 4) | cur[p]];
            else cur[p] = bm_at<MW>(bm_load<MW>(s_cm[p][c]), hd ? s_q0[p] : cur[p]);
            st[p][j >> 4] |= (uint64_t)cur[p] << (4 * (j & 15));
        }
    }
    // Then the instances ending in the run, one loop step per end.
    for (uint32_t rest = m_end; rest != 0u; rest &= rest - 1u) {
        const uint32_t j = (uint32_t)__ffs(rest) - 1u;
        const uint32_t upto = j == 31u ? kAll : (2u << j) - 1u;
        const uint32_t slot = cexcl[0] + __popc(r.m_head & upto);     // 1-based, within the tile
        const uint64_t id = (uint64_t)id_base + slot - 1u;
        if (id < a.inst_limit) {
            const uint32_t sh = 4u * (j & 15u);
            if (sparse) s_end[slot] = (uint16_t)(tid * ITEMS + j);
            else
#pragma clang loop unroll(full)
            for (int p = 0; p < PMAX; ++p) {
                if (p > 0 && p >= (int)P) continue;
                // both halves shifted before the choice, and kept apart so that
                // the choice is not turned into an indexed register array
                uint32_t s0 = (uint32_t)(st[p][0] >> sh) & 15u, s1 = (uint32_t)(st[p][ITEMS / 16 - 1] >> sh) & 15u;
                asm("" : "+v"(s0), "+v"(s1));
                uint32_t qe = ITEMS > 16 && j >= 16u ? s1 : s0;
                if constexpr (PE) {
                    // the parent's entries after the instance's last own event
                    const uint32_t g = q.bound[my0 + j];
                    if (!(g & kPeNoneAfter)) {
                        const uint2 m = q.suf[prop_index<PMAX>(a, p) * q.cap + (g & kPeIndex)];
                        qe = ((qe & 8u ? m.y : m.x) >> (4 * (qe & 7u))) & 15u;
                    }
                }
                s_iv[p * kIvStride + slot] = a.emit_state ? qe : (s_lab[p][qe >> 3] >> (4 * (qe & 7u))) & 15u;
            }
            if (kParents && L >= 2) s_par[slot] = (uint16_t)(par_local + __popc(m_par & upto));
            my_lo = min(my_lo, (uint32_t)id);
            my_hi = max(my_hi, (uint32_t)id + 1u);
            if (structure && a.inst_keys) s_pos[slot] = (uint16_t)(tid * ITEMS + j);
        } else {
            err |= kErrCapacity;
        }
    }
    // On request, the verdict timeline, from the states kept above.  The
    // verdicts after an event go to the event's trace index, which rides in the
    // word between class and key: all properties of the launch packed 4 bits
    // each (16 bits for up to four), spread over the properties' rows by
    // k_event_unpack.  Conclusive verdicts are final (Def. 5), so the monitor
    // enters a conclusive state at most once per instance: the word where it
    // does writes its 1-based sorted position (the head's position when q0
    // itself is conclusive), the word ending an instance that never got there
    // writes kNever; k_inst_conclusive turns positions into prefix lengths.
    // Those words are found as bit masks and visited one by one; the rest is
    // straight code.  10M events, three properties: 399 us with a byte store per
    // property and a walk word by word, 148 us with packed stores, 133 us this
    // way.  What bounds it is the 10M stores at random places (about 100 us;
    // stores that bypass the L2 took 336 us in all).
    if (timeline) {
        uint32_t evi[ITEMS];
#pragma unroll
        for (int k = 0; k < ITEMS; ++k) evi[k] = 0;
        if (a.event_pack) {
            const uint4* wp = reinterpret_cast<const uint4*>(a.words + (r.cnt ? my0 : 0));
#pragma unroll
            for (int k = 0; k < ITEMS / 2; ++k) {
                const uint4 v = wp[k];
                evi[2 * k] = (uint32_t)((((uint64_t)v.y << 32) | v.x) >> a.index_shift) & a.index_mask;
                evi[2 * k + 1] = (uint32_t)((((uint64_t)v.w << 32) | v.z) >> a.index_shift) & a.index_mask;
            }
        }
        uint32_t lab[PMAX][2], conc[PMAX];
        auto label = [&](int p, uint32_t q) {
            return ((MW == 2 || q < 8u ? lab[p][0] : lab[p][1]) >> (4u * (MW == 2 ? q : q & 7u))) & 15u;
        };
        auto conclusive = [](uint32_t l) { return (0x21u >> l) & 1u; };       // F (0) or T (5)
#pragma unroll
        for (int p = 0; p < PMAX; ++p) {
            lab[p][0] = s_lab[p][0];
            lab[p][1] = s_lab[p][1];
            conc[p] = 0;
        }
#pragma clang loop unroll(full)
        for (int j = 0; j < ITEMS; ++j) {
            uint32_t pack = 0;
#pragma clang loop unroll(full)
            for (int p = 0; p < PMAX; ++p) {
                if (p > 0 && p >= (int)P) continue;
                const uint32_t l = label(p, (uint32_t)(st[p][j >> 4] >> (4 * (j & 15))) & 15u);
                pack |= l << (4 * p);
                conc[p] |= conclusive(l) << j;
            }
            if (a.event_pack && (uint32_t)j < r.cnt) {
                if (PMAX <= 4) reinterpret_cast<uint16_t*>(a.event_pack)[evi[j]] = (uint16_t)pack;
                else a.event_pack[evi[j]] = pack;
            }
        }
        if (a.inst_conc) {
            auto inst_of = [&](uint32_t j) {
                return (uint64_t)id_base + cexcl[0] + __popc(r.m_head & (j == 31u ? kAll : (2u << j) - 1u)) - 1u;
            };
            if (structure)
                for (uint32_t rest = r.m_head; rest != 0u; rest &= rest - 1u) {
                    const uint32_t j = (uint32_t)__ffs(rest) - 1u;
                    const uint64_t id = inst_of(j);
                    if (id < a.inst_limit) a.inst_start[id] = (uint32_t)(my0 + j);
                }
#pragma clang loop unroll(full)
            for (int p = 0; p < PMAX; ++p) {
                if (p > 0 && p >= (int)P) continue;
                // conclusive before each word: q0's verdict at a head, else the previous word's
                const uint32_t at_head = conclusive(label(p, s_q0[p])) ? r.m_head : 0u;
                const uint32_t before = (((conc[p] << 1) | conclusive(label(p, cur0[p]))) & ~r.m_head) | at_head;
                const uint32_t enters = conc[p] & ~before & valid, never = m_end & ~conc[p];
                for (uint32_t rest = at_head | enters | never; rest != 0u; rest &= rest - 1u) {
                    const uint32_t j = (uint32_t)__ffs(rest) - 1u;
                    const uint64_t id = inst_of(j);
                    if (id >= a.inst_limit) continue;
                    uint32_t* out = a.inst_conc + a.prop_idx[p] * a.inst_stride + id;
                    const uint32_t pos = (uint32_t)(my0 + j);
                    if ((at_head >> j) & 1u) *out = pos;
                    else if ((enters >> j) & 1u) *out = pos + 1u;
                    if ((never >> j) & 1u) *out = kNever;
                }
            }
        }
    }
    // nodes of levels 1.. open at their first word (a level-m head is also a
    // level-(m+1) head); few words do: a loop over them
    if (structure && L >= 2) {
        for (uint32_t rest = m_par; rest != 0u; rest &= rest - 1u) {
            const int j = __ffs(rest) - 1;
            const uint32_t upto = j == 31 ? kAll : (2u << j) - 1u;
#pragma unroll
            for (int m = kMaxLevels - 1; m >= 1; --m) {
                if (m >= (int)L || !((r.m_lvl[m] >> j) & 1u)) continue;
                const uint64_t id = (uint64_t)tcnt[m] + cexcl[m] + __popc(r.m_lvl[m] & upto) - 1u;
                const int mc = m < 3 ? m + 1 : 3;
                const uint32_t child = m == (int)L - 1 ? tcnt[0] + cexcl[0] + __popc(r.m_head & upto) - 1u
                                                       : tcnt[mc] + cexcl[mc] + __popc(r.m_lvl[mc] & upto) - 1u;
                if (id < a.node_limit[m]) {
                    a.node_start[m][id] = child;
                    if (a.node_keys[m]) a.node_keys[m][id] = a.words[my0 + j] >> a.prefix_shift[m];
                    uint32_t* cn = a.node_counts[m];
                    if (cn)
                        for (uint32_t p = 0; p < a.n_props_all; ++p) {
                            uint2* q = reinterpret_cast<uint2*>(cn + (p * a.node_stride[m] + id) * 6);
                            q[0] = make_uint2(0u, 0u);
                            q[1] = make_uint2(0u, 0u);
                            q[2] = make_uint2(0u, 0u);
                        }
                } else {
                    err |= kErrCapacity;
                }
            }
        }
    }
    if (err) atomicOr(a.err, err);
    // the instances ending in this tile have consecutive ids: write their
    // verdicts (and parents) contiguously from LDS
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1) {
        my_lo = min(my_lo, (uint32_t)__shfl_xor(my_lo, off, 64));
        my_hi = max(my_hi, (uint32_t)__shfl_xor(my_hi, off, 64));
    }
    if (lane == 0) {
        s_red[0][w] = my_lo;
        s_red[1][w] = my_hi;
    }
    __syncthreads();
    uint32_t lo = s_red[0][0], hi = s_red[1][0];
    for (int i = 1; i < kMsThreads / 64; ++i) {
        lo = min(lo, s_red[0][i]);
        hi = max(hi, s_red[1][i]);
    }
    uint32_t bins[OWN ? PMAX : 1];              // this thread's verdicts, six counts of 5 bits (at most 16 words)
#pragma unroll
    for (int p = 0; p < (OWN ? PMAX : 1); ++p) bins[p] = 0;
    if (lo < hi) {
        const uint32_t cnt_iv = hi - lo, slot0 = lo + 1u - id_base;
        if (sparse) {
            for (uint32_t i = tid; i < cnt_iv; i += kMsThreads) {
                const uint32_t pos = s_end[slot0 + i], t = pos / ITEMS, j = pos % ITEMS;
                const uint32_t heads = s_hd[t] & (j == 31u ? kAll : (2u << j) - 1u);
                const uint32_t from = heads ? 31u - (uint32_t)__clz(heads) : 0u;
                uint32_t q[PMAX];
#pragma unroll
                for (int p = 0; p < PMAX; ++p) q[p] = heads ? (p < (int)P ? s_q0[p] : 0u) : (s_cur[t] >> (4 * p)) & 15u;
                uint64_t sym = s_cls[from >> 4][t] >> (4 * (from & 15u));
                for (uint32_t k = from; k <= j; ++k, sym >>= 4) {
                    if (ITEMS > 16 && k == 16u) sym = s_cls[ITEMS / 16 - 1][t];
                    const uint32_t c = (uint32_t)sym & 15u;
#pragma clang loop unroll(full)
                    for (int p = 0; p < PMAX; ++p) {
                        if (p > 0 && p >= (int)P) continue;
                        if constexpr (SYM) q[p] = s_next[p][(c << 4) | q[p]];
                        else q[p] = bm_at<MW>(bm_load<MW>(s_cm[p][c]), q[p]);
                    }
                }
#pragma clang loop unroll(full)
                for (int p = 0; p < PMAX; ++p) {
                    if (p > 0 && p >= (int)P) continue;
                    const uint32_t v = a.emit_state ? q[p] : (s_lab[p][q[p] >> 3] >> (4 * (q[p] & 7u))) & 15u;
                    a.inst_verdict[a.prop_idx[p] * a.inst_stride + lo + i] = (uint8_t)v;
                    if constexpr (OWN) bins[p] += 1u << (5u * v);
                }
            }
        } else {
#pragma clang loop unroll(full)
            for (int p = 0; p < PMAX; ++p) {
                if (p > 0 && p >= (int)P) continue;
                for (uint32_t i = tid; i < cnt_iv; i += kMsThreads) {
                    const uint32_t v = s_iv[p * kIvStride + slot0 + i];
                    a.inst_verdict[a.prop_idx[p] * a.inst_stride + lo + i] = (uint8_t)v;
                    if constexpr (OWN) bins[p] += 1u << (5u * v);
                }
            }
        }
        if (structure && a.inst_parent && L >= 2)
            for (uint32_t i = tid; i < cnt_iv; i += kMsThreads) a.inst_parent[lo + i] = par_tile + s_par[slot0 + i];
        // the keys in one stream as well: 10M events with 2.9M instances and
        // parent events took 112 us with each key written where its instance
        // ends, 60 us so
        if (structure && a.inst_keys)
            for (uint32_t i = tid; i < cnt_iv; i += kMsThreads) a.inst_keys[lo + i] = a.words[base + s_pos[slot0 + i]] >> a.cbits;
    }
    // One-level trees: the tile's verdicts are counted here, into one of the
    // copies of the root's bins, instead of by a launch of their own (7.6 us for
    // 1,000 instances; 16,384 socket events 41.3 -> 34.7 us a pass,
    // 8.4M 169.1 -> 162.7 us).
    if constexpr (OWN) if (a.root_bins && lo < hi) {
        __shared__ uint32_t s_bins[PMAX][3][kMsThreads / 64];
#pragma unroll
        for (int p = 0; p < PMAX; ++p) {
            if (p > 0 && p >= (int)P) continue;
#pragma unroll
            for (int h = 0; h < 3; ++h) {       // two bins a word: at most 16 x 64 each
                const uint32_t x = wave_incl_sum(((bins[p] >> (10 * h)) & 31u) | (((bins[p] >> (10 * h + 5)) & 31u) << 16));
                if (lane == 63) s_bins[p][h][w] = x;
            }
        }
        __syncthreads();
        if (tid < (int)P * 6) {
            const uint32_t p = (uint32_t)tid / 6u, b = (uint32_t)tid % 6u;
            uint32_t x = 0;
#pragma unroll
            for (int i = 0; i < kMsThreads / 64; ++i) x += s_bins[p][b >> 1][i];
            x = (x >> (16 * (b & 1u))) & 0xFFFFu;
            if (x) atomicAdd(a.root_bins + ((blockIdx.x % kRootCopies) * kMaxProps + prop_index<PMAX>(a, p)) * 6u + b, x);
        }
    }
    // the thread holding the last word publishes the totals
    if (structure && r.cnt && my0 + r.cnt == n) {
        const uint32_t cnt[4] = {(uint32_t)__popc(r.m_head), (uint32_t)__popc(r.m_lvl[1]), (uint32_t)__popc(r.m_lvl[2]),
                                 (uint32_t)__popc(r.m_lvl[3])};
#pragma unroll
        for (int m = 0; m < kMaxLevels; ++m) {
            if (m >= (int)L) break;
            const uint32_t tot_m = tcnt[m] + cexcl[m] + cnt[m];
            a.sizes[m] = tot_m;
            a.sizes32[m] = tot_m;
        }
    }
}

// The packed verdicts of one launch's properties (4 bits each, by trace index)
// as one byte per event in every property's row; 15 is an event of no
// instance.  8 events per thread: 32 bytes in, 8 bytes out per property, rows
// that start at any byte.  10M events, three properties: 10.9 us (50 MB, 4.6 TB/s).
template <int WORDS>
__global__ __launch_bounds__(256) void k_event_unpack(ScanArgs a) {
    const uint64_t lanes = (uint64_t)gridDim.x * blockDim.x, n8 = a.n_events / 8;
    for (uint64_t t = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; t <= n8; t += lanes) {
        const uint32_t cnt = t < n8 ? 8u : (uint32_t)(a.n_events - 8 * n8);
        // (room for 8 past the end)
        const uint4* src = reinterpret_cast<const uint4*>(a.event_pack) + WORDS * t;
        uint32_t v[8];
        const uint4 lo = src[0];
        if constexpr (WORDS == 1) {
            const uint32_t d[4] = {lo.x, lo.y, lo.z, lo.w};
#pragma unroll
            for (int k = 0; k < 8; ++k) v[k] = (d[k >> 1] >> (16 * (k & 1))) & 0xFFFFu;
        } else {
            const uint4 hi = src[1];
            const uint32_t d[8] = {lo.x, lo.y, lo.z, lo.w, hi.x, hi.y, hi.z, hi.w};
#pragma unroll
            for (int k = 0; k < 8; ++k) v[k] = d[k];
        }
        for (uint32_t p = 0; p < a.n_props; ++p) {
            uint32_t o[2] = {0, 0};
#pragma unroll
            for (int k = 0; k < 8; ++k) {
                const uint32_t x = (v[k] >> (4 * p)) & 15u;
                o[k >> 2] |= (x == 15u ? 255u : x) << (8 * (k & 3));
            }
            uint8_t* dst = a.event_verdict + a.prop_idx[p] * a.n_events + 8 * t;
            if (cnt == 8u) __builtin_memcpy(dst, o, 8);
            else
                for (uint32_t k = 0; k < cnt; ++k) dst[k] = (uint8_t)(o[k >> 2] >> (8 * (k & 3)));
        }
    }
}

hipError_t launch_event_unpack(const ScanArgs& a, hipStream_t s) {
    const uint64_t want = (a.n_events / 8 + 256) / 256;
    const dim3 grid((uint32_t)(want < 4096 ? want : 4096));
    if (a.n_props <= 4) hipLaunchKernelGGL(k_event_unpack<1>, grid, dim3(256), 0, s, a);
    else hipLaunchKernelGGL(k_event_unpack<2>, grid, dim3(256), 0, s, a);
    return hipGetLastError();
}

template <int PMAX, int MW, int ITEMS, bool TL, bool PE, bool SYM>
static void launch_down(const ScanArgs& d, const PeParam<PE>& q, bool own, dim3 grid, uint32_t lds, hipStream_t s) {
    if constexpr (ITEMS == 16) {
        if (own) {
            hipLaunchKernelGGL((k_ms_down<PMAX, MW, ITEMS, TL, PE, SYM, true>), grid, dim3(kMsThreads), lds, s, d, q);
            return;
        }
    }
    hipLaunchKernelGGL((k_ms_down<PMAX, MW, ITEMS, TL, PE, SYM, false>), grid, dim3(kMsThreads), lds, s, d, q);
}

template <int PMAX, int MW, int ITEMS, bool PE, bool SYM>
static void launch_ms_t(const ScanArgs& a, const PeParam<PE>& q, hipStream_t s) {
    const uint32_t tiles = (uint32_t)((a.n + kMsThreads * ITEMS - 1) / (kMsThreads * ITEMS));
    const dim3 grid(tiles ? tiles : 1);
    ScanArgs r = a;
    r.tiles = tiles;
    hipLaunchKernelGGL((k_ms_reduce<PMAX, MW, ITEMS, PE, SYM>), grid, dim3(kMsThreads), 0, s, r, q);
    // one spine block takes kSpineThreads x chunk records per pass; beyond two
    // passes the chunks are spread over blocks
    constexpr uint32_t kPass = (uint32_t)kSpineThreads * spine_chunk_items<4 + PMAX * MW>();
    const bool own = ITEMS == 16 && tiles <= kOwnTiles;
    if (own) {
    } else if (tiles <= 2 * kPass || !a.chunk_agg || !a.chunk_pre) {
        hipLaunchKernelGGL((k_ms_spine<PMAX, MW, ITEMS, 0>), dim3(1), dim3(kSpineThreads), 0, s, r);
    } else {
        r.spine_chunk = kPass;
        const uint32_t nchunks = (tiles + kPass - 1) / kPass;
        hipLaunchKernelGGL((k_ms_spine<PMAX, MW, ITEMS, 1>), dim3(nchunks), dim3(kSpineThreads), 0, s, r);
        hipLaunchKernelGGL((k_ms_spine<PMAX, MW, ITEMS, 2>), dim3(1), dim3(kSpineThreads), 0, s, r);
        hipLaunchKernelGGL((k_ms_spine<PMAX, MW, ITEMS, 3>), dim3(nchunks), dim3(kSpineThreads), 0, s, r);
    }
    ScanArgs d = r;
    d.read_desc = 1;
    const uint32_t lds = a.structure && a.inst_keys ? 2u * (kMsThreads * ITEMS + 1) : 0u;
    if constexpr (!PE) {
        if (a.inst_conc || a.event_pack) {
            launch_down<PMAX, MW, ITEMS, true, false, SYM>(d, q, own, grid, lds, s);
            return;
        }
    }
    launch_down<PMAX, MW, ITEMS, false, PE, SYM>(d, q, own, grid, lds, s);
}

template <int PMAX, int MW, int ITEMS, bool PE>
static void launch_ms_s(const ScanArgs& a, const PeParam<PE>& q, hipStream_t s) {
    if constexpr (!PE && (PMAX >= 4 || MW == 4)) {
        if (a.class_mask <= 7u) {
            launch_ms_t<PMAX, MW, ITEMS, PE, true>(a, q, s);
            return;
        }
    }
    launch_ms_t<PMAX, MW, ITEMS, PE, false>(a, q, s);
}

template <int ITEMS, bool PE>
static void launch_ms_items(const ScanArgs& a, const PeParam<PE>& q, hipStream_t s) {
    if (a.max_states <= 8) {
        if (a.n_props <= 1) launch_ms_s<1, 2, ITEMS, PE>(a, q, s);
        else if (a.n_props <= 2) launch_ms_s<2, 2, ITEMS, PE>(a, q, s);
        else if (a.n_props <= 4) launch_ms_s<4, 2, ITEMS, PE>(a, q, s);
        else launch_ms_s<8, 2, ITEMS, PE>(a, q, s);
    } else {
        if (a.n_props <= 1) launch_ms_s<1, 4, ITEMS, PE>(a, q, s);
        else if (a.n_props <= 2) launch_ms_s<2, 4, ITEMS, PE>(a, q, s);
        else launch_ms_s<4, 4, ITEMS, PE>(a, q, s);
    }
}

// items: words per thread, 16 (4,096-word tiles) or 32 (8,192-word tiles; not
// with parent events).  The workspace arrays are sized for 16 (the more tiles).
hipError_t launch_mapscan(const ScanArgs& a, int items, const ParentArgs* pe, hipStream_t s) {
    if (a.n_props < 1 || a.n_props > (a.max_states <= 8 ? 8u : 4u) || (a.structure && a.n_props > 4) ||
        !a.desc || !a.agg || !a.prefix || !a.trec || (items != 16 && items != 32) ||
        (pe && (items != 16 || a.inst_conc || a.event_pack)))
        return hipErrorInvalidValue;
    if (pe) launch_ms_items<16, true>(a, *pe, s);
    else if (items == 16) launch_ms_items<16, false>(a, NoParent{}, s);
    else launch_ms_items<32, false>(a, NoParent{}, s);
    return hipGetLastError();
}

}  // namespace ltl4c
