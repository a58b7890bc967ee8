// First pass of Algorithm 2 (Filter-Junctions with E = Bloom filter) and the
// sentinel set, for gfx950.
//
//   k_sentinels   normalised first and last k-mer of every string (the
//                 sentinel vertices of the Preliminaries section, both
//                 strands): a hash table of them per set, plus two bit
//                 prefilters
//   k_fill        loop 1 of Algorithm 1 with every position marked: every
//                 normalised (k+1)-mer goes into its set's filter (load first,
//                 atomicOr only for bits still clear)
//   k_query       loop 2 of Algorithm 1: a position stays marked when it is a
//                 string end, a sentinel k-mer, or when any of its six
//                 neighbour (k+1)-mers other than the actual predecessor and
//                 successor edge tests present (in = 1 and out = 1 fails).
//                 Writes the C1 bitmap with one wave ballot per 64 positions.
//
// Both filter layouts share the tile loop (template flag BLOCKED):
//   standard  h bits anywhere in the filter; the query probes its six
//             neighbours level by level (bit t of every neighbour still
//             possibly present, so up to six loads are in flight per lane)
//   blocked   all h bits of an edge x.m.y in the 64-bit block of its
//             normalised middle m (see MiddleKey); a position's out-edges
//             share the block of its out-middle v[1..k-1], its in-edges the
//             block of its in-middle v[0..k-2] -- the out-middle of the
//             position before, passed by a wave shuffle -- so a position
//             costs one random load.
//
// Sequence reads: each workgroup stages its tile's packed words (plus one
// word before and five after, covering predecessor, successor and the
// longest window) in LDS with coalesced 64-bit loads, in both base orders;
// lanes then cut their k-mers' windows out of LDS (Stage).
#include <algorithm>

#include "device.hpp"

namespace tp {

__global__ void k_zero(uint4 *p, uint64_t n) {
    for (uint64_t i = blockIdx.x * (uint64_t)blockDim.x + threadIdx.x; i < n;
         i += (uint64_t)gridDim.x * blockDim.x)
        p[i] = make_uint4(0, 0, 0, 0);
}

__global__ void k_zero_bytes(uint8_t *p, uint64_t n) {
    uint64_t i = blockIdx.x * (uint64_t)blockDim.x + threadIdx.x;
    if (i < n)
        p[i] = 0;
}

__global__ void k_fill_u64(uint64_t *p, uint64_t n, uint64_t v) {
    for (uint64_t i = blockIdx.x * (uint64_t)blockDim.x + threadIdx.x; i < n;
         i += (uint64_t)gridDim.x * blockDim.x)
        p[i] = v;
}

__global__ __launch_bounds__(BLOCK) void k_clear(ClearList c) {
    for (uint32_t q = 0; q < c.n; ++q) {
        uint4 *p = (uint4 *)c.r[q].p;
        const uint4 *src = (const uint4 *)c.r[q].src;
        const uint32_t v = c.r[q].v;
        for (uint64_t i = blockIdx.x * (uint64_t)BLOCK + threadIdx.x; i < c.r[q].n16;
             i += (uint64_t)gridDim.x * BLOCK)
            p[i] = src ? src[i] : make_uint4(v, v, v, v);
    }
}

// One workgroup: the copies, and the sums of the sketch (a tree of exact
// powers of two, so the same in every run).
__global__ __launch_bounds__(BLOCK) void k_publish(ClearList c, const uint32_t *hll,
                                                   SketchSum *sketch) {
    __shared__ double wz[BLOCK / 64];
    __shared__ uint32_t w0[BLOCK / 64];
    for (uint32_t q = 0; q < c.n; ++q)
        for (uint64_t i = threadIdx.x; i < c.r[q].n16; i += BLOCK)
            ((uint4 *)c.r[q].p)[i] = ((const uint4 *)c.r[q].src)[i];
    if (!hll)
        return;
    double z = 0;
    uint32_t zeros = 0;
    for (uint32_t i = threadIdx.x; i < HLL_M; i += BLOCK) {
        const uint32_t r = hll[i];
        z += __longlong_as_double((long long)(1023 - r) << 52);  // 2^-r (r <= 64)
        zeros += r == 0;
    }
    for (int d = 32; d; d >>= 1) {
        z += __shfl_xor(z, d, 64);
        zeros += __shfl_xor(zeros, d, 64);
    }
    if ((threadIdx.x & 63) == 0) {
        wz[threadIdx.x >> 6] = z;
        w0[threadIdx.x >> 6] = zeros;
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        for (uint32_t q = 1; q < BLOCK / 64; ++q) {
            z += wz[q];
            zeros += w0[q];
        }
        sketch->z = z;
        sketch->zeros = zeros;
    }
}

static uint32_t grid_for(uint64_t n, uint32_t cap = 8192) {
    uint64_t g = (n + BLOCK - 1) / BLOCK;
    return (uint32_t)(g < 1 ? 1 : (g > cap ? cap : g));
}

hipError_t launch_clear(const ClearList &c, hipStream_t s) {
    uint64_t most = 0;
    for (uint32_t q = 0; q < c.n; ++q)
        most = std::max(most, c.r[q].n16);
    if (most)
        hipLaunchKernelGGL(k_clear, dim3(grid_for(most)), dim3(BLOCK), 0, s, c);
    return hipGetLastError();
}

hipError_t launch_publish(const ClearList &copies, const uint32_t *hll, SketchSum *sketch,
                          hipStream_t s) {
    hipLaunchKernelGGL(k_publish, dim3(1), dim3(BLOCK), 0, s, copies, hll, sketch);
    return hipGetLastError();
}

hipError_t launch_zero(void *p, uint64_t bytes, hipStream_t s) {
    if (bytes == 0)
        return hipSuccess;
    uint64_t n16 = bytes / 16, tail = bytes % 16;
    if (n16) {
        hipLaunchKernelGGL(k_zero, dim3(grid_for(n16)), dim3(BLOCK), 0, s, (uint4 *)p, n16);
    }
    if (tail) {
        hipLaunchKernelGGL(k_zero_bytes, dim3(1), dim3(BLOCK), 0, s, (uint8_t *)p + n16 * 16,
                           tail);
    }
    return hipGetLastError();
}

hipError_t launch_fill_u64(uint64_t *p, uint64_t n, uint64_t v, hipStream_t s) {
    if (n == 0)
        return hipSuccess;
    hipLaunchKernelGGL(k_fill_u64, dim3(grid_for(n)), dim3(BLOCK), 0, s, p, n, v);
    return hipGetLastError();
}

// Stage the packed words of tile `tile`: word i of the stage is global word
// tile*TILE_WORDS - 1 + i (zero outside the buffer).
__device__ __forceinline__ void stage_tile(const SeqArgs &a, uint64_t tile, Stage &sg) {
    const int64_t w0 = (int64_t)(tile * TILE_WORDS) - 1;
    for (uint32_t i = threadIdx.x; i < STAGE_WORDS; i += blockDim.x) {
        const int64_t gw = w0 + (int64_t)i;
        stage_word(sg, i, (gw >= 0 && (uint64_t)gw < a.seq_words) ? a.seq[gw] : 0ull);
    }
}

// ------------------------------------------------------------ sentinels (a0)

// Sentinel i: the first (i even) or last k-mer of string i / 2.
template <class T>
__device__ __forceinline__ Strands<T> sentinel_at(const SeqArgs &a, uint32_t i) {
    const DString &s = a.strings[i / 2];
    const uint64_t p = i & 1 ? s.gend - a.k : s.gstart;
    return strands(KT<T>::window(a.seq + (p >> 5), (uint32_t)(p & 31), a.k), a.k);
}

// Each set's sentinel table and the prefilters (empty beforehand): thread i
// inserts sentinel i by claiming a slot's claim word; a k-mer that another
// sentinel of the set has already claimed (read again from the sequence) is
// not inserted twice.  Lookups run in later kernels, after every value is in
// place.
template <class T>
__global__ __launch_bounds__(BLOCK) void k_sentinels(SeqArgs a, uint32_t n, T *tab, uint32_t *owner,
                                                     uint32_t *pf, uint32_t *pf_g,
                                                     uint32_t pf_log2) {
    const uint32_t i = blockIdx.x * BLOCK + threadIdx.x;
    if (i >= n)
        return;
    const bool single = a.single != 0;
    const Strands<T> st = sentinel_at<T>(a, i);
    const T v = norm(st, single), mid_ones = KT<T>::ones(2 * (a.k - 1));
    const uint32_t b = prefilter_bit(slot_hash(v), pf_log2);
    atomicOr(&pf[b >> 5], 1u << (b & 31));
    const MiddleKey in = middle_key((T)(st.fwd >> 2), (T)(st.rc & mid_ones), single, 0);
    const MiddleKey out = middle_key((T)(st.fwd & mid_ones), (T)(st.rc >> 2), single, 0);
    const uint32_t c = prefilter_bit_g((uint32_t)(in.g >> 32) + (uint32_t)(out.g >> 32), pf_log2);
    atomicOr(&pf_g[c >> 5], 1u << (c & 31));
    const SetDesc &d = a.sets[a.strings[i / 2].set];
    if (!d.sent_tab_log2)
        return;
    const uint32_t mask = (1u << d.sent_tab_log2) - 1;
    T *t = tab + d.sent_tab_off;
    uint32_t *o = owner + d.sent_tab_off;
    uint32_t s = sent_home(v, d.sent_tab_log2);
    for (uint32_t probe = 0; probe <= mask; ++probe) {
        const uint32_t prev = atomicCAS(&o[s], ~0u, i);
        if (prev == ~0u) {
            t[s] = v;
            return;
        }
        if (norm(sentinel_at<T>(a, prev), single) == v)
            return;  // the same k-mer, inserted by another sentinel
        s = (s + 1) & mask;
    }
}

void clear_sentinels(ClearList &c, int W, const SentArgs &sa, uint32_t *tab_owner,
                     uint64_t tab_slots) {
    c.add((void *)sa.prefilter, 2ull * 4 * prefilter_words(sa.pf_log2));
    c.add((void *)sa.table, tab_slots * 8 * W, ~0u);
    c.add(tab_owner, tab_slots * 4, ~0u);
}

hipError_t launch_sentinels(int W, const SeqArgs &a, const SentArgs &sa, uint32_t *tab_owner,
                            hipStream_t s) {
    static_assert((4u << SENT_TAB_MIN_LOG2) % 16 == 0, "claim words clear in 16-byte pieces");
    if (sa.n == 0)
        return hipSuccess;
    return by_width(W, [&](auto tag) {
        using T = decltype(tag);
        hipLaunchKernelGGL(k_sentinels<T>, dim3((sa.n + BLOCK - 1) / BLOCK), dim3(BLOCK), 0, s, a,
                           sa.n, (T *)sa.table, tab_owner, (uint32_t *)sa.prefilter,
                           (uint32_t *)sa.prefilter + prefilter_words(sa.pf_log2), sa.pf_log2);
        return hipGetLastError();
    });
}

// ---------------------------------------------------------------- fill (a1)

// Standard layout: h words, loads issued together, atomicOr for clear bits.
template <class T>
__device__ __forceinline__ uint32_t insert_standard(const BloomArgs &f, const Strands<T> &e,
                                                    bool single) {
    const BloomHash bh = bloom_hash(norm(e, single));
    uint64_t idx[16];
    uint32_t cur[16];
#pragma unroll
    for (uint32_t t = 0; t < 16; ++t) {
        if (t < f.h) {
            idx[t] = (bh.h1 + (uint64_t)t * bh.h2) & f.mask;
            cur[t] = __hip_atomic_load(&f.words[idx[t] >> 5], __ATOMIC_RELAXED,
                                       __HIP_MEMORY_SCOPE_AGENT);
        }
    }
    uint32_t atomics = 0;
#pragma unroll
    for (uint32_t t = 0; t < 16; ++t) {
        if (t < f.h) {
            const uint32_t bit = 1u << (idx[t] & 31);
            if (!(cur[t] & bit)) {
                __hip_atomic_fetch_or(&f.words[idx[t] >> 5], bit, __ATOMIC_RELAXED,
                                      __HIP_MEMORY_SCOPE_AGENT);
                ++atomics;
            }
        }
    }
    return atomics;
}

// Blocked layout: one 64-bit block keyed by the edge's middle.  With a
// dedup table dd (LDS), an edge whose effect on the filter -- block, offset,
// stride and pair, which fix the bits it sets -- some lane of this workgroup
// has already sent is skipped: that lane's load and atomic complete within
// the kernel, and filter bits are only ever set.  Lanes racing on one entry
// both send.
__device__ __forceinline__ uint32_t insert_blocked(const BloomArgs &f, const MiddleKey &key,
                                                   uint32_t j, unsigned long long *dd) {
    unsigned long long *blocks = (unsigned long long *)f.words;
    if (dd) {
        const unsigned long long id =
            (unsigned long long)key.block << 16 | key.a | key.d << 6 | j << 12;
        unsigned long long *slot = &dd[(key.block * 16 + j) & (FILL_DD - 1)];
        if (*slot == id)
            return 0;
        *slot = id;
    }
    const uint64_t m = pair_mask(key.a, key.d, j, f.h);
    const unsigned long long cur =
        __hip_atomic_load(&blocks[key.block], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    if ((cur & m) == m)
        return 0;
    __hip_atomic_fetch_or(&blocks[key.block], (unsigned long long)m, __ATOMIC_RELAXED,
                          __HIP_MEMORY_SCOPE_AGENT);
    return 1;
}

// The blocked filter's key of the (k+1)-mer at r, and its pair.
template <class T>
__device__ __forceinline__ MiddleKey edge_key(const Stage &sg, uint32_t r, uint32_t k, bool single,
                                              uint64_t nblock_mask, uint32_t *pair) {
    uint32_t x, y;
    const Strands<T> m = kmer_between<T>(sg, r + 1, k - 1, &x, &y);
    const MiddleKey key = middle_key(m.fwd, m.rc, single, nblock_mask);
    *pair = pair_index(key.orient, x, y);
    return key;
}

// Whether a round inserts the (k+1)-mer at r: one of its k-mers is in the
// round's class.
template <class T>
__device__ __forceinline__ bool edge_in_class(const Stage &sg, uint32_t r, uint32_t k, bool single,
                                              uint32_t lo, uint32_t hi) {
    return in_class(class_subrange(norm(kmer_at<T>(sg, r, k), single)), lo, hi) ||
           in_class(class_subrange(norm(kmer_at<T>(sg, r + 1, k), single)), lo, hi);
}

template <class T, bool BLOCKED>
__global__ __launch_bounds__(BLOCK) void k_fill(SeqArgs a, BloomArgs pool, Counters *cnt) {
    __shared__ Stage sg;
    __shared__ unsigned long long block_atomics;
    extern __shared__ unsigned long long dd_lds[];  // FILL_DD entries when deduplicating
    const uint32_t L = a.k + 1;
    const bool single = a.single != 0;
    unsigned long long *dd = BLOCKED && a.fill_dedup ? dd_lds : nullptr;
    uint32_t dd_set = ~0u;  // the set whose filter effects dd holds
    if (threadIdx.x == 0)
        block_atomics = 0;
    uint32_t my_atomics = 0;
    // with dedup, runs of homologous tiles
    RunCursor rc = run_cursor(a, dd ? (a.chunk > FILL_CHUNK ? a.chunk : FILL_CHUNK) : a.chunk);
    for (uint64_t tile; run_next(a, rc, &tile);) {
        const uint64_t t0 = tile * TILE;
        const TileInfo ti = a.tiles[tile];
        const uint32_t lo = ti.str_lo, hi = ti.str_hi;
        if (lo == hi)
            continue;
        __syncthreads();
        stage_tile(a, tile, sg);
        if (dd && ti.set != dd_set) {
            // block indices are relative to the set's own filter
            for (uint32_t q = threadIdx.x; q < FILL_DD; q += BLOCK)
                dd[q] = ~0ull;
            dd_set = ti.set;
        }
        __syncthreads();
        const TileSet ts = tile_set_of(a, pool, ti.set);
        const bool one = lo + 1 == hi;
        Span sp = one ? span_of(a.strings, lo, t0) : Span{0, -1};
        const Part part = tile_part(a);
        for (uint32_t it = part.lo; it < part.hi; ++it) {
            const uint32_t q = it * BLOCK + threadIdx.x, r = q + 32;
            if (!one && (int32_t)q >= sp.ge)
                sp = span_at(a.strings, lo, hi, t0, q);
            if ((int32_t)q < sp.gs || (int32_t)(q + L) > sp.ge)
                continue;
            if (a.classes && !edge_in_class<T>(sg, r, a.k, single, ts.cls_lo, ts.cls_hi))
                continue;
            if (BLOCKED) {
                uint32_t j;
                const MiddleKey key = edge_key<T>(sg, r, a.k, single, ts.f.mask >> 6, &j);
                my_atomics += insert_blocked(ts.f, key, j, dd);
            } else {
                my_atomics += insert_standard(ts.f, kmer_at<T>(sg, r, L), single);
            }
        }
    }
    if (my_atomics)
        atomicAdd(&block_atomics, (unsigned long long)my_atomics);
    __syncthreads();
    if (threadIdx.x == 0 && block_atomics)
        atomicAdd(&cnt->fill_atomics, block_atomics);
}

static size_t fill_lds_bytes(const SeqArgs &a, bool blocked) {
    return blocked && a.fill_dedup ? FILL_DD * sizeof(unsigned long long) : 0;
}

hipError_t launch_fill(int W, const SeqArgs &a, const BloomArgs &pool, Counters *cnt,
                       uint32_t grid, hipStream_t s) {
    if (a.n_tiles == 0)
        return hipSuccess;
    return by_width(W, [&](auto tag) {
        using T = decltype(tag);
        if (pool.blocked)
            hipLaunchKernelGGL((k_fill<T, true>), dim3(grid), dim3(BLOCK), fill_lds_bytes(a, true),
                               s, a, pool, cnt);
        else
            hipLaunchKernelGGL((k_fill<T, false>), dim3(grid), dim3(BLOCK), 0, s, a, pool, cnt);
        return hipGetLastError();
    });
}

// ------------------------------------------------------- binned fill (a1)
//
// The same filter as k_fill, built without random atomics: a chunk of tiles
// at a time, every edge's filter effect becomes an item, the items are
// partitioned by region of the pool, and each region is applied in LDS.  A
// filter is the OR of its edges' bits, so the order of application does not
// matter, and an item that finds no room in its bucket is applied to the pool
// directly (the pool is zeroed first and a region is read before its items
// are ORed in).
//
//   k_bin_items    batches of a few tiles: the items of the batch, sorted by
//                  bucket in LDS, appended to their buckets
//   k_bin_split    buckets of several regions: batches of a bucket's items,
//                  sorted by region in LDS, appended to their regions
//   k_bin_apply    per region: the region's blocks in LDS, its items ORed in,
//                  the blocks written back
//
// An item is 4 bytes: its block within the bucket (21 bits), and the 11 bits
// that fix the filter bits it sets -- the pairs' masks are 32 templates (one
// per odd stride d) rotated by s = a + j*h*d mod 64, so (d, s) stand for the
// offset, stride and pair.  Room per bucket and region is laid out from the
// edge count (a hash spreads them evenly), so nothing is counted beforehand:
// an item is written and read once per level, 8 or 16 bytes an edge in all.
//
// The standard filter's items are one per edge and hash function: the block
// within the bucket and 6 bits for the bit in it.

constexpr uint32_t BIN_EFFECT_BITS = 11, BIN_BIT_BITS = 6;
template <bool STD> constexpr uint32_t effect_bits() { return STD ? BIN_BIT_BITS : BIN_EFFECT_BITS; }

__device__ __forceinline__ uint32_t bin_effect(const MiddleKey &m, uint32_t j, uint32_t h) {
    return (m.d >> 1) << 6 | ((m.a + j * h * m.d) & 63u);
}

// Filter bits of template t (one per odd stride, t = bits u*d mod 64, u < h)
// rotated left by s.
__device__ __forceinline__ uint64_t rotl64(uint64_t t, uint32_t s) {
    return t << s | t >> ((64u - s) & 63u);
}

__device__ __forceinline__ uint64_t stride_template(uint32_t d, uint32_t h) {
    uint64_t m = 0;
    for (uint32_t t = 0; t < h; ++t)
        m |= 1ull << ((t * d) & 63u);
    return m;
}

// An item without room, of the bucket that starts at block block0: straight
// into the pool (load first, as insert_blocked does).
template <bool STD>
__device__ __forceinline__ uint32_t bin_direct(const BloomArgs &pool, uint64_t block0,
                                               uint32_t item) {
    unsigned long long *p =
        (unsigned long long *)pool.words + block0 + (item >> effect_bits<STD>());
    const uint64_t m = STD ? 1ull << (item & 63u)
                           : rotl64(stride_template((item >> 5 & 62u) | 1u, pool.h), item & 63u);
    const unsigned long long cur =
        __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    if ((cur & m) == m)
        return 0;
    __hip_atomic_fetch_or(p, (unsigned long long)m, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    return 1;
}

// A batch's tile: its range of strings, its set's filter, and its string when
// it has just one.
struct BinTile {
    uint64_t t0;
    uint64_t mask;       // the set's filter bits - 1
    uint32_t block0;     // its first block in the pool
    uint32_t lo, hi, cls_lo, cls_hi;
    Span sp;
};

// Stage a batch: entries [e0, e0 + TILES) of the first-pass order, those from
// end on empty.  Whole workgroup; ends synchronised.
template <uint32_t TILES, uint32_t NT>
__device__ __forceinline__ void bin_stage(const SeqArgs &a, uint64_t e0, uint64_t end, Stage *sg,
                                          BinTile *tl) {
    const uint32_t nt = (uint32_t)min((uint64_t)TILES, end - e0);
    if (threadIdx.x < TILES) {
        BinTile x{};
        x.sp = Span{0, -1};  // (no string: no edge)
        if (threadIdx.x < nt) {
            const uint64_t tile = a.tile_order[e0 + threadIdx.x];
            const TileInfo ti = a.tiles[tile];
            const SetDesc &d = a.sets[ti.set];
            x.t0 = tile * TILE;
            x.lo = ti.str_lo;
            x.hi = ti.str_hi;
            x.block0 = (uint32_t)(d.bloom_off >> 1);
            x.mask = d.bloom_mask;
            x.cls_lo = d.cls_lo;
            x.cls_hi = d.cls_hi;
            if (x.lo + 1 == x.hi)
                x.sp = span_of(a.strings, x.lo, x.t0);
        }
        tl[threadIdx.x] = x;
    }
    for (uint32_t i = threadIdx.x; i < nt * STAGE_WORDS; i += NT) {
        const uint32_t j = i / STAGE_WORDS, u = i % STAGE_WORDS;
        const int64_t gw = (int64_t)((uint64_t)a.tile_order[e0 + j] * TILE_WORDS) - 1 + u;
        stage_word(sg[j], u, (gw >= 0 && (uint64_t)gw < a.seq_words) ? a.seq[gw] : 0ull);
    }
    __syncthreads();
}

// The edges are those k_fill inserts: every (k+1)-mer within a string, of the
// round's class when there are rounds.
template <class T, uint32_t NB, uint32_t NT, uint32_t PER, bool CLASSES>
__global__ __launch_bounds__(NT) __attribute__((amdgpu_waves_per_eu(KT<T>::W <= 2 && !CLASSES ? 8 : 4)))
void k_bin_items(SeqArgs a, BloomArgs pool, BinArgs b,
                                                         Counters *cnt) {
    constexpr uint32_t TILES = NT * PER / TILE;
    __shared__ BinSort<NB, NT, PER> sh;
    __shared__ Stage sg[TILES];
    __shared__ BinTile tl[TILES];
    const uint32_t L = a.k + 1, k = a.k;
    const bool single = a.single != 0;
    const uint32_t lpb = bin_lanes(b.n_buckets, NT * PER);
    const uint64_t batches = (b.t_hi - b.t_lo + TILES - 1) / TILES;
    const auto off = [&](uint32_t i) { return b.off[i]; };
    uint32_t atomics = 0;
    for (uint32_t i = threadIdx.x; i < NB; i += NT)
        sh.cnt[i] = 0;
    for (uint64_t batch = blockIdx.x; batch < batches; batch += gridDim.x) {
        bin_stage<TILES, NT>(a, b.t_lo + batch * TILES, b.t_hi, sg, tl);
        uint32_t item[PER], at[PER];
#pragma unroll
        for (uint32_t q = 0; q < PER; ++q) {
            item[q] = 0;
            at[q] = ~0u;
            const uint32_t j = q * NT / TILE, p = (q * NT & (TILE - 1)) + threadIdx.x;
            const BinTile &x = tl[j];
            const Span sp = x.hi - x.lo > 1 ? span_at(a.strings, x.lo, x.hi, x.t0, p) : x.sp;
            if ((int32_t)p < sp.gs || (int32_t)(p + L) > sp.ge)
                continue;
            if (CLASSES && !edge_in_class<T>(sg[j], p + 32, k, single, x.cls_lo, x.cls_hi))
                continue;
            uint32_t pair;
            const MiddleKey key = edge_key<T>(sg[j], p + 32, k, single, x.mask >> 6, &pair);
            const uint32_t block = x.block0 + (uint32_t)key.block;
            item[q] = (block & ((1u << b.bucket_log2) - 1)) << BIN_EFFECT_BITS |
                      bin_effect(key, pair, pool.h);
            const uint32_t bucket = block >> b.bucket_log2;
            at[q] = bucket << 14 | atomicAdd(&sh.cnt[bucket], 1u);
        }
        bin_append(sh, item, at, b.n_buckets, lpb, b.cursor, off, b.items_a,
                            [&](uint32_t bucket, uint32_t it) {
                                atomics += bin_direct<false>(
                                    pool, (uint64_t)bucket << b.bucket_log2, it);
                            });
    }
    if (atomics)
        atomicAdd(&cnt->fill_atomics, (unsigned long long)atomics);
}

// The standard filter's items: PER positions per thread, hashed once, then
// their bits appended one hash function at a time (h batches).
template <class T, uint32_t NB, uint32_t NT, uint32_t PER, bool CLASSES>
__global__ __launch_bounds__(NT) void k_bin_items_std(SeqArgs a, BloomArgs pool, BinArgs b,
                                                      Counters *cnt) {
    constexpr uint32_t TILES = NT * PER / TILE;
    __shared__ BinSort<NB, NT, PER> sh;
    __shared__ Stage sg[TILES];
    __shared__ BinTile tl[TILES];
    const uint32_t L = a.k + 1, k = a.k;
    const bool single = a.single != 0;
    const uint32_t lpb = bin_lanes(b.n_buckets, NT * PER);
    const uint64_t batches = (b.t_hi - b.t_lo + TILES - 1) / TILES;
    const auto off = [&](uint32_t i) { return b.off[i]; };
    uint32_t atomics = 0;
    for (uint32_t i = threadIdx.x; i < NB; i += NT)
        sh.cnt[i] = 0;
    for (uint64_t batch = blockIdx.x; batch < batches; batch += gridDim.x) {
        bin_stage<TILES, NT>(a, b.t_lo + batch * TILES, b.t_hi, sg, tl);
        uint64_t h1[PER], h2[PER];
        uint32_t in = 0;  // positions with an edge
#pragma unroll
        for (uint32_t q = 0; q < PER; ++q) {
            h1[q] = h2[q] = 0;
            const uint32_t j = q * NT / TILE, p = (q * NT & (TILE - 1)) + threadIdx.x;
            const BinTile &x = tl[j];
            const Span sp = x.hi - x.lo > 1 ? span_at(a.strings, x.lo, x.hi, x.t0, p) : x.sp;
            if ((int32_t)p < sp.gs || (int32_t)(p + L) > sp.ge)
                continue;
            if (CLASSES && !edge_in_class<T>(sg[j], p + 32, k, single, x.cls_lo, x.cls_hi))
                continue;
            const BloomHash bh = bloom_hash(norm(kmer_at<T>(sg[j], p + 32, L), single));
            h1[q] = bh.h1;
            h2[q] = bh.h2;
            in |= 1u << q;
        }
        for (uint32_t t = 0; t < pool.h; ++t) {
            uint32_t item[PER], at[PER];
#pragma unroll
            for (uint32_t q = 0; q < PER; ++q) {
                item[q] = 0;
                at[q] = ~0u;
                if (!((in >> q) & 1u))
                    continue;
                const BinTile &x = tl[q * NT / TILE];
                const uint64_t bit = ((uint64_t)x.block0 << 6) + (h1[q] & x.mask);
                h1[q] += h2[q];
                const uint32_t bucket = (uint32_t)(bit >> (6 + b.bucket_log2));
                item[q] = (uint32_t)bit & ((64u << b.bucket_log2) - 1);
                at[q] = bucket << 14 | atomicAdd(&sh.cnt[bucket], 1u);
            }
            bin_append(sh, item, at, b.n_buckets, lpb, b.cursor, off, b.items_a,
                                    [&](uint32_t bucket, uint32_t it) {
                                        atomics += bin_direct<true>(
                                            pool, (uint64_t)bucket << b.bucket_log2, it);
                                    });
        }
    }
    if (atomics)
        atomicAdd(&cnt->fill_atomics, (unsigned long long)atomics);
}

// One batch of one bucket's items (blockIdx.y: the bucket, blockIdx.x: the
// batch) appended to the bucket's regions.
template <bool STD>
__global__ __launch_bounds__(BIN_BLOCK) void k_bin_split(BloomArgs pool, BinArgs b,
                                                         Counters *cnt) {
    constexpr uint32_t NT = BIN_BLOCK, PER = BIN_PER, NB = 1u << (BIN_LOCAL_LOG2 - BIN_REGION_LOG2);
    __shared__ BinSort<NB, NT, PER> sh;
    const uint32_t bucket = blockIdx.y, shift = b.region_log2 + effect_bits<STD>();
    const uint32_t sub = 1u << (b.bucket_log2 - b.region_log2), r0 = bucket * sub;
    const uint64_t o = b.off[bucket];
    const uint64_t n = min((uint64_t)b.cursor[bucket], b.off[bucket + 1] - o);
    const uint64_t i0 = (uint64_t)blockIdx.x * BIN_BATCH;
    if (i0 >= n)
        return;
    for (uint32_t i = threadIdx.x; i < NB; i += NT)
        sh.cnt[i] = 0;
    uint32_t item[PER], at[PER], atomics = 0;
#pragma unroll
    for (uint32_t q = 0; q < PER; ++q) {
        const uint64_t i = i0 + q * NT + threadIdx.x;
        item[q] = i < n ? b.items_a[o + i] : 0;
    }
    __syncthreads();
#pragma unroll
    for (uint32_t q = 0; q < PER; ++q) {
        const uint32_t reg = item[q] >> shift;
        at[q] = i0 + q * NT + threadIdx.x < n ? reg << 14 | atomicAdd(&sh.cnt[reg], 1u) : ~0u;
    }
    const uint32_t nb = min(sub, b.n_regions - r0);
    bin_append(sh, item, at, nb, bin_lanes(nb, NT * PER), b.cursor + b.n_buckets + r0,
               [&](uint32_t i) { return b.roff[r0 + i]; }, b.items_b, [&](uint32_t, uint32_t it) {
                            atomics += bin_direct<STD>(pool, (uint64_t)bucket << b.bucket_log2, it);
                        });
    if (atomics)
        atomicAdd(&cnt->fill_atomics, (unsigned long long)atomics);
}

// One workgroup per region (of at most 2^REGION_LOG2 blocks): the region's
// blocks in LDS, its items ORed in, the blocks written back.  Counts the items that set a bit not yet set and, in
// the last chunk of a one-set pool, the filter's bits.
template <uint32_t REGION_LOG2, bool STD>
__global__ __launch_bounds__(BIN_BLOCK) void k_bin_apply(BloomArgs pool, BinArgs b, Counters *cnt) {
    constexpr uint32_t NT = BIN_BLOCK, U = 4;
    __shared__ __align__(16) unsigned long long reg[1u << REGION_LOG2];
    __shared__ uint64_t tmpl[32];
    __shared__ uint32_t fresh_wg, bits_wg;
    const uint64_t r = blockIdx.x, blk0 = r << b.region_log2;
    const uint32_t nb = (uint32_t)min(1ull << b.region_log2, b.n_blocks - blk0);
    const bool split = b.bucket_log2 != b.region_log2;
    const uint64_t o = split ? b.roff[r] : b.off[r];
    const uint64_t room = (split ? b.roff[r + 1] : b.off[r + 1]) - o;
    const uint64_t n = min((uint64_t)b.cursor[split ? b.n_buckets + r : r], room);
    const uint32_t *items = (split ? b.items_b : b.items_a) + o;
    if (threadIdx.x < 32)
        tmpl[threadIdx.x] = stride_template(2 * threadIdx.x + 1, pool.h);
    if (threadIdx.x == 0)
        fresh_wg = bits_wg = 0;
    // blocks in pairs (the pool's size and every region's start are even)
    ulonglong2 *blocks = (ulonglong2 *)((unsigned long long *)pool.words + blk0);
    ulonglong2 *reg2 = (ulonglong2 *)reg;
    for (uint32_t i = threadIdx.x; i < nb / 2; i += NT)
        reg2[i] = blocks[i];
    __syncthreads();
    const uint32_t lmask = (1u << b.region_log2) - 1;
    uint32_t fresh = 0, bits = 0;
    for (uint64_t i = threadIdx.x; i < n; i += U * NT) {
        uint32_t v[U];
#pragma unroll
        for (uint32_t q = 0; q < U; ++q)
            v[q] = i + (uint64_t)q * NT < n ? items[i + (uint64_t)q * NT] : 0u;
#pragma unroll
        for (uint32_t q = 0; q < U; ++q) {
            if (i + (uint64_t)q * NT >= n)
                continue;
            if (STD) {
                const uint32_t m = 1u << (v[q] & 31u);
                const uint32_t old = atomicOr((uint32_t *)reg + (v[q] >> 5 & (2 * lmask + 1)), m);
                fresh += (old & m) == 0;
            } else {
                const uint64_t m = rotl64(tmpl[v[q] >> 6 & 31u], v[q] & 63u);
                const unsigned long long old =
                    atomicOr(&reg[(v[q] >> BIN_EFFECT_BITS) & lmask], (unsigned long long)m);
                fresh += (old & m) != m;
            }
        }
    }
    if (fresh)
        atomicAdd(&fresh_wg, fresh);
    __syncthreads();
    for (uint32_t i = threadIdx.x; i < nb / 2; i += NT) {
        const ulonglong2 x = reg2[i];
        blocks[i] = x;
        bits += (uint32_t)(__popcll(x.x) + __popcll(x.y));
    }
    if (b.popcount)
        atomicAdd(&bits_wg, bits);
    __syncthreads();
    if (threadIdx.x == 0 && fresh_wg)
        atomicAdd(&cnt->fill_atomics, (unsigned long long)fresh_wg);
    if (threadIdx.x == 0 && b.popcount && bits_wg)
        atomicAdd(&b.popcount->bloom_popcount, (unsigned long long)bits_wg);
}

// Items per thread of k_bin_items.  Twelve leave room for two workgroups per
// CU, in registers (64, with a few spilled) and LDS, so that one's sort runs
// beside the other's hashing: 62 x 5 Mbp at k = 25 1.57 ms (1.50 with the runs
// written by a loop without a test for room), against 1.80 with sixteen and one
// workgroup and 1.69 with eight (more claims).  Four-word
// k-mers and rounds (two more k-mers to hash) need the registers of one
// workgroup per CU.
template <class T, bool CLASSES> struct ItemsPer {
    static constexpr uint32_t N = KT<T>::W == 4 ? 8 : CLASSES ? 16 : 12;
};

// PER items per thread (SPER positions with the standard filter).
template <class T, uint32_t NB, bool CLASSES, uint32_t PER, uint32_t SPER>
static void bin_items_n(const SeqArgs &a, const BloomArgs &pool, const BinArgs &b, Counters *cnt,
                        hipStream_t s) {
    constexpr uint32_t NT = BIN_BLOCK, TILES = NT * PER / TILE, STILES = NT * SPER / TILE;
    const uint64_t n = b.t_hi - b.t_lo;
    if (pool.blocked)
        hipLaunchKernelGGL((k_bin_items<T, NB, NT, PER, CLASSES>),
                           dim3((uint32_t)min((n + TILES - 1) / TILES, 2ull * b.n_cu)), dim3(NT),
                           0, s, a, pool, b, cnt);
    else
        hipLaunchKernelGGL((k_bin_items_std<T, NB, NT, SPER, CLASSES>),
                           dim3((uint32_t)min((n + STILES - 1) / STILES, (uint64_t)b.n_cu)),
                           dim3(NT), 0, s, a, pool, b, cnt);
}

// A tile to a workgroup where the larger batches would be fewer than the CUs
// (0.4 Mbp, 195 tiles, standard filter: 25 workgroups 37 us, 195 21 us).
template <class T, uint32_t NB, bool CLASSES>
static void bin_items_t(const SeqArgs &a, const BloomArgs &pool, const BinArgs &b, Counters *cnt,
                        hipStream_t s) {
    constexpr uint32_t PER = ItemsPer<T, CLASSES>::N;
    if (NB == BIN_BUCKETS && (b.t_hi - b.t_lo) * TILE < (uint64_t)b.n_cu * BIN_BLOCK * PER)
        bin_items_n<T, BIN_BUCKETS, CLASSES, TILE / BIN_BLOCK, TILE / BIN_BLOCK>(a, pool, b, cnt, s);
    else
        bin_items_n<T, NB, CLASSES, PER, 16>(a, pool, b, cnt, s);
}

template <class T>
static void bin_items_w(const SeqArgs &a, const BloomArgs &pool, const BinArgs &b, Counters *cnt,
                        hipStream_t s) {
    auto *fn = b.n_buckets <= BIN_BUCKETS
                   ? (a.classes ? bin_items_t<T, BIN_BUCKETS, true> : bin_items_t<T, BIN_BUCKETS, false>)
                   : (a.classes ? bin_items_t<T, BIN_MAX_BUCKETS, true>
                                : bin_items_t<T, BIN_MAX_BUCKETS, false>);
    fn(a, pool, b, cnt, s);
}

hipError_t launch_fill_binned(int W, const SeqArgs &a, const BloomArgs &pool, Counters *cnt,
                              BinArgs b, uint32_t tiles_per_chunk, hipStream_t s) {
    if (a.n_tiles == 0)
        return hipSuccess;
    const bool split = b.bucket_log2 != b.region_log2;
    const uint64_t n_cursor = b.n_buckets + (split ? b.n_regions : 0u);
    SetCounters *const popcount = b.popcount;
    return by_width(W, [&](auto tag) {
        using T = decltype(tag);
        for (uint64_t t0 = 0; t0 < a.n_tiles; t0 += tiles_per_chunk) {
            b.t_lo = t0;
            b.t_hi = min(a.n_tiles, t0 + tiles_per_chunk);
            b.popcount = b.t_hi == a.n_tiles ? popcount : nullptr;
            hipError_t e = t0 || !b.cleared
                               ? launch_zero(b.cursor, n_cursor * sizeof(unsigned long long), s)
                               : hipSuccess;
            if (e != hipSuccess)
                return e;
            bin_items_w<T>(a, pool, b, cnt, s);
            if (split)
                hipLaunchKernelGGL(pool.blocked ? k_bin_split<false> : k_bin_split<true>,
                                   dim3(b.slices, b.n_buckets), dim3(BIN_BLOCK), 0, s, pool, b,
                                   cnt);
            auto *apply = b.region_log2 <= BIN_REGION_LOG2
                              ? (pool.blocked ? k_bin_apply<BIN_REGION_LOG2, false>
                                              : k_bin_apply<BIN_REGION_LOG2, true>)
                              : (pool.blocked ? k_bin_apply<BIN_REGION_LOG2 + 1, false>
                                              : k_bin_apply<BIN_REGION_LOG2 + 1, true>);
            hipLaunchKernelGGL(apply, dim3(b.n_regions), dim3(BIN_BLOCK), 0, s, pool, b, cnt);
            e = hipGetLastError();
            if (e != hipSuccess)
                return e;
        }
        return hipSuccess;
    });
}

// --------------------------------------------------------------- query (a2)

// Standard layout: membership of the six neighbour (k+1)-mers, N of them at a
// time, those probed level by level.  True when some neighbour has all h bits
// set (the neighbours after it are then not probed).
template <uint32_t N, class T>
__device__ __forceinline__ bool any_present_standard(const BloomArgs &f, const Strands<T> &st,
                                                     uint32_t k, uint32_t pa, uint32_t sb,
                                                     bool single, uint32_t &probes) {
    for (uint32_t i0 = 0; i0 < 6; i0 += N) {
        uint64_t h1[N], h2[N];
#pragma unroll
        for (uint32_t i = 0; i < N; ++i) {
            // out-neighbour v.c for the j-th base c other than the successor,
            // in-neighbour c.v for the j-th other than the predecessor
            const uint32_t j = (i0 + i) >> 1;
            const bool out = ((i0 + i) & 1) == 0;
            const uint32_t c = j + (j >= (out ? sb : pa));
            Strands<T> e;
            e.fwd = out ? (T)((st.fwd << 2) | (T)c) : (T)(((T)c << (2 * k)) | st.fwd);
            e.rc = out ? (T)(st.rc | ((T)(3 - c) << (2 * k))) : (T)((st.rc << 2) | (T)(3 - c));
            const BloomHash bh = bloom_hash(norm(e, single));
            h1[i] = bh.h1;
            h2[i] = bh.h2;
        }
        uint32_t alive = (1u << N) - 1;
        for (uint32_t t = 0; t < f.h && alive; ++t) {
            probes += __popc(alive);
            uint32_t v[N];
            uint32_t b[N];
#pragma unroll
            for (uint32_t n = 0; n < N; ++n) {
                const uint64_t idx = (h1[n] + (uint64_t)t * h2[n]) & f.mask;
                b[n] = (uint32_t)(idx & 31);
                v[n] = ((alive >> n) & 1u) ? __hip_atomic_load(&f.words[idx >> 5], __ATOMIC_RELAXED,
                                                                __HIP_MEMORY_SCOPE_AGENT)
                                            : 0u;
            }
#pragma unroll
            for (uint32_t n = 0; n < N; ++n)
                if (!((v[n] >> b[n]) & 1u))
                    alive &= ~(1u << n);
        }
        if (alive)
            return true;
    }
    return false;
}

// Value of the lane below (DPP wave shift right by one); lane 0 gets lane0.
__device__ __forceinline__ uint32_t from_below(uint32_t x, uint32_t lane0) {
    return (uint32_t)__builtin_amdgcn_update_dpp((int)lane0, (int)x, 0x138, 0xF, 0xF, false);
}
__device__ __forceinline__ uint64_t from_below(uint64_t x, uint64_t lane0) {
    return ((uint64_t)from_below((uint32_t)(x >> 32), (uint32_t)(lane0 >> 32)) << 32) |
           from_below((uint32_t)x, (uint32_t)lane0);
}

__device__ __forceinline__ uint64_t lane63(uint64_t x) {
    return ((uint64_t)(uint32_t)__builtin_amdgcn_readlane((int)(x >> 32), 63) << 32) |
           (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)x, 63);
}

// A flag of the lane below (mask: the lanes that have it), lane 0 the one
// carried; the mask's top bit carries on to the next step.
__device__ __forceinline__ bool flag_below(uint64_t mask, uint32_t &carry) {
    const uint64_t below = mask << 1 | carry;
    carry = (uint32_t)(mask >> 63);
    return __builtin_amdgcn_inverse_ballot_w64(below);
}

// What lanes pass on of a middle is its G, whose low word holds the key (offset
// a in bits 0-5; d >> 1 in bits 7-11, the byte offset of its stride's masks in
// pm), and its orientation as two flags.
constexpr uint32_t KEY_STRIDE = 0xF80u;

// w rotated right by s (mod 64).
__device__ __forceinline__ uint64_t rotr64(uint64_t w, uint32_t s) {
    const uint32_t lo = (uint32_t)w, hi = (uint32_t)(w >> 32);
    const bool sw = (s & 32u) != 0;  // rotating by 32 swaps the halves
    const uint32_t x = sw ? hi : lo, y = sw ? lo : hi;
    return (uint64_t)__builtin_amdgcn_alignbit(x, y, s) << 32 | __builtin_amdgcn_alignbit(y, x, s);
}

// The pair tests.  Rotating a block right by its key's offset a leaves pair
// j's bits at (j*h + t)*d mod 64, t < h: 32 x 16 masks (stride, pair), which a
// workgroup keeps in LDS (pm), so a test is a mask load and two bit
// operations.  A pair is 4p + q for the edge p.m.q in its middle's
// orientation, so with two bits each for p and q the three other edges of a
// side differ from the actual one by an exclusive-or.
//
// Nonzero bits of mask j that block w (rotated) lacks.
__device__ __forceinline__ uint32_t lacking(const uint64_t *pm, uint32_t at, uint64_t w) {
    const uint64_t m = *(const uint64_t *)((const char *)pm + at);
    return ((uint32_t)m & ~(uint32_t)w) | ((uint32_t)(m >> 32) & ~(uint32_t)(w >> 32));
}

// Whether some edge x.m.c (OUT) or c.m.y (in) other than the actual x.m.y is
// present in the middle's rotated block w.  Palindromic middles take each
// edge's own orientation.
template <bool OUT>
__device__ __forceinline__ uint32_t others_lacking(const uint64_t *pm, uint32_t key, bool rev,
                                                   uint64_t w, uint32_t x, uint32_t y) {
    const uint32_t base = key & KEY_STRIDE;
    const uint32_t pair = rev ? (15u - 4 * y - x) : (4 * x + y);
    const uint32_t at = base | pair << 3;
    // the varied base sits in the pair's low two bits, or its high two
    const uint32_t e = OUT == rev ? 32u : 8u;
    return min(min(lacking(pm, at ^ e, w), lacking(pm, at ^ (2 * e), w)),
               lacking(pm, at ^ (3 * e), w));
}

template <bool OUT>
__device__ __forceinline__ uint32_t others_lacking_palindrome(const uint64_t *pm, uint32_t key,
                                                              uint64_t w, uint32_t x,
                                                              uint32_t y) {
    uint32_t least = ~0u;
    for (uint32_t i = 1; i < 4; ++i) {
        const uint32_t p = OUT ? x : x ^ i, q = OUT ? y ^ i : y;
        least = min(least, lacking(pm, (key & KEY_STRIDE) | pair_index(2, p, q) << 3, w));
    }
    return least;
}

// What the two layouts' queries share per workgroup: the candidate words of
// a tile, the counters, the sketch of distinct candidate k-mers.
struct QueryShared {
    uint32_t pf[(1u << PF_MAX_LOG2) / 32];
    uint32_t hll[HLL_M];
    unsigned long long block_probes, cand_lds;
};

// A candidate k-mer's 64-bit hash into the sketch: the top HLL_LOG2 bits choose
// the register, the others give the rank.
__device__ __forceinline__ void sketch_add(QueryShared &qs, uint64_t hash) {
    const uint64_t rest = hash << HLL_LOG2;
    const uint32_t rank = rest ? (uint32_t)__clzll(rest) + 1 : 64 - HLL_LOG2 + 1;
    atomicMax(&qs.hll[(uint32_t)(hash >> (64 - HLL_LOG2))], rank);
}

template <uint32_t NT>
__device__ __forceinline__ void query_begin(QueryShared &qs, const uint32_t *prefilter,
                                            uint32_t pf_log2) {
    for (uint32_t i = threadIdx.x; i < prefilter_words(pf_log2); i += NT)
        qs.pf[i] = prefilter[i];
    for (uint32_t i = threadIdx.x; i < HLL_M; i += NT)
        qs.hll[i] = 0;
    if (threadIdx.x == 0)
        qs.block_probes = 0;
}

template <uint32_t NT>
__device__ __forceinline__ void query_end(const SeqArgs &a, QueryShared &qs, SetSum &cand,
                                          uint32_t my_probes, Counters *cnt, uint32_t *hll_out) {
    setsum_flush(cand, &qs.cand_lds, &a.set_cnt[0].candidates, SETCNT_STRIDE);
    if (my_probes)
        atomicAdd(&qs.block_probes, (unsigned long long)my_probes);
    __syncthreads();
    if (threadIdx.x == 0 && qs.block_probes)
        atomicAdd(&cnt->query_probes, qs.block_probes);
    if (a.sketch) {
        for (uint32_t i = threadIdx.x; i < HLL_M; i += NT) {
            const uint32_t v = qs.hll[i];
            if (v && v > __hip_atomic_load(&hll_out[i], __ATOMIC_RELAXED,
                                           __HIP_MEMORY_SCOPE_AGENT))
                atomicMax(&hll_out[i], v);
        }
    }
}

// A tile that no string touches: all-zero candidate words (every part of it
// writes them).
__device__ __forceinline__ void query_no_string(uint64_t tile, uint64_t *c1, uint64_t *c1u,
                                                uint32_t round) {
    if (threadIdx.x < TILE / 64) {
        c1[tile * (TILE / 64) + threadIdx.x] = 0;
        if (c1u && round == 0)
            c1u[tile * (TILE / 64) + threadIdx.x] = 0;
    }
}

// Blocked layout.  Each wave walks its own run of 512 consecutive positions
// of the tile, 64 at a time; a lane hashes its out-middle, loads that block,
// rotates it, and passes key and block to the lane above, whose in-middle it
// is; lane 63's carry to the next step's lane 0.  So a position hashes one
// middle and issues one random load.  Bound by instruction issue where the
// filter sits in the last-level cache (62 x 5 Mbp, b = 2^30, k = 25: 293
// vector instructions a position and 2.87 ms when k-mers were reversed and
// shifted in registers, each pair test rotated the block by itself and the
// sketch and the prefilter hashed on their own; now 200 and 2.29 ms; k = 100
// 7.0 -> 4.4 ms), by random loads where it does not (1.6 Gbp, a 1 GiB filter:
// 26.8 -> 26.3 ms).
template <class T, bool CLASSES>
__global__ __launch_bounds__(BLOCK) __attribute__((amdgpu_waves_per_eu(KT<T>::W == 1 ? 5 : 1)))
void k_query_blocked(SeqArgs a, BloomArgs pool, SentArgs sa, uint64_t *c1, uint64_t *c1u,
                     uint32_t round, Counters *cnt, uint32_t *hll_out) {
    __shared__ Stage sg;
    __shared__ QueryShared qs;
    __shared__ uint64_t pm[32 * 16];  // pair j of odd stride d at (d >> 1) * 16 + j
    SetSum cand = setsum_begin();
    const uint32_t k = a.k;
    const bool single = a.single != 0;
    const T *sent = (const T *)sa.table;
    const uint32_t lane = threadIdx.x & 63;
    const T mid_ones = KT<T>::ones(2 * (k - 1));
    query_begin<BLOCK>(qs, sa.prefilter + prefilter_words(sa.pf_log2), sa.pf_log2);
    for (uint32_t i = threadIdx.x; i < 32 * 16; i += BLOCK)
        pm[i] = pair_mask(0, 2 * (i >> 4) + 1, i & 15, pool.h);
    uint32_t my_probes = 0;

    RunCursor rc = run_cursor(a, a.chunk);
    for (uint64_t tile; run_next(a, rc, &tile);) {
        const uint64_t t0 = tile * TILE;
        const TileInfo ti = a.tiles[tile];
        const uint32_t lo = ti.str_lo, hi = ti.str_hi;
        if (lo == hi) {
            query_no_string(tile, c1, c1u, round);
            continue;
        }
        __syncthreads();
        stage_tile(a, tile, sg);
        __syncthreads();
        const TileSet ts = tile_set_of(a, pool, ti.set);
        const unsigned long long *blocks = (const unsigned long long *)ts.f.words;
        setsum_switch(cand, ts.set, &qs.cand_lds, &a.set_cnt[0].candidates, SETCNT_STRIDE);
        const bool one = lo + 1 == hi;
        Span sp = one ? span_of(a.strings, lo, t0) : Span{0, -1};
        const uint32_t run0 = (threadIdx.x >> 6) * (TILE / (BLOCK / 64));
        uint32_t carry_lo = 0, carry_hi = 0, carry_rev = 0, carry_pal = 0;
        uint64_t carry_w = 0;
        const Part part = tile_part(a);
        for (uint32_t it = part.lo; it < part.hi; ++it) {
            const uint32_t q = run0 + it * 64 + lane, r = q + 32;
            if (!one && (int32_t)q >= sp.ge)
                sp = span_at(a.strings, lo, hi, t0, q);
            const bool valid = (int32_t)q >= sp.gs && (int32_t)(q + k) <= sp.ge;
            // evaluated in this round: every valid position, or with classes
            // those whose k-mer is in the round's class
            bool live = valid;
            if (CLASSES && valid)
                live = in_class(class_subrange(norm(kmer_at<T>(sg, r, k), single)), ts.cls_lo,
                                ts.cls_hi);
            // the bases around: before the k-mer, its first, its last, after it
            const T u = up_from<T>(sg, r - 1), d = down_from<T>(sg, r + k + 1);
            const uint32_t pa = (uint32_t)u & 3u, v0 = ((uint32_t)u >> 2) & 3u;
            const uint32_t sb = (uint32_t)d & 3u, vk = k > 1 ? ((uint32_t)d >> 2) & 3u : v0;
            const MiddleKey m = middle_key((T)((d >> 2) & mid_ones), (T)(~(u >> 4) & mid_ones),
                                           single, ts.f.mask >> 6);
            const uint32_t kout = (uint32_t)m.g, gout = (uint32_t)(m.g >> 32);
            const bool rev_out = m.orient == 1, pal_out = m.orient == 2;
            // a valid lane loads its out-middle's block when it or the
            // position above is evaluated; the position above uses it as its
            // in-middle's (an evaluated position that is not a string start
            // has a valid predecessor in its string).  Lane 63's position
            // above is the next step's lane 0.
            const bool live_above = CLASSES ? __shfl_down(live, 1, 64) != 0 : true;
            uint64_t wo = 0;
            if (valid && (!CLASSES || live || lane == 63 || live_above)) {
                wo = __hip_atomic_load(&blocks[m.block], __ATOMIC_RELAXED,
                                       __HIP_MEMORY_SCOPE_AGENT);
                ++my_probes;
            }
            wo = rotr64(wo, m.a);
            uint32_t kin = from_below(kout, carry_lo), gin = from_below(gout, carry_hi);
            uint64_t wi = from_below(wo, carry_w);
            bool rev_in = flag_below(ballot64(rev_out), carry_rev);
            bool pal_in = flag_below(ballot64(pal_out), carry_pal);
            carry_lo = (uint32_t)__builtin_amdgcn_readlane((int)kout, 63);
            carry_hi = (uint32_t)__builtin_amdgcn_readlane((int)gout, 63);
            carry_w = lane63(wo);
            const bool first = (int32_t)q == sp.gs, last = (int32_t)(q + k) == sp.ge;
            if (live && (first || (it == part.lo && lane == 0))) {
                // the position before is another wave's or part's, or there is
                // none (its middle is then part of the sketch's hash only)
                const Strands<T> s = kmer_at<T>(sg, r, k - 1);
                const MiddleKey mi = middle_key(s.fwd, s.rc, single, ts.f.mask >> 6);
                kin = (uint32_t)mi.g;
                gin = (uint32_t)(mi.g >> 32);
                rev_in = mi.orient == 1;
                pal_in = mi.orient == 2;
                if (!first) {
                    wi = rotr64(__hip_atomic_load(&blocks[mi.block], __ATOMIC_RELAXED,
                                                  __HIP_MEMORY_SCOPE_AGENT), mi.a);
                    ++my_probes;
                }
            }
            uint32_t least = min(others_lacking<true>(pm, kout, rev_out, wo, v0, sb),
                                 others_lacking<false>(pm, kin, rev_in, wi, pa, vk));
            const bool pal = live && (pal_out || pal_in);
            if (__builtin_amdgcn_ballot_w64(pal)) {
                if (pal)
                    least = min(pal_out ? others_lacking_palindrome<true>(pm, kout, wo, v0, sb)
                                        : others_lacking<true>(pm, kout, rev_out, wo, v0, sb),
                                pal_in ? others_lacking_palindrome<false>(pm, kin, wi, pa, vk)
                                       : others_lacking<false>(pm, kin, rev_in, wi, pa, vk));
            }
            bool mark = live && (first || last || least == 0);
            if (live && !mark && ts.sent_log2 &&
                prefilter_hit(qs.pf, prefilter_bit_g(gin + gout, sa.pf_log2)))
                mark = in_sentinels(norm(kmer_at<T>(sg, r, k), single), sent + ts.sent_off,
                                    ts.sent_log2);
            const uint64_t word = ballot64(mark);
            if (lane == 0) {
                const uint64_t at = (t0 + q) >> 6;
                c1[at] = word;
                if (c1u)
                    c1u[at] = round ? c1u[at] | word : word;
                cand.v += (unsigned long long)__popcll(word);
            }
            if (a.sketch && mark)
                // the k-mer's hash: the 64-bit sum of its two middles' G values
                // (an unordered pair, the same for both orientations)
                sketch_add(qs, ((uint64_t)gin << 32 | kin) + ((uint64_t)gout << 32 | kout));
        }
    }
    query_end<BLOCK>(a, qs, cand, my_probes, cnt, hll_out);
}

// Standard layout: a lane tests its position's six neighbours level by level,
// some 10 random words a position, which is what bounds it (57-63 G words/s).
// A position inside its string is marked or not by its k-mer and the bases
// before and after it alone, and homologous tiles repeat most of those windows:
// so a workgroup takes up to 32 consecutive tiles of the first-pass order
// together and keeps a table of the windows it has decided (LDS: the position
// of one, its verdict, some bits of its hash); a window found there, compared
// base by base with the staged sequence, is not probed again.  62 x 5 Mbp,
// b = 2^30, k = 25: 3.30 G words and 41.1 ms without the table, 1.99 G and 31.4
// with 8 tiles (512 threads, 8192 windows), 1.62 G and 25.7 with 16 (1024,
// 16384), 1.50 G and 24.4 with 32; 1.44 G and 23.5 with a tile's windows looked
// up before any is probed, and 19.8 with the neighbours probed two at a time.
constexpr uint32_t QS_TILES = 32, QS_BLOCK = 1024, QS_SEEN = 16384;
constexpr uint32_t QS_NONE = ~0u;
// Neighbours probed at once: a present one ends the test, so fewer words the
// fewer at once (half the positions are candidates there: 23.5 ms with all six,
// 20.7 with three, 19.8 with two, 19.1 with one), but a longer chain of loads
// (8 x 5 Mbp 2.48, -, 2.37, 2.40).
constexpr uint32_t QS_AT_ONCE = 2;

// Inputs of fewer tiles than this take the plain form: a tile (or a part of
// one) to a workgroup of 256 threads, no table.  Query of 1024, 1536, 2048, 3072
// and 4096 tiles, 16 bits a position, plain: 8 related genomes at k = 25 0.115,
// 0.166, 0.208, 0.313 and 0.383 ms, at k = 100 0.136, 0.196, 0.261, 0.428 and
// 0.601; with the table 0.130, 0.181, 0.179, 0.263 and 0.287, and 0.170, 0.242,
// 0.266, 0.417 and 0.517.  A random genome, whose windows never repeat, pays for
// the table at every size: 0.291 and 0.318 ms at 2048 tiles, 4.14 and 4.27 at 16384.
static bool query_seen(uint64_t n_tiles) { return n_tiles >= 2048; }

struct QsTile {
    uint64_t t0;
    uint32_t lo, hi;
    Span sp;
};

// The bases r - 1 .. r + k around the k-mer at r: all but the last in w (which
// holds 2k + 2 bits), the last apart.
template <class T>
__device__ __forceinline__ T seen_window(const Stage &sg, uint32_t r, uint32_t k, uint32_t *after) {
    const T d = down_from<T>(sg, r + k + 1);
    *after = (uint32_t)d & 3u;
    return up_from<T>(sg, r - 1) & KT<T>::ones(2 * k + 2);
}

// The verdict on the k-mer at r of a staged tile, at an end of its string or
// within it; its hash to *hash when it was of the round's class.
template <uint32_t N, bool CLASSES, class T>
__device__ __forceinline__ bool standard_mark(const SeqArgs &a, const SentArgs &sa,
                                              const QueryShared &qs, const TileSet &ts,
                                              const Stage &sg, uint32_t r, bool end,
                                              uint64_t *hash, uint32_t &probes) {
    uint32_t pa, sb;
    const bool single = a.single != 0;
    const Strands<T> st = kmer_between<T>(sg, r, a.k, &pa, &sb);
    const T canon = norm(st, single);
    if (CLASSES && !in_class(class_subrange(canon), ts.cls_lo, ts.cls_hi))
        return false;
    *hash = slot_hash(canon);
    return end ||
           (ts.sent_log2 && prefilter_hit(qs.pf, prefilter_bit(*hash, sa.pf_log2)) &&
            in_sentinels(canon, (const T *)sa.table + ts.sent_off, ts.sent_log2)) ||
           any_present_standard<N>(ts.f, st, a.k, pa, sb, single, probes);
}

template <class T, bool CLASSES>
__global__ __launch_bounds__(BLOCK)
void k_query_standard(SeqArgs a, BloomArgs pool, SentArgs sa, uint64_t *c1, uint64_t *c1u,
                      uint32_t round, Counters *cnt, uint32_t *hll_out) {
    __shared__ Stage sg;
    __shared__ QueryShared qs;
    SetSum cand = setsum_begin();
    const uint32_t k = a.k;
    query_begin<BLOCK>(qs, sa.prefilter, sa.pf_log2);
    uint32_t my_probes = 0;
    const Part part = tile_part(a);
    RunCursor rc = run_cursor(a, a.chunk);
    for (uint64_t tile; run_next(a, rc, &tile);) {
        const uint64_t t0 = tile * TILE;
        const TileInfo ti = a.tiles[tile];
        const uint32_t lo = ti.str_lo, hi = ti.str_hi;
        if (lo == hi) {
            query_no_string(tile, c1, c1u, round);
            continue;
        }
        __syncthreads();
        stage_tile(a, tile, sg);
        __syncthreads();
        const TileSet ts = tile_set_of(a, pool, ti.set);
        setsum_switch(cand, ts.set, &qs.cand_lds, &a.set_cnt[0].candidates, SETCNT_STRIDE);
        const Span one = lo + 1 == hi ? span_of(a.strings, lo, t0) : Span{0, -1};
        for (uint32_t q = part.lo * BLOCK + threadIdx.x; q < part.hi * BLOCK; q += BLOCK) {
            const Span sp = lo + 1 == hi ? one : span_at(a.strings, lo, hi, t0, q);
            bool mark = false;
            uint64_t hash = 0;
            if ((int32_t)q >= sp.gs && (int32_t)(q + k) <= sp.ge)
                mark = standard_mark<6, CLASSES, T>(a, sa, qs, ts, sg, q + 32,
                                                 (int32_t)q == sp.gs || (int32_t)(q + k) == sp.ge,
                                                 &hash, my_probes);
            const uint64_t word = ballot64(mark);
            if ((threadIdx.x & 63) == 0) {
                const uint64_t i = (t0 + q) >> 6;
                c1[i] = word;
                if (c1u)
                    c1u[i] = round ? c1u[i] | word : word;
                cand.v += (unsigned long long)__popcll(word);
            }
            if (a.sketch && mark)
                sketch_add(qs, hash);
        }
    }
    query_end<BLOCK>(a, qs, cand, my_probes, cnt, hll_out);
}

// With the table.  A tile in two steps: every position looks its window up,
// those not found go to a list; then the lanes walk the list.  (Probed where
// the look-up failed, most lanes of every wave waited for a few.)
template <class T, bool CLASSES>
__global__ __launch_bounds__(QS_BLOCK)
void k_query_standard_seen(SeqArgs a, BloomArgs pool, SentArgs sa, uint64_t *c1, uint64_t *c1u,
                           uint32_t round, Counters *cnt, uint32_t *hll_out) {
    constexpr uint32_t NT = QS_BLOCK, TILES = QS_TILES, AT_END = 1u << 31;
    __shared__ Stage sg[TILES];
    __shared__ QsTile tl[TILES];
    __shared__ uint32_t tset[TILES];
    __shared__ uint32_t seen[QS_SEEN];  // hash bits << 17 | verdict << 16 | tile << 11 | position
    __shared__ QueryShared qs;
    __shared__ uint16_t todo[TILE];     // positions of the tile to decide
    __shared__ uint32_t todo_x[TILE];   // their windows: hash bits << 14 | place in seen, or AT_END
    // by the tile's parity in its batch: its candidate words, the positions in todo
    __shared__ uint64_t words[2][TILE / 64];
    __shared__ uint32_t n_todo[2];
    SetSum cand = setsum_begin();
    const uint32_t k = a.k, lane = threadIdx.x & 63;
    query_begin<NT>(qs, sa.prefilter, sa.pf_log2);
    if (threadIdx.x < 2)
        n_todo[threadIdx.x] = 0;
    uint32_t my_probes = 0, par = 0;
    // as many tiles as leave every workgroup a few batches
    const uint64_t per = a.n_tiles / (4ull * gridDim.x);
    const uint32_t most = per < 1 ? 1u : per > TILES ? TILES : (uint32_t)per;
    const Part part = tile_part(a);
    RunCursor rc = run_cursor(a, max(a.chunk, most));
    uint64_t tile;
    while (run_next(a, rc, &tile)) {
        const uint64_t j0 = rc.c + rc.gi - 1;  // the walk's entry of the first tile
        uint32_t m = 1;
        while (m < most && rc.gi + m - 1 < rc.G && j0 + m < rc.end)
            ++m;
        __syncthreads();  // the last batch is done with
        if (threadIdx.x < m) {
            const uint64_t x = rc.ordered ? (uint64_t)a.tile_order[j0 + threadIdx.x]
                                          : j0 + threadIdx.x;
            const TileInfo ti = a.tiles[x];
            QsTile t{x * TILE, ti.str_lo, ti.str_hi, Span{0, -1}};
            if (t.lo + 1 == t.hi)
                t.sp = span_of(a.strings, t.lo, t.t0);
            tl[threadIdx.x] = t;
            tset[threadIdx.x] = ti.set;
        }
        for (uint32_t i = threadIdx.x; i < QS_SEEN; i += NT)
            seen[i] = QS_NONE;
        __syncthreads();
        const uint32_t set = tset[0];  // tiles of one set (a verdict is of its filter)
        uint32_t n = 1;
        while (n < m && tset[n] == set)
            ++n;
        rc.gi += n - 1;
        for (uint32_t i = threadIdx.x; i < n * STAGE_WORDS; i += NT) {
            const uint32_t j = i / STAGE_WORDS, u = i % STAGE_WORDS;
            const int64_t gw = (int64_t)(tl[j].t0 / 32) - 1 + u;
            stage_word(sg[j], u, (gw >= 0 && (uint64_t)gw < a.seq_words) ? a.seq[gw] : 0ull);
        }
        const TileSet ts = tile_set_of(a, pool, set);
        setsum_switch(cand, set, &qs.cand_lds, &a.set_cnt[0].candidates, SETCNT_STRIDE);
        __syncthreads();
        for (uint32_t j = 0; j < n; ++j, par ^= 1) {
            const QsTile &t = tl[j];
            for (uint32_t q = part.lo * BLOCK + threadIdx.x; q < part.hi * BLOCK; q += NT) {
                const Span sp = t.lo + 1 == t.hi   ? t.sp
                                : t.lo == t.hi     ? Span{0, -1}
                                                   : span_at(a.strings, t.lo, t.hi, t.t0, q);
                bool mark = false, ask = false;
                uint32_t x = AT_END;
                if ((int32_t)q >= sp.gs && (int32_t)(q + k) <= sp.ge) {
                    ask = true;
                    if ((int32_t)q != sp.gs && (int32_t)(q + k) != sp.ge) {
                        uint32_t sb;
                        const T w = seen_window<T>(sg[j], q + 32, k, &sb);
                        x = (uint32_t)(((KT<T>::mixed(w) + sb) * 0x9E3779B97F4A7C15ull) >> 35);
                        static_assert(QS_SEEN == 1u << 14, "29 bits: 15 compared, 14 the place");
                        const uint32_t e = seen[x & (QS_SEEN - 1)];
                        if (e >> 17 == x >> 14 && e != QS_NONE) {
                            uint32_t sb2;
                            if (seen_window<T>(sg[e >> 11 & 31u], (e & (TILE - 1)) + 32, k, &sb2) == w &&
                                sb2 == sb) {
                                ask = false;
                                mark = (e >> 16) & 1u;
                            }
                        }
                    }
                }
                const uint64_t word = ballot64(mark), asks = ballot64(ask);
                uint32_t at = 0;
                if (lane == 0) {
                    words[par][q >> 6] = word;
                    if (asks)
                        at = atomicAdd(&n_todo[par], (uint32_t)__popcll(asks));
                }
                at = (uint32_t)__builtin_amdgcn_readfirstlane((int)at) +
                     __builtin_amdgcn_mbcnt_hi((uint32_t)(asks >> 32),
                                               __builtin_amdgcn_mbcnt_lo((uint32_t)asks, 0));
                if (ask) {
                    todo[at] = (uint16_t)q;
                    todo_x[at] = x;
                }
            }
            __syncthreads();  // the list and the words are whole
            const uint32_t n_ask = n_todo[par];
            for (uint32_t i = threadIdx.x; i < n_ask; i += NT) {
                const uint32_t q = todo[i], x = todo_x[i];
                uint64_t hash = 0;
                const bool mark = standard_mark<QS_AT_ONCE, CLASSES, T>(a, sa, qs, ts, sg[j], q + 32,
                                                            x == AT_END, &hash, my_probes);
                if (x != AT_END)
                    seen[x & (QS_SEEN - 1)] = x >> 14 << 17 | (mark ? 1u : 0u) << 16 | j << 11 | q;
                if (mark) {
                    atomicOr((uint32_t *)words[par] + (q >> 5), 1u << (q & 31u));
                    if (a.sketch)  // (a found window's k-mer is in it already)
                        sketch_add(qs, hash);
                }
            }
            __syncthreads();  // (the next tile's step one reads the verdicts)
            if (threadIdx.x >= part.lo * (BLOCK / 64) && threadIdx.x < part.hi * (BLOCK / 64)) {
                const uint64_t i = t.t0 / 64 + threadIdx.x, word = words[par][threadIdx.x];
                c1[i] = word;
                if (c1u)
                    c1u[i] = round ? c1u[i] | word : word;
                cand.v += (unsigned long long)__popcll(word);
            }
            if (threadIdx.x == 0)
                n_todo[par] = 0;
        }
    }
    query_end<NT>(a, qs, cand, my_probes, cnt, hll_out);
}

hipError_t launch_query(int W, const SeqArgs &a, const BloomArgs &pool, const SentArgs &sa,
                        uint64_t *c1, uint64_t *c1u, uint32_t round, Counters *cnt,
                        uint32_t *hll, uint32_t grid, hipStream_t s) {
    if (a.n_tiles == 0)
        return hipSuccess;
    return by_width(W, [&](auto tag) {
        using T = decltype(tag);
        const bool seen = !pool.blocked && query_seen(a.n_tiles);
        auto *fn = pool.blocked ? (a.classes ? k_query_blocked<T, true> : k_query_blocked<T, false>)
                   : seen ? (a.classes ? k_query_standard_seen<T, true>
                                       : k_query_standard_seen<T, false>)
                          : (a.classes ? k_query_standard<T, true> : k_query_standard<T, false>);
        hipLaunchKernelGGL(fn, dim3(grid), dim3(seen ? QS_BLOCK : BLOCK), 0, s, a, pool, sa, c1, c1u,
                           round, cnt, hll);
        return hipGetLastError();
    });
}

// ------------------------------------------------- class census (rounds)

// Per set, CLASS_Q counters: every (k+1)-mer adds one to the subrange of
// each distinct class subrange among its two normalised k-mers (Multiple
// Rounds section: counters estimate the (k+1)-mers that touch each class).
// A workgroup counts in LDS and adds its counts to the set's counters when
// its tiles move to another set, and at the end.
template <class T>
__global__ __launch_bounds__(BLOCK) void k_census(SeqArgs a, unsigned long long *counters) {
    __shared__ Stage sg;
    __shared__ uint32_t hist[CLASS_Q];
    const uint32_t L = a.k + 1;
    const bool single = a.single != 0;
    for (uint32_t i = threadIdx.x; i < CLASS_Q; i += BLOCK)
        hist[i] = 0;
    uint32_t cur_set = ~0u;
    auto flush = [&]() {
        __syncthreads();
        if (cur_set != ~0u)
            for (uint32_t i = threadIdx.x; i < CLASS_Q; i += BLOCK) {
                const uint32_t v = hist[i];
                if (v)
                    atomicAdd(&counters[(uint64_t)cur_set * CLASS_Q + i], (unsigned long long)v);
                hist[i] = 0;
            }
        __syncthreads();
    };
    RunCursor rc = run_cursor(a, a.chunk);
    for (uint64_t tile; run_next(a, rc, &tile);) {
        const uint64_t t0 = tile * TILE;
        const TileInfo ti = a.tiles[tile];
        const uint32_t lo = ti.str_lo, hi = ti.str_hi;
        if (lo == hi)
            continue;
        if (ti.set != cur_set) {
            flush();
            cur_set = ti.set;
        }
        __syncthreads();
        stage_tile(a, tile, sg);
        __syncthreads();
        const bool one = lo + 1 == hi;
        Span sp = one ? span_of(a.strings, lo, t0) : Span{0, -1};
        for (uint32_t it = 0; it < TILE / BLOCK; ++it) {
            const uint32_t q = it * BLOCK + threadIdx.x;
            if (!one && (int32_t)q >= sp.ge)
                sp = span_at(a.strings, lo, hi, t0, q);
            if ((int32_t)q < sp.gs || (int32_t)(q + L) > sp.ge)
                continue;
            const uint32_t x = class_subrange(norm(kmer_at<T>(sg, q + 32, a.k), single));
            const uint32_t y = class_subrange(norm(kmer_at<T>(sg, q + 33, a.k), single));
            atomicAdd(&hist[x], 1u);
            if (y != x)
                atomicAdd(&hist[y], 1u);
        }
    }
    flush();
}

hipError_t launch_census(int W, const SeqArgs &a, unsigned long long *counters, uint32_t grid,
                         hipStream_t s) {
    hipError_t e = launch_zero(counters, (uint64_t)a.n_sets * CLASS_Q * 8, s);
    if (e != hipSuccess || a.n_tiles == 0)
        return e;
    return by_width(W, [&](auto tag) {
        hipLaunchKernelGGL(k_census<decltype(tag)>, dim3(grid), dim3(BLOCK), 0, s, a, counters);
        return hipGetLastError();
    });
}

// Greedy partition of the Multiple Rounds section on the device, one thread
// per set (the host's class_partition, for runs without host waits): class c
// takes the longest run of consecutive subranges, at least one while any
// remain, whose counter sum times the number of classes stays within the
// total; the last class takes every remaining subrange.
__global__ void k_partition(const unsigned long long *census, uint32_t n_sets, uint32_t rounds,
                            uint32_t *bounds) {
    const uint32_t set = blockIdx.x * blockDim.x + threadIdx.x;
    if (set >= n_sets)
        return;
    const unsigned long long *e = census + (uint64_t)set * CLASS_Q;
    uint32_t *bound = bounds + (uint64_t)set * (rounds + 1);
    unsigned __int128 total = 0;
    for (uint32_t i = 0; i < CLASS_Q; ++i)
        total += e[i];
    uint32_t next = 0;
    for (uint32_t c = 0; c < rounds; ++c) {
        bound[c] = next;
        if (c + 1 == rounds) {
            next = CLASS_Q;
            continue;
        }
        unsigned __int128 sum = 0;
        for (uint32_t taken = 0; next < CLASS_Q; ++taken, ++next) {
            if (taken > 0 && (sum + e[next]) * rounds > total)
                break;
            sum += e[next];
        }
    }
    bound[rounds] = CLASS_Q;
}

__global__ void k_set_round(SetDesc *sets, const uint32_t *bounds, uint32_t n_sets,
                            uint32_t rounds, uint32_t round) {
    const uint32_t set = blockIdx.x * blockDim.x + threadIdx.x;
    if (set >= n_sets)
        return;
    sets[set].cls_lo = bounds[(uint64_t)set * (rounds + 1) + round];
    sets[set].cls_hi = bounds[(uint64_t)set * (rounds + 1) + round + 1];
}

hipError_t launch_partition(const unsigned long long *census, uint32_t n_sets, uint32_t rounds,
                            uint32_t *bounds, hipStream_t s) {
    if (n_sets == 0)
        return hipSuccess;
    hipLaunchKernelGGL(k_partition, dim3((n_sets + 63) / 64), dim3(64), 0, s, census, n_sets,
                       rounds, bounds);
    return hipGetLastError();
}

hipError_t launch_set_round(SetDesc *sets, const uint32_t *bounds, uint32_t n_sets,
                            uint32_t rounds, uint32_t round, hipStream_t s) {
    if (n_sets == 0)
        return hipSuccess;
    hipLaunchKernelGGL(k_set_round, dim3((n_sets + 63) / 64), dim3(64), 0, s, sets, bounds,
                       n_sets, rounds, round);
    return hipGetLastError();
}

hipError_t pass1_occupancy(KernelId which, int W, bool blocked, bool fill_dedup, uint64_t n_tiles,
                           int *blocks) {
    return by_width(W, [&](auto tag) {
        using T = decltype(tag);
        const bool seen = !blocked && query_seen(n_tiles);
        const void *fn =
            which == K_FILL
                ? (blocked ? (const void *)k_fill<T, true> : (const void *)k_fill<T, false>)
            : blocked ? (const void *)k_query_blocked<T, false>
            : seen    ? (const void *)k_query_standard_seen<T, false>
                      : (const void *)k_query_standard<T, false>;
        const size_t dyn = which == K_FILL && blocked && fill_dedup
                               ? FILL_DD * sizeof(unsigned long long) : 0;
        return hipOccupancyMaxActiveBlocksPerMultiprocessor(
            blocks, fn, which == K_QUERY && seen ? QS_BLOCK : BLOCK, dyn);
    });
}

// ----------------------------------------------------- filter popcount per set

// Workgroup b counts 16-byte pieces [b*chunk, (b+1)*chunk) of the pool (sets'
// filters start and end on whole pieces); a thread adds its running count to a
// set's counter whenever its pieces cross into another set (set regions are
// consecutive in the pool).  At the end the threads whose last set is the last
// set of the chunk add in LDS first, so a chunk inside one set costs one
// device atomic.  A chunk is at least 16 KiB: atomics on one counter queue up
// (with 1 KiB chunks a 2 MiB filter took 28 us), and at most a 2048th of the
// pool (1.4 GB over 128 sets: 1.14 ms by words, 0.32 by these pieces).
__global__ __launch_bounds__(BLOCK) void k_popcount(const uint4 *pool, uint64_t n, uint64_t chunk,
                                                    const uint64_t *starts, uint32_t n_sets,
                                                    SetCounters *sc) {
    __shared__ unsigned long long sum;
    const uint64_t b0 = blockIdx.x * chunk;
    const uint64_t b1 = b0 + chunk < n ? b0 + chunk : n;
    // last set that starts at or before piece i
    auto set_of = [&](uint64_t i) {
        uint32_t lo = 0, hi = n_sets;
        while (hi - lo > 1) {
            const uint32_t mid = (lo + hi) >> 1;
            if (starts[mid] <= 4 * i)
                lo = mid;
            else
                hi = mid;
        }
        return lo;
    };
    if (threadIdx.x == 0)
        sum = 0;
    const uint32_t first_set = set_of(b0), last_set = set_of(b1 - 1);
    uint32_t set = first_set;
    uint64_t end = starts[set + 1] / 4;
    uint32_t c = 0;  // (a thread's pieces of one chunk hold well under 2^32 bits)
    constexpr uint32_t U = 4;
    for (uint64_t i0 = b0 + threadIdx.x; i0 < b1; i0 += U * BLOCK) {
        uint4 v[U];
#pragma unroll
        for (uint32_t q = 0; q < U; ++q)
            v[q] = i0 + q * BLOCK < b1 ? pool[i0 + q * BLOCK] : make_uint4(0, 0, 0, 0);
#pragma unroll
        for (uint32_t q = 0; q < U; ++q) {
            const uint64_t i = i0 + q * BLOCK;
            if (i >= end && i < b1) {
                if (c)
                    atomicAdd(&sc[set].bloom_popcount, (unsigned long long)c);
                c = 0;
                set = set_of(i);
                end = starts[set + 1] / 4;
            }
            c += __popc(v[q].x) + __popc(v[q].y) + __popc(v[q].z) + __popc(v[q].w);
        }
    }
    __syncthreads();
    if (c) {
        if (set == last_set)
            atomicAdd(&sum, (unsigned long long)c);
        else
            atomicAdd(&sc[set].bloom_popcount, (unsigned long long)c);
    }
    __syncthreads();
    if (threadIdx.x == 0 && sum)
        atomicAdd(&sc[last_set].bloom_popcount, sum);
}

hipError_t launch_popcount(const uint32_t *pool, uint64_t n_words, const uint64_t *bloom_starts,
                           uint32_t n_sets, SetCounters *set_cnt, hipStream_t s) {
    if (n_words == 0 || n_sets == 0)
        return hipSuccess;
    const uint64_t n = n_words / 4;
    const uint32_t grid = (uint32_t)std::min<uint64_t>(2048, (n + 1023) / 1024);
    const uint64_t chunk = (n + grid - 1) / grid;
    hipLaunchKernelGGL(k_popcount, dim3((uint32_t)((n + chunk - 1) / chunk)), dim3(BLOCK), 0, s,
                       (const uint4 *)pool, n, chunk, bloom_starts, n_sets, set_cnt);
    return hipGetLastError();
}

}  // namespace tp
