// Second pass of Algorithm 2 (Filter-Junctions with E = exact set) over the
// first-pass candidates C1, for gfx950.
//
// The exact set is kept per vertex rather than per edge: an open-addressing
// table keyed by the normalised candidate k-mer v holds an 8-bit mask, bits
// 0-3 the bases c with c.v an edge (in) and bits 4-7 the bases c with v.c an
// edge (out), both for v in normalised orientation.  Every occurrence of an
// edge next to a candidate vertex lies next to a candidate position, because
// a candidate set never splits the positions of one normalised k-mer
// (Single Round section), so recording the predecessor and successor edge of
// every candidate position yields exactly the in/out edge sets that loop 2 of
// Algorithm 1 counts.  This stores one entry per distinct candidate k-mer
// instead of up to 8 per junction (Theoretical Analysis section).
//
//   k_record   loop 1: insert-or-find the normalised k-mer (one atomicCAS on
//              its slot word), then atomicOr its edge bits (skipped when the
//              word read already has them).
//   k_decide   loop 2: a candidate stays a junction when its k-mer is a
//              sentinel or has more than one in- or out-edge; one wave
//              ballot per 64 positions writes the J bitmap.
#include <type_traits>

#include "device.hpp"

namespace tp {

// The second pass walks up to P2_TILES tiles of one set at a time.  Their
// candidates are listed first (their positions), and the lanes walk
// the list, so that every lane holds a candidate: a 16-bit-a-position filter
// leaves some 8% of them, spread over every wave, and a round the same of its
// class.  Several tiles at once, because a tile's own chain of dependent steps
// (the claim of it, its record, its words, the set's flag) takes as long as
// its lookups.  Walked by position and tile by tile, then listed tile by tile,
// then in batches of four: 128 sets of 654 Mbp at k = 31 record 5.5, 5.1 and
// 2.2 ms, decision 3.9, 3.8 and 1.4; 1 Gbp at k = 63 record 8.9, 6.1 and 2.5,
// decision 6.6, 5.7 and 1.9; four rounds of 80 Mbp at k = 25 record 2.0, 2.0
// and 0.7, decision 2.4, 2.3 and 0.9.
constexpr uint32_t P2_TILES = 4;
// The batch's tiles take turns in the list, P2_RUN positions each: homologous
// tiles (a slab walk's batch) then look a k-mer up at about the same time and hit
// its line.  8 related genomes of 5 Mbp, k = 25, every position a candidate:
// decision 0.68 ms listed tile by tile, 0.52, 0.41 and 0.41 with runs of 512, 128
// and 32; 62 x 5 Mbp with 2.5 bits a position 1.43, 1.42, 1.41 and 1.48 (a wave's
// lanes in four tiles' stages).
constexpr uint32_t P2_RUN = 128;

struct P2Tile {
    uint64_t t0;
    uint32_t lo, hi;  // its strings
    Span sp;          // its string when it has just one
};

struct P2Batch {
    Stage sg[P2_TILES];
    P2Tile tile[P2_TILES];
    uint32_t set[P2_TILES];
    uint64_t w[P2_TILES * TILE / 64];   // candidate words
    uint16_t at[P2_TILES * TILE];       // candidates: tile << 11 | position
    uint32_t wsum[16];                  // (up to 1024 threads)
    uint32_t skip;
};
static_assert(TILE == 1u << 11, "candidate positions");

// Whether a set's table overflowed in this attempt (thread 0 only): the
// device-coherent flag is read again when the set changes and every 8th
// batch, so the workgroups do not all read one counter line per batch.  A late
// reading only delays the skip; the attempt is redone either way.
struct OverflowFlag {
    uint32_t set = ~0u, age = 0, value = 0;
};

__device__ __forceinline__ uint32_t overflow_seen(const SeqArgs &a, uint32_t set, OverflowFlag &f) {
    if (set != f.set || (++f.age & 7) == 0) {
        f.value = (uint32_t)__hip_atomic_load(&a.set_cnt[set].overflow, __ATOMIC_RELAXED,
                                              __HIP_MEMORY_SCOPE_AGENT);
        f.set = set;
        f.age = 0;
    }
    return f.value;
}

// The next batch of the walk (at most `most` tiles of one chunk and one set),
// staged, and its candidates listed: false at the walk's end, else its tiles
// in *n, its candidates in *total and its set.  A set whose table overflowed
// in this attempt is redone with a larger table, so its work is skipped (skip:
// other workgroups may set the flag at any time, so one thread reads it and
// the whole workgroup takes that one reading).  Whole workgroup; ends
// synchronised.
template <uint32_t NT>
__device__ __forceinline__ bool next_batch(const SeqArgs &a, RunCursor &rc, uint32_t most,
                                           const uint64_t *c1, P2Batch &b, OverflowFlag &flag,
                                           uint32_t *n, uint32_t *total, uint32_t *set) {
    uint64_t first;
    if (!run_next(a, rc, &first))
        return false;
    const uint64_t j0 = rc.c + rc.gi - 1;  // the walk's entry of the first tile
    uint32_t m = 1;
    while (m < most && rc.gi + m - 1 < rc.G && j0 + m < rc.end)
        ++m;
    __syncthreads();  // the last batch is done with
    if (threadIdx.x < m) {
        const uint64_t tile = rc.ordered ? (uint64_t)a.tile_order[j0 + threadIdx.x] : j0 + threadIdx.x;
        const TileInfo ti = a.tiles[tile];
        P2Tile x;
        x.t0 = tile * TILE;
        x.lo = ti.str_lo;
        x.hi = ti.str_hi;
        x.sp = x.lo + 1 == x.hi ? span_of(a.strings, x.lo, x.t0) : Span{0, -1};
        b.tile[threadIdx.x] = x;
        b.set[threadIdx.x] = ti.set;
    }
    __syncthreads();
    *set = b.set[0];
    uint32_t take = 1;
    while (take < m && b.set[take] == *set)
        ++take;
    rc.gi += take - 1;
    *n = take;
    for (uint32_t i = threadIdx.x; i < take * STAGE_WORDS; i += NT) {
        const uint32_t j = i / STAGE_WORDS, u = i % STAGE_WORDS;
        const int64_t gw = (int64_t)(b.tile[j].t0 / 32) - 1 + u;
        stage_word(b.sg[j], u, (gw >= 0 && (uint64_t)gw < a.seq_words) ? a.seq[gw] : 0ull);
    }
    for (uint32_t i = threadIdx.x; i < P2_TILES * TILE / 64; i += NT) {
        const uint32_t j = i / (TILE / 64);
        b.w[i] = j < take ? c1[b.tile[j].t0 / 64 + i % (TILE / 64)] : 0ull;
    }
    if (threadIdx.x == 0)
        b.skip = overflow_seen(a, *set, flag);
    __syncthreads();
    // a thread lists PER positions
    constexpr uint32_t PER = P2_TILES * TILE / NT;
    static_assert(PER == 8 || PER == 16 || PER == 32, "a piece of one 32-bit word");
    static_assert(P2_RUN % PER == 0 && TILE % P2_RUN == 0, "whole pieces");
    const uint32_t lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    constexpr uint32_t RUN = P2_RUN / PER;
    const uint32_t jt = threadIdx.x / RUN % P2_TILES,
                   p0 = (threadIdx.x / RUN / P2_TILES * RUN + threadIdx.x % RUN) * PER;
    uint32_t bits = ((const uint32_t *)b.w)[jt * (TILE / 32) + p0 / 32];
    if (PER < 32)
        bits = bits >> (p0 & 31u) & ((1u << (PER & 31u)) - 1);
    const uint32_t c = (uint32_t)__popc(bits);
    uint32_t x = c;
#pragma unroll
    for (uint32_t d = 1; d < 64; d <<= 1) {
        const uint32_t y = __shfl_up(x, d, 64);
        x += lane >= d ? y : 0;
    }
    if (lane == 63)
        b.wsum[wave] = x;
    __syncthreads();
    uint32_t at = x - c, sum = 0;
#pragma unroll
    for (uint32_t q = 0; q < NT / 64; ++q) {
        at += q < wave ? b.wsum[q] : 0;
        sum += b.wsum[q];
    }
    for (; bits; bits &= bits - 1)
        b.at[at++] = (uint16_t)(jt * TILE + p0 + (uint32_t)__builtin_ctz(bits));
    *total = sum;
    __syncthreads();
    return true;
}

// Tiles per batch of a launch: enough batches to go round.
__host__ __device__ inline uint32_t batch_tiles(uint64_t n_tiles, uint32_t grid) {
    const uint64_t per = n_tiles / (4ull * grid);
    return per < 1 ? 1u : per > P2_TILES ? P2_TILES : (uint32_t)per;
}

// The walk of a second-pass kernel: chunks of whole batches.
__device__ __forceinline__ RunCursor batch_run(const SeqArgs &a, bool slabs, uint32_t chunk) {
    return slabs ? run_cursor(a, chunk) : linear_run(a, chunk);
}

// The table of a tile's set: the pools shifted to its region.
__device__ __forceinline__ TableArgs table_of(const SeqArgs &a, const TableArgs &pool,
                                              uint32_t set) {
    const SetDesc &d = a.sets[set];
    TableArgs t = pool;
    t.keys = pool.keys + d.table_off;
    t.cap_m = d.table_m;
    t.cap_e = d.table_e;
    t.lomask = (1ull << d.table_e) - 1;
    return t;
}

// A lookup starts at the key's home slot (home_slot of its hash) and goes on
// to the slots after it, a pair of slots at a time.  Two table modes, fixed
// per run (the kernels are instantiated for each):
//   P2    capacity 2^e: the home slot is the low e hash bits and probes wrap
//         at the capacity (a mask on the path from key to address);
//   any   capacity m << e (m < 2^32): m blocks of 2^e slots.  The home
//         slot's block is the high word of m * (top 32 hash bits), its slot
//         in the block the low e hash bits, uniform over [0, m << e); probes
//         wrap within the block, so a lookup never leaves its home block
//         (which lets the record insert block by block, see k_rbin_apply).
//
// Home slots are even, so a lookup can read the pair of slots it starts in
// with one 16-byte load (capacities and set regions are multiples of 64
// slots, so pairs never straddle them).
template <bool P2>
__device__ __forceinline__ uint64_t home_slot(const TableArgs &t, uint64_t h) {
    if (P2)
        return h & t.lomask & ~1ull;
    const uint64_t top = __umulhi((uint32_t)(h >> 32), t.cap_m);
    return ((top << t.cap_e) | (h & t.lomask)) & ~1ull;
}

template <bool P2, class T>
__device__ __forceinline__ uint64_t first_slot(const TableArgs &t, T key) {
    return home_slot<P2>(t, slot_hash(key));
}

// The next pair of slots after the pair starting at s (s even).
template <bool P2>
__device__ __forceinline__ uint64_t next_pair(const TableArgs &t, uint64_t s) {
    return P2 ? (s + 2) & t.lomask : (s & ~t.lomask) | ((s + 2) & t.lomask);
}

typedef HIP_vector_type<unsigned long long, 2> u64x2;

// Words of slots s and s + 1 (s even), one 16-byte load.  The record reads
// pairs too, with plain loads: a word read stale can only be empty where a
// key now is (slots go from empty to a key, never back; mask bits are only
// set), which costs a failed claim or an extra OR, never a wrong answer.
__device__ __forceinline__ u64x2 load_pair(const TableArgs &t, uint64_t s) {
    return *(const u64x2 *)(t.keys + s);
}

// Slot words.  Packed (k <= 27): key << 8 | edge bits.  Reference (k >= 28):
// the key does not fit beside its edge bits, so the word holds instead where
// the sequence reads it, tag | p << 8 | edge bits, p the global base index of
// the occurrence that claimed the slot and tag the bits above it (ref_tag).
// A word whose tag matches is compared with the packed sequence at p, so a
// lookup is as exact as one that stores the key.  One 64-bit word per slot
// whatever k: a claim is one compare-and-swap, where storing the key took an
// atomic per key word and one to publish it (and those atomics, at the
// device's ~27 G/s, were the whole record), and the table is cleared, probed
// and cached at a half to a quarter of the bytes.  62 x 5 Mbp, b = 2^30: 73M
// keys at k = 63, record 16.3 -> 6.0 ms and decision 6.6 -> 3.9 (5.2 and 2.8 with
// the listed walk); 135M keys at k = 100, 27.3 -> 8.5 and 10.6 -> 6.2 (8.1 and
// 3.7).  The compare reads two to
// five words of the sequence, mostly lines that neighbouring positions read
// too (consecutive k-mers were claimed by consecutive positions).

// The tag: hash bits above the position and the edge bits.  Any-size tables
// take the block from the high hash word, so there the low word's top bits
// come first (they are free of the home slot's).
template <bool P2>
__device__ __forceinline__ uint64_t ref_tag(const TableArgs &t, uint64_t h) {
    const uint64_t x = P2 ? h : (h << 32 | h >> 32);
    return x >> t.ref_shift << t.ref_shift;
}

// Whether the sequence reads the k-mer st, on either strand, at the position
// that slot word names: x ^ ones is the value of the reverse complement of
// the window x, and it is st.rc when x is st as read, st.fwd when x is its
// reverse complement.  (The words read past the k-mer lie within the input's
// last 64 bytes at most.)
template <class T>
__device__ __forceinline__ bool ref_is(const SeqArgs &a, const TableArgs &t,
                                       unsigned long long word, const Strands<T> &st) {
    const uint64_t p = (word & ((1ull << t.ref_shift) - 1)) >> 8;
    const T z = ~KT<T>::win((const uint32_t *)a.seq + (p >> 4), (uint32_t)(p & 15)) &
                KT<T>::ones(2 * a.k);
    return z == st.rc || (!a.single && z == st.fwd);
}

// Insert-or-find by slot pairs, starting with the pair pr of slots s, s + 1
// (s even): claim an empty slot for own (the key's slot word with the edge
// bits m) by atomicCAS, or OR the edge bits into the key's slot.  same(w):
// whether the slot word w is the key's.  1 when this call claimed a new slot,
// 0 when the key was present, -1 on overflow.
template <bool P2, class Same>
__device__ __forceinline__ int insert_pair(const TableArgs &t, unsigned long long own, uint32_t m,
                                           uint64_t s, u64x2 pr, Same &&same, uint32_t &probes) {
    for (uint32_t i = 0; i < MAX_PROBE / 2; ++i) {
        if (i)
            pr = load_pair(t, s);
        ++probes;
#pragma unroll
        for (uint32_t half = 0; half < 2; ++half) {
            const uint64_t slot = s + half;
            unsigned long long cur = half ? pr.y : pr.x;
            if (cur == EMPTY_KEY) {
                cur = atomicCAS(&t.keys[slot], EMPTY_KEY, own);
                if (cur == EMPTY_KEY)
                    return 1;
            }
            if (same(cur)) {
                if ((cur & m) != m)
                    __hip_atomic_fetch_or(&t.keys[slot], (unsigned long long)m, __ATOMIC_RELAXED,
                                          __HIP_MEMORY_SCOPE_AGENT);
                return 0;
            }
        }
        s = next_pair<P2>(t, s);
    }
    return -1;
}

// Edge bits of the key's slot (same(w) as above), or -1 when absent; pr
// holds the words of slots s and s + 1 (s even).
template <bool P2, class Same>
__device__ __forceinline__ int find_pair(const TableArgs &t, uint64_t s, u64x2 pr, Same &&same,
                                         uint32_t &probes) {
    for (uint32_t i = 0; i < MAX_PROBE / 2; ++i) {
        if (i)
            pr = load_pair(t, s);
        ++probes;
#pragma unroll
        for (uint32_t half = 0; half < 2; ++half) {
            const unsigned long long w = half ? pr.y : pr.x;
            if (w == EMPTY_KEY)
                return -1;
            if (same(w))
                return (int)(w & 0xFFu);
        }
        s = next_pair<P2>(t, s);
    }
    return -1;
}

// Host-side dispatch on the k-mer width, the table mode and the slot words:
// f(value of the k-mer type, power-of-two table, reference words); packed
// words are one-word k-mers'.
template <class F> hipError_t by_table(int W, const TableArgs &t, F &&f) {
    return by_width(W, [&](auto tag) {
        if constexpr (KT<decltype(tag)>::W == 1) {
            if (t.packed)
                return t.pow2 ? f(tag, std::true_type{}, std::false_type{})
                              : f(tag, std::false_type{}, std::false_type{});
        }
        return t.pow2 ? f(tag, std::true_type{}, std::true_type{})
                      : f(tag, std::false_type{}, std::true_type{});
    });
}

// ------------------------------------------------------------- record (a3)

// The normalised k-mer of position q of a staged tile, in the string sp, and
// in m its edge bits: the predecessor's base as an in-bit and the successor's
// as an out-bit, for the orientation in which the k-mer is normalised (both
// orientations for a palindrome).
template <class T>
__device__ __forceinline__ T record_key(const Stage &sg, uint32_t q, uint32_t k, const Span &sp,
                                        bool single, uint32_t &m, Strands<T> &st) {
    uint32_t pa, sb;
    st = kmer_between<T>(sg, q + 32, k, &pa, &sb);
    const uint32_t has_pred = (int32_t)q > sp.gs, has_succ = (int32_t)(q + k) < sp.ge;
    m = 0;
    T canon = st.fwd;
    if (single || st.fwd <= st.rc) {
        // the k-mer as read is normalised: pred.v enters, v.succ leaves
        m = has_pred << pa | has_succ << (4 + sb);
    }
    if (!single && st.rc <= st.fwd) {
        // its reverse complement is normalised: comp(succ) enters, comp(pred)
        // leaves
        m |= has_succ << (3 - sb) | has_pred << (7 - pa);
        canon = st.rc;
    }
    return canon;
}

// The span that position q of a tile lies in.
__device__ __forceinline__ Span record_span(const SeqArgs &a, const P2Tile &tl, uint32_t q) {
    return tl.lo + 1 == tl.hi ? tl.sp : span_at(a.strings, tl.lo, tl.hi, tl.t0, q);
}

template <class T, bool P2, bool REF>
__global__ __launch_bounds__(BLOCK) void k_record(SeqArgs a, const uint64_t *c1, TableArgs pool,
                                                  Counters *cnt) {
    __shared__ P2Batch b;
    __shared__ unsigned long long block_probes, keys_lds;
    OverflowFlag flag;
    SetSum keys = setsum_begin();
    const uint32_t k = a.k;
    const bool single = a.single != 0;
    if (threadIdx.x == 0)
        block_probes = 0;
    uint32_t my_probes = 0;
    // memory order spreads homologous tiles' claims out in time; runs of them
    // on one workgroup keep their slots hot without the concurrent claims of
    // the plain first-pass order
    const uint32_t order = a.pass2_slabs, most = batch_tiles(a.n_tiles, gridDim.x);
    const uint32_t chunk = max(a.chunk, (order & 4) ? RECORD_RUN : most);
    RunCursor rc = batch_run(a, (order & 5) != 0, chunk);
    uint32_t n, total, set;
    while (next_batch<BLOCK>(a, rc, most, c1, b, flag, &n, &total, &set)) {
        if (b.skip)
            continue;
        const TableArgs t = table_of(a, pool, set);
        setsum_switch(keys, set, &keys_lds, &a.set_cnt[0].table_keys, SETCNT_STRIDE);
        bool overflow = false;
        for (uint32_t i = threadIdx.x; i < total; i += BLOCK) {
            const uint32_t q = b.at[i] & (TILE - 1);
            const P2Tile &tl = b.tile[b.at[i] / TILE];
            const Stage &sg = b.sg[b.at[i] / TILE];
            const Span sp = record_span(a, tl, q);
            if ((int32_t)q < sp.gs)
                continue;  // not a k-mer start: never marked by the first pass
            uint32_t m;
            Strands<T> st;
            const T canon = record_key<T>(sg, q, k, sp, single, m, st);
            const uint64_t hash = slot_hash(canon);
            const uint64_t slot = home_slot<P2>(t, hash);
            const u64x2 pr = load_pair(t, slot);
            int rc;
            if constexpr (REF) {
                const unsigned long long own = ref_tag<P2>(t, hash) | (tl.t0 + q) << 8 | m;
                rc = insert_pair<P2>(t, own, m, slot, pr, [&](unsigned long long x) {
                    return (x ^ own) >> t.ref_shift == 0 && ref_is(a, t, x, st);
                }, my_probes);
            } else {
                const uint64_t key = (uint64_t)canon;
                rc = insert_pair<P2>(t, key << 8 | m, m, slot, pr, [&](unsigned long long x) {
                    return x >> 8 == key;
                }, my_probes);
            }
            if (rc > 0)
                ++keys.v;
            else if (rc < 0)
                overflow = true;
        }
        if (overflow)
            atomicExch(&a.set_cnt[set].overflow, 1ull);
    }
    setsum_flush(keys, &keys_lds, &a.set_cnt[0].table_keys, SETCNT_STRIDE);
    if (my_probes)
        atomicAdd(&block_probes, (unsigned long long)my_probes);
    __syncthreads();
    if (threadIdx.x == 0 && block_probes)
        atomicAdd(&cnt->table_probes, block_probes);
}

hipError_t launch_record(int W, const SeqArgs &a, const uint64_t *c1, const TableArgs &pool,
                         Counters *cnt, uint32_t grid, hipStream_t s) {
    if (a.n_tiles == 0)
        return hipSuccess;
    return by_table(W, pool, [&](auto tag, auto p2, auto ref) {
        hipLaunchKernelGGL((k_record<decltype(tag), decltype(p2)::value, decltype(ref)::value>),
                           dim3(grid), dim3(BLOCK), 0, s, a, c1, pool, cnt);
        return hipGetLastError();
    });
}

// ------------------------------------------------------ binned record (a3)
//
// The table k_record builds, built block by block instead of by random
// atomics.  A lookup never leaves the block of its home slot (2^e slots,
// e <= TABLE_BLOCK_LOG2), so blocks are independent: a pass takes the blocks
// [r_lo, r_hi); every candidate whose home block is among them becomes an
// item, the slot word it contributes (key << 8 | edge bits, packed slots);
// the items are partitioned by block in one or two streaming steps, as the
// binned fill's are (bin_append: buckets of up to RBIN_SUB blocks, then
// blocks); and each block is built in LDS from empty and written out whole.
// Same keys and edge bits as k_record (slots within a block may differ: they
// follow the order of insertion), no table clear and no random access.  Every
// pass walks the candidates again; the passes are as many as the scratch
// needs.
//
//   k_rbin_items    the candidates listed (next_batch), their items collected
//                   in LDS until they fill a batch, the batch appended to the
//                   buckets
//   k_rbin_split    buckets of several blocks: batches of a bucket's items
//                   appended to its blocks
//   k_rbin_apply    per block: built in LDS, written out; new keys counted
//   k_rbin_spill    the items that found no room, after the last pass: into
//                   the finished table, as k_record inserts them
//
// Bound by the candidates' walk and the items' memory traffic (8 bytes, written
// and read once per level): 1.6 Gbp, 450M candidates, a 4 GiB table, items 4.2
// ms, split 1.8, apply 3.0, against 17.1 of k_record, whose random atomics move
// a line in and out each, and 0.9 of the table's clear; 62 x 5 Mbp 1.3, 0.5 and
// 0.6 against 3.2.  Items by workgroups of 1024 threads, one to a CU, 6.0 ms,
// two (64 registers) 4.8, of 256, three to a CU, 7.3.  Apply with every item's
// probes on their own 3.9 ms (of the smaller table), by lanes at their own pace
// 3.6.
//
// A bucket's and a block's room come from the candidate count, as a hash
// spreads keys evenly and a key comes up about once per genome; a k-mer of
// many thousand copies fills its block's, and the rest of its items spill.

// Home block of a packed slot word (its key is word >> 8).
template <bool P2>
__device__ __forceinline__ uint64_t rbin_block(const TableArgs &t, uint64_t item) {
    return first_slot<P2>(t, item >> 8) >> t.cap_e;
}

// One item to the spilled ones (divergent: the active lanes share one claim).
__device__ __forceinline__ void rbin_spill(const RecBinArgs &rb, uint64_t item) {
    const uint64_t act = __builtin_amdgcn_ballot_w64(true);
    const uint32_t before =
        __builtin_amdgcn_mbcnt_hi((uint32_t)(act >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)act, 0));
    unsigned long long base = 0;
    if (before == 0)
        base = atomicAdd(&rb.ctl[0], (unsigned long long)__popcll(act));
    base = (unsigned long long)__builtin_amdgcn_readfirstlane((int)(base >> 32)) << 32 |
           (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)base);
    if (base + before < rb.spill_cap)
        rb.spill[base + before] = item;
    else
        atomicExch(&rb.ctl[1], 1ull);
}

template <bool P2>
__global__ __launch_bounds__(RBIN_BLOCK) __attribute__((amdgpu_waves_per_eu(4)))
void k_rbin_items(SeqArgs a, const uint64_t *c1, TableArgs t, RecBinArgs rb) {
    constexpr uint32_t NT = RBIN_BLOCK, PER = RBIN_PER, CAP = NT * PER;
    __shared__ P2Batch b;
    __shared__ BinSort<RBIN_MAX_BUCKETS, NT, PER, uint64_t> sh;
    OverflowFlag flag;
    const uint32_t k = a.k;
    const bool single = a.single != 0;
    const uint32_t lpb = bin_lanes(rb.n_buckets, CAP);
    for (uint32_t i = threadIdx.x; i < RBIN_MAX_BUCKETS; i += NT)
        sh.cnt[i] = 0;
    // the n collected items to their buckets (sh.srt holds them, then holds
    // them sorted)
    const auto append = [&](uint32_t n) {
        uint64_t item[PER];
        uint32_t at[PER];
        __syncthreads();  // all are collected
#pragma unroll
        for (uint32_t q = 0; q < PER; ++q) {
            const uint32_t i = q * NT + threadIdx.x;
            item[q] = i < n ? sh.srt[i] : BIN_NONE;
            at[q] = ~0u;
            if (item[q] != BIN_NONE) {
                const uint32_t bucket =
                    (uint32_t)((rbin_block<P2>(t, item[q]) - rb.r_lo) >> rb.sub_log2);
                at[q] = bucket << 14 | atomicAdd(&sh.cnt[bucket], 1u);
            }
        }
        bin_append(sh, item, at, rb.n_buckets, lpb, rb.cursor,
                   [&](uint32_t i) { return i * rb.room_a; }, rb.items_a,
                   [&](uint32_t, uint64_t it) { rbin_spill(rb, it); });
    };
    uint32_t n, total, set, have = 0;
    const uint32_t most = batch_tiles(a.n_tiles, gridDim.x);
    RunCursor rc = linear_run(a, max(a.chunk, most));
    while (next_batch<NT>(a, rc, most, c1, b, flag, &n, &total, &set)) {
        for (uint32_t done = 0; done < total;) {
            const uint32_t m = min(total - done, CAP - have);
            for (uint32_t i = threadIdx.x; i < m; i += NT) {
                const uint32_t c = b.at[done + i], q = c & (TILE - 1);
                const P2Tile &tl = b.tile[c / TILE];
                const Span sp = record_span(a, tl, q);
                uint64_t item = BIN_NONE;
                if ((int32_t)q >= sp.gs) {  // (a k-mer start)
                    uint32_t mask;
                    Strands<uint64_t> st;
                    item = record_key<uint64_t>(b.sg[c / TILE], q, k, sp, single, mask, st) << 8;
                    item |= mask;
                    const uint64_t r = rbin_block<P2>(t, item);
                    if (r < rb.r_lo || r >= rb.r_hi)
                        item = BIN_NONE;
                }
                sh.srt[have + i] = item;
            }
            done += m;
            have += m;
            if (have == CAP) {
                append(CAP);
                have = 0;
            }
        }
    }
    append(have);
}

// One batch of one bucket's items (blockIdx.y: the bucket, blockIdx.x: the
// batch) appended to the bucket's blocks.
template <bool P2>
__global__ __launch_bounds__(BIN_BLOCK) void k_rbin_split(TableArgs t, RecBinArgs rb) {
    constexpr uint32_t NT = BIN_BLOCK, PER = RBIN_SPLIT_PER;
    __shared__ BinSort<RBIN_SUB, NT, PER, uint64_t> sh;
    const uint32_t bucket = blockIdx.y, nb = 1u << rb.sub_log2;
    const uint64_t *in = rb.items_a + bucket * rb.room_a;
    const uint64_t n = min((uint64_t)rb.cursor[bucket], rb.room_a);
    const uint64_t i0 = (uint64_t)blockIdx.x * (NT * PER);
    if (i0 >= n)
        return;
    for (uint32_t i = threadIdx.x; i < RBIN_SUB; i += NT)
        sh.cnt[i] = 0;
    uint64_t item[PER];
    uint32_t at[PER];
#pragma unroll
    for (uint32_t q = 0; q < PER; ++q) {
        const uint64_t i = i0 + q * NT + threadIdx.x;
        item[q] = i < n ? in[i] : BIN_NONE;
    }
    __syncthreads();
#pragma unroll
    for (uint32_t q = 0; q < PER; ++q) {
        at[q] = ~0u;
        if (item[q] != BIN_NONE) {
            const uint32_t sub = (uint32_t)(rbin_block<P2>(t, item[q]) - rb.r_lo) & (nb - 1);
            at[q] = sub << 14 | atomicAdd(&sh.cnt[sub], 1u);
        }
    }
    const uint64_t r0 = (uint64_t)bucket << rb.sub_log2;
    bin_append(sh, item, at, nb, bin_lanes(nb, NT * PER), rb.cursor + rb.n_buckets + r0,
               [&](uint32_t i) { return (r0 + i) * rb.room_b; }, rb.items_b,
               [&](uint32_t, uint64_t it) { rbin_spill(rb, it); });
}

// One workgroup per block of the pass: the block built in LDS from empty (an
// item claims an empty slot by compare-and-swap, or ORs its edge bits into
// its key's slot; probes wrap within the block), then written out whole.
// Nothing once items were lost (only kernels before this one set ctl[1]): the
// attempt is done again directly.
template <bool P2>
__global__ __launch_bounds__(BIN_BLOCK) void k_rbin_apply(TableArgs t, RecBinArgs rb,
                                                          SetCounters *sc, Counters *cnt) {
    constexpr uint32_t NT = BIN_BLOCK;
    __shared__ __align__(16) unsigned long long reg[1u << TABLE_BLOCK_LOG2];
    __shared__ unsigned long long fresh_wg, probes_wg;
    __shared__ uint32_t over_wg;
    if (rb.ctl[1])
        return;
    const uint32_t nb = 1u << t.cap_e;  // slots per block
    const uint64_t r = blockIdx.x;
    ulonglong2 *reg2 = (ulonglong2 *)reg;
    for (uint32_t i = threadIdx.x; i < nb / 2; i += NT)
        reg2[i] = make_ulonglong2(EMPTY_KEY, EMPTY_KEY);
    if (threadIdx.x == 0) {
        fresh_wg = probes_wg = 0;
        over_wg = 0;
    }
    __syncthreads();
    const bool split = rb.sub_log2 != 0;
    const uint64_t *items = split ? rb.items_b + r * rb.room_b : rb.items_a + r * rb.room_a;
    const uint64_t n = min((uint64_t)rb.cursor[split ? rb.n_buckets + r : r],
                           split ? rb.room_b : rb.room_a);
    uint32_t fresh = 0, probes = 0;
    bool over = false;
    constexpr uint32_t U = 4;
    // a lane works through U items at its own pace: an item that is done with
    // gives way to the lane's next in the same step, so that a wave takes the
    // steps of its slowest lane over U items, not of each item's slowest lane
    for (uint64_t i = threadIdx.x; i < n; i += U * NT) {
        uint64_t v[U];
        uint32_t s[U], left = 0, tries = 0;
#pragma unroll
        for (uint32_t q = 0; q < U; ++q) {
            const uint64_t j = i + (uint64_t)q * NT;
            v[q] = j < n ? items[j] : BIN_NONE;
            left += j < n;
        }
#pragma unroll
        for (uint32_t q = 0; q < U; ++q)
            s[q] = (uint32_t)first_slot<P2>(t, v[q] >> 8) & (nb - 1);
        probes += left;
        while (left) {
            const unsigned long long cur =
                atomicCAS(&reg[s[0]], EMPTY_KEY, (unsigned long long)v[0]);
            const unsigned long long m = v[0] & 0xFFu;
            bool done = cur == EMPTY_KEY;
            fresh += done;
            if (!done && cur >> 8 == v[0] >> 8) {
                if ((cur & m) != m)
                    atomicOr(&reg[s[0]], m);
                done = true;
            }
            if (!done) {
                s[0] = (s[0] + 1) & (nb - 1);
                probes += (s[0] & 1) == 0;  // a new pair of slots
                if (++tries == MAX_PROBE)
                    done = over = true;
            }
            if (done) {
#pragma unroll
                for (uint32_t q = 0; q + 1 < U; ++q) {
                    v[q] = v[q + 1];
                    s[q] = s[q + 1];
                }
                tries = 0;
                --left;
            }
        }
    }
    if (fresh)
        atomicAdd(&fresh_wg, (unsigned long long)fresh);
    if (probes)
        atomicAdd(&probes_wg, (unsigned long long)probes);
    if (over)
        over_wg = 1;
    __syncthreads();
    ulonglong2 *dst = (ulonglong2 *)(t.keys + ((rb.r_lo + r) << t.cap_e));
    for (uint32_t i = threadIdx.x; i < nb / 2; i += NT)
        dst[i] = reg2[i];
    if (threadIdx.x == 0) {
        if (fresh_wg)
            atomicAdd(&sc->table_keys, fresh_wg);
        if (probes_wg)
            atomicAdd(&cnt->table_probes, probes_wg);
        if (over_wg)
            atomicExch(&sc->overflow, 1ull);
    }
}

// The spilled items into the finished table; once items were lost, the set's
// flag instead, so that the decision skips its tiles.
template <bool P2>
__global__ __launch_bounds__(BLOCK) void k_rbin_spill(TableArgs t, RecBinArgs rb, SetCounters *sc,
                                                      Counters *cnt) {
    if (rb.ctl[1]) {
        if (blockIdx.x == 0 && threadIdx.x == 0)
            atomicExch(&sc->overflow, 1ull);
        return;
    }
    const uint64_t n = min((uint64_t)rb.ctl[0], rb.spill_cap);
    uint32_t keys = 0, probes = 0;
    for (uint64_t i = (uint64_t)blockIdx.x * BLOCK + threadIdx.x; i < n;
         i += (uint64_t)gridDim.x * BLOCK) {
        const uint64_t item = rb.spill[i], key = item >> 8, slot = first_slot<P2>(t, key);
        const int got = insert_pair<P2>(t, item, (uint32_t)item & 0xFFu, slot, load_pair(t, slot),
                                        [&](unsigned long long x) { return x >> 8 == key; },
                                        probes);
        keys += got > 0;
        if (got < 0)
            atomicExch(&sc->overflow, 1ull);
    }
    if (keys)
        atomicAdd(&sc->table_keys, (unsigned long long)keys);
    if (probes)
        atomicAdd(&cnt->table_probes, (unsigned long long)probes);
}

// About 256 buckets, of up to RBIN_SUB blocks (a batch of k_rbin_items then
// leaves in runs of some 24 items), or a block to each where that makes at most
// RBIN_MAX_BUCKETS.  Room for a bin's share and six standard deviations of it,
// its keys coming up once per genome; spill for a sixteenth of the items.
RecBinShape rbin_shape(uint64_t candidates, uint64_t n_blocks, uint64_t blocks, uint32_t genomes) {
    RecBinShape s{};
    if (blocks > RBIN_MAX_BUCKETS)
        while (s.sub_log2 < RBIN_SUB_LOG2 && (blocks - 1) >> s.sub_log2 >= RBIN_MAX_BUCKETS / 2)
            ++s.sub_log2;
    s.n_buckets = (uint32_t)((blocks + (1ull << s.sub_log2) - 1) >> s.sub_log2);
    const double per = (double)candidates / (double)n_blocks;
    const auto room = [&](double mean) {
        return ((uint64_t)(1.02 * mean + 6 * std::sqrt(mean * genomes)) + 64 + 15) / 16 * 16;
    };
    s.room_a = room(per * (double)std::min<uint64_t>(blocks, 1ull << s.sub_log2));
    s.room_b = s.sub_log2 ? room(per) : 0;
    s.spill = candidates / 16 + 65536;
    const uint64_t whole = (uint64_t)s.n_buckets << s.sub_log2;
    s.cursors = (s.n_buckets + (s.sub_log2 ? whole : 0) + 1) / 2 * 2;  // (whole 16-byte pieces)
    s.bytes = 8 * (32 + s.cursors + s.n_buckets * s.room_a + whole * s.room_b + s.spill);
    return s;
}

hipError_t launch_record_binned(const SeqArgs &a, const uint64_t *c1, const TableArgs &t,
                                RecBinArgs rb, uint32_t passes, uint64_t n_blocks,
                                SetCounters *set_cnt, Counters *cnt, hipStream_t s) {
    if (n_blocks == 0 || passes == 0)
        return hipSuccess;
    const uint64_t per_pass = (n_blocks + passes - 1) / passes;
    auto run = [&](auto p2) -> hipError_t {
        constexpr bool P2 = decltype(p2)::value;
        hipError_t e = launch_zero(rb.ctl, 2 * sizeof(unsigned long long), s);
        for (uint64_t r0 = 0; r0 < n_blocks && e == hipSuccess; r0 += per_pass) {
            rb.r_lo = r0;
            rb.r_hi = min(n_blocks, r0 + per_pass);
            e = launch_zero(rb.cursor, rb.cursors * sizeof(unsigned long long), s);
            if (e != hipSuccess)
                break;
            const uint32_t grid =
                (uint32_t)std::max<uint64_t>(1, std::min<uint64_t>(2ull * rb.n_cu, a.n_tiles));
            hipLaunchKernelGGL(k_rbin_items<P2>, dim3(grid), dim3(RBIN_BLOCK), 0, s, a, c1, t, rb);
            if (rb.sub_log2)
                hipLaunchKernelGGL(
                    k_rbin_split<P2>,
                    dim3((uint32_t)((rb.room_a + BIN_BLOCK * RBIN_SPLIT_PER - 1) /
                                    (BIN_BLOCK * RBIN_SPLIT_PER)), rb.n_buckets),
                    dim3(BIN_BLOCK), 0, s, t, rb);
            hipLaunchKernelGGL(k_rbin_apply<P2>, dim3((uint32_t)(rb.r_hi - rb.r_lo)),
                               dim3(BIN_BLOCK), 0, s, t, rb, set_cnt, cnt);
            e = hipGetLastError();
        }
        if (e != hipSuccess)
            return e;
        hipLaunchKernelGGL(k_rbin_spill<P2>, dim3(4 * rb.n_cu), dim3(BLOCK), 0, s, t, rb, set_cnt,
                           cnt);
        return hipGetLastError();
    };
    return t.pow2 ? run(std::true_type{}) : run(std::false_type{});
}

// ------------------------------------------------------------- decide (a4)

// Lookups a decision thread keeps in flight at once (a pair of slots each).
constexpr uint32_t DECIDE_GROUP = 2;

template <class T, bool P2, bool REF>
__global__ __launch_bounds__(BLOCK) void k_decide(SeqArgs a, SentArgs sa, const uint64_t *c1,
                                                  TableArgs pool, uint64_t *jbits,
                                                  bool accumulate, Counters *cnt) {
    __shared__ P2Batch b;
    __shared__ uint32_t jw[P2_TILES * TILE / 32];  // the batch's junction words
    __shared__ uint32_t pf[(1u << PF_MAX_LOG2) / 32];
    __shared__ unsigned long long block_probes, junc_lds;
    OverflowFlag flag;
    SetSum junc = setsum_begin();
    const uint32_t k = a.k;
    const bool single = a.single != 0;
    const T *sent = (const T *)sa.table;
    for (uint32_t i = threadIdx.x; i < prefilter_words(sa.pf_log2); i += BLOCK)
        pf[i] = sa.prefilter[i];
    if (threadIdx.x == 0)
        block_probes = 0;
    unsigned long long my_missing = 0;
    uint32_t my_probes = 0;
    // homologous tiles at once (slab order) share table lines in L2; lookups
    // do not contend, unlike the record's atomics
    const uint32_t most = batch_tiles(a.n_tiles, gridDim.x);
    RunCursor rc = batch_run(a, (a.pass2_slabs & 2) != 0, max(a.chunk, most));
    uint32_t n, total, set;
    while (next_batch<BLOCK>(a, rc, most, c1, b, flag, &n, &total, &set)) {
        const uint32_t jt = threadIdx.x / (TILE / 64);  // this thread's junction word: its tile
        uint64_t *const jdst = jbits + (jt < n ? b.tile[jt].t0 / 64 + threadIdx.x % (TILE / 64) : 0);
        if (b.skip) {
            // this attempt's table overflowed: its results are discarded (the
            // run is redone, or reports the overflow); the tiles' junction
            // words are still defined
            if (!accumulate && jt < n)
                *jdst = 0;
            continue;
        }
        const TableArgs t = table_of(a, pool, set);
        const SetDesc &sd = a.sets[set];
        const T *stab = sent + sd.sent_tab_off;
        const uint32_t slog2 = sd.sent_tab_log2;
        setsum_switch(junc, set, &junc_lds, &a.set_cnt[0].junctions, SETCNT_STRIDE);
        jw[threadIdx.x] = 0;
        static_assert(P2_TILES * TILE / 32 == BLOCK, "a junction half-word per thread");
        __syncthreads();
        // A thread's candidates in groups: the group's candidate k-mers and
        // home slots are computed from LDS alone, then every table word (and,
        // on a sentinel-prefilter hit, the sentinel-table word) is loaded at
        // once, so that several random reads are in flight per lane before
        // any is needed; then each lookup is resolved.  (The k-mer itself is
        // read again from LDS where a lookup needs it, so that a group of
        // wide k-mers fits the registers.)
        for (uint32_t i0 = threadIdx.x; i0 < total; i0 += DECIDE_GROUP * BLOCK) {
            constexpr uint32_t G = DECIDE_GROUP;
            uint64_t slot[G];
            unsigned long long id[G];  // packed: the key; reference: its tag
            u64x2 cur[G];
            uint32_t ss[G], pos[G];
            T sx[G];
            uint32_t look = 0, maybe_sent = 0;
#pragma unroll
            for (uint32_t j = 0; j < G; ++j) {
                slot[j] = 0;
                id[j] = 0;
                ss[j] = 0;
                pos[j] = 0;
                if (i0 + j * BLOCK < total) {
                    pos[j] = b.at[i0 + j * BLOCK];
                    const T canon = norm(kmer_at<T>(b.sg[pos[j] / TILE], pos[j] % TILE + 32, k),
                                         single);
                    look |= 1u << j;
                    const uint64_t hash = slot_hash(canon);
                    slot[j] = home_slot<P2>(t, hash);
                    id[j] = REF ? ref_tag<P2>(t, hash) : (uint64_t)canon;
                    if (slog2 && prefilter_hit(pf, prefilter_bit(hash, sa.pf_log2))) {
                        maybe_sent |= 1u << j;
                        ss[j] = sent_home(canon, slog2);
                    }
                }
            }
#pragma unroll
            for (uint32_t j = 0; j < G; ++j) {
                cur[j].x = cur[j].y = 0;
                if ((look >> j) & 1u)
                    cur[j] = load_pair(t, slot[j]);
                sx[j] = ((maybe_sent >> j) & 1u) ? stab[ss[j]] : T(0);
            }
#pragma unroll
            for (uint32_t j = 0; j < G; ++j) {
                if (!((look >> j) & 1u))
                    continue;
                const uint32_t q = pos[j] % TILE, tj = pos[j] / TILE;
                bool junction = false;
                if ((maybe_sent >> j) & 1u) {
                    const T canon = norm(kmer_at<T>(b.sg[tj], q + 32, k), single);
                    junction = sent_probe_from(stab, slog2, canon, ss[j], sx[j]);
                }
                if (!junction) {
                    const int m = find_pair<P2>(t, slot[j], cur[j], [&](unsigned long long x) {
                        if (!REF)
                            return x >> 8 == id[j];
                        if ((x ^ id[j]) >> t.ref_shift != 0)
                            return false;
                        // this position's own word, or one that reads the same k-mer
                        return (x & ((1ull << t.ref_shift) - 1)) >> 8 == b.tile[tj].t0 + q ||
                               ref_is(a, t, x, kmer_at<T>(b.sg[tj], q + 32, k));
                    }, my_probes);
                    if (m < 0)
                        ++my_missing;
                    else
                        junction = __popc((uint32_t)m & 15u) > 1 || __popc((uint32_t)m >> 4) > 1;
                }
                if (junction)
                    atomicOr(&jw[pos[j] >> 5], 1u << (pos[j] & 31));
            }
        }
        __syncthreads();
        if (jt < n) {
            const uint64_t x = (uint64_t)jw[2 * threadIdx.x + 1] << 32 | jw[2 * threadIdx.x];
            *jdst = accumulate ? *jdst | x : x;
            junc.v += (unsigned long long)__popcll(x);
        }
    }
    setsum_flush(junc, &junc_lds, &a.set_cnt[0].junctions, SETCNT_STRIDE);
    if (my_probes)
        atomicAdd(&block_probes, (unsigned long long)my_probes);
    if (my_missing)
        atomicAdd(&cnt->missing, my_missing);
    __syncthreads();
    if (threadIdx.x == 0 && block_probes)
        atomicAdd(&cnt->table_probes, block_probes);
}

// Resident workgroups per CU (the fewest over the kernel's table modes and
// slot words).
hipError_t pass2_occupancy(KernelId which, int W, int *blocks) {
    *blocks = 1 << 30;
    for (uint32_t v = 0; v < 4; ++v) {
        TableArgs t{};
        t.pow2 = v & 1;
        t.packed = v >> 1;
        const hipError_t e = by_table(W, t, [&](auto tag, auto p2, auto ref) {
            using T = decltype(tag);
            constexpr bool P2 = decltype(p2)::value, REF = decltype(ref)::value;
            int n = 0;
            const void *fn = which == K_RECORD ? (const void *)k_record<T, P2, REF>
                                               : (const void *)k_decide<T, P2, REF>;
            const hipError_t x = hipOccupancyMaxActiveBlocksPerMultiprocessor(&n, fn, BLOCK, 0);
            *blocks = std::min(*blocks, n);
            return x;
        });
        if (e != hipSuccess)
            return e;
    }
    return hipSuccess;
}

hipError_t launch_decide(int W, const SeqArgs &a, const SentArgs &sa, const uint64_t *c1,
                         const TableArgs &pool, uint64_t *jbits, bool accumulate, Counters *cnt,
                         uint32_t grid, hipStream_t s) {
    if (a.n_tiles == 0)
        return hipSuccess;
    return by_table(W, pool, [&](auto tag, auto p2, auto ref) {
        hipLaunchKernelGGL((k_decide<decltype(tag), decltype(p2)::value, decltype(ref)::value>),
                           dim3(grid), dim3(BLOCK), 0, s, a, sa, c1, pool, jbits, accumulate, cnt);
        return hipGetLastError();
    });
}

}  // namespace tp
