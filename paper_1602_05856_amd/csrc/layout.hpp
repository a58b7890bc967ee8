// Data layout in HBM and the kernel launch interface shared by the host
// runtime and the gfx950 kernels.
//
// A plan holds one or more independent genome sets (a batch); a plain build
// is a batch of one set.  Global base index: all genomes of all sets live in
// one 2-bit packed buffer, genome g starting at base index gbase[g], a
// multiple of TILE (so every tile belongs to one genome, hence one set).
// Position bitmaps (candidates C1, junctions J) have one bit per global base
// index; bit i of 64-bit word w is index 64*w + i.  Work is cut into tiles of
// TILE consecutive indices; a tile's bitmap words are written by the wave
// that owns them, so no bitmap atomics are needed.  Each set has its own
// Bloom filter, sentinel list and exact table, carved out of shared pools and
// described by a SetDesc.
//
// Tile order of the first pass: homologous tiles (the same offset in every
// genome) form a slab; slab s goes to XCD s mod 8, and the workgroups of one
// XCD walk its slabs in order, so the filter lines probed by similar genomes
// at similar offsets are fetched into that XCD's L2 once and then hit there.
// The second pass walks tiles in memory order, in that order, or in runs of
// it (tp_config.pass2_slabs).
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace tp {

constexpr uint32_t TILE = 2048;                    // positions per tile
constexpr uint32_t TILE_WORDS = TILE / 32;         // packed 64-bit words per tile
constexpr uint32_t STAGE_WORDS = TILE_WORDS + 6;   // + 1 word before, 5 after (128-base windows)
constexpr uint32_t BLOCK = 256;                    // threads per workgroup
constexpr uint32_t GENOME_ALIGN = TILE;            // bases
constexpr uint32_t NXCD = 8;                       // accelerator dies (L2 domains)
constexpr uint32_t HLL_LOG2 = 12;                  // distinct-count sketch registers
constexpr uint32_t HLL_M = 1u << HLL_LOG2;
constexpr uint32_t PF_MAX_LOG2 = 16;               // sentinel prefilter bits (max)
// Bitmap words per compaction block: few for a small bitmap, whose blocks
// would else be too few to fill the device (at 0.4 Mbp, 4 blocks: the emit took
// 27 us), many for a large one (one workgroup scans the blocks' counts).
constexpr uint32_t SCAN_ROUND = 256;               // words a block takes at once
inline uint32_t scan_words(uint64_t nwords) { return nwords <= (1u << 18) ? SCAN_ROUND : 2048u; }
inline uint64_t scan_blocks(uint64_t nwords) {
    return (nwords + scan_words(nwords) - 1) / scan_words(nwords);
}
constexpr uint32_t FILL_CHUNK = 8;                 // deduplicating fill: tiles per visit
constexpr uint32_t RECORD_RUN = 8;                 // record in runs: tiles per visit
constexpr uint32_t FILL_DD = 4096;                 // deduplicating fill: LDS table entries
constexpr uint64_t EMPTY_KEY = ~0ull;
constexpr uint32_t MAX_PROBE = 1u << 12;           // exact-table probe bound (then regrow)
constexpr uint64_t TABLE_ALIGN = 64;               // set tables start and end on 512-byte key rows
constexpr uint64_t TABLE_TAIL = MAX_PROBE;         // spare slots past a set's capacity (never probed)
constexpr uint32_t TABLE_BLOCK_LOG2 = 13;          // any-size tables: blocks of 8192 slots (probes wrap)
static_assert(TABLE_TAIL % TABLE_ALIGN == 0, "set regions stay aligned");
constexpr uint32_t CLASS_Q_LOG2 = 10;              // k-mer class subranges (rounds)
constexpr uint32_t CLASS_Q = 1u << CLASS_Q_LOG2;
// Binned fill: the filter pool in regions of up to 2^14
// blocks (one workgroup's LDS), buckets of one or more regions.
constexpr uint32_t BIN_REGION_LOG2 = 13;           // 8192 blocks = 64 KiB (2^14 at most)
constexpr uint32_t BIN_MIN_REGION_LOG2 = 8;        // 2 KiB, of small pools
constexpr uint32_t BIN_BUCKETS = 1024;
constexpr uint32_t BIN_MAX_BUCKETS = 2048;         // pools up to 2^32 blocks (32 GiB)
constexpr uint32_t BIN_LOCAL_LOG2 = 21;            // an item's block bits: buckets of up to 2^21 blocks
constexpr uint32_t BIN_BLOCK = 1024;               // threads of the binned fill's kernels
constexpr uint32_t BIN_PER = 16;                   // the split's items per thread per batch
constexpr uint32_t BIN_BATCH = BIN_BLOCK * BIN_PER;
constexpr uint32_t BIN_CHUNK_TILES_MAX = 1u << 20; // 2^31 positions per chunk (explicit)
// Binned record: up to RBIN_MAX_BUCKETS buckets of up to RBIN_SUB table blocks.
constexpr uint32_t RBIN_MAX_BUCKETS = 512;
constexpr uint32_t RBIN_SUB_LOG2 = 9;
constexpr uint32_t RBIN_SUB = 1u << RBIN_SUB_LOG2;
constexpr uint32_t RBIN_BLOCK = 512;               // threads of its items kernel
constexpr uint32_t RBIN_PER = 12;                  // its items per thread per batch
constexpr uint32_t RBIN_SPLIT_PER = 8;             // the split's (of BIN_BLOCK threads)

// A string of S: a maximal N-free run of one genome, of length >= k.
struct DString {
    uint64_t gstart;  // global base index of its first base
    uint64_t gend;    // one past its last base
    uint32_t genome;  // global genome index (over all sets)
    uint32_t set;
};

// Per-tile facts computed on the host: its set and the strings that hold
// positions in it (so no tile kernel searches the string list).
struct TileInfo {
    uint32_t set;
    uint32_t str_lo, str_hi;  // strings overlapping [tile * TILE, (tile + 1) * TILE)
    uint32_t pad;
};

struct SetDesc {
    uint64_t bloom_off;         // first 32-bit word of its filter in the filter pool
    uint64_t bloom_mask;        // filter bits - 1
    uint64_t table_off;         // first slot of its table in the table pools (multiple of 64)
    uint64_t sent_tab_off;      // first slot of its sentinel table in the sentinel pool
    uint32_t table_m, table_e;  // its table has m << e home slots (region: + TABLE_TAIL)
    uint32_t cls_lo, cls_hi;    // current round: class subranges [cls_lo, cls_hi)
    uint32_t sent_tab_log2;     // its sentinel table has 2^log2 slots (at most half full)
    uint32_t pad;
};

// Device counters of one run, per set.
struct SetCounters {
    unsigned long long candidates;  // |C1|
    unsigned long long bloom_popcount;
    // second-pass fields, cleared before every table attempt
    unsigned long long junctions;   // |J|
    unsigned long long table_keys;  // keys claimed in the exact table
    unsigned long long overflow;    // probe bound or spin bound hit
    unsigned long long pad[3];
};
constexpr uint32_t SET_PASS2_OFFSET = 2;  // first second-pass field
constexpr uint32_t SET_PASS2_FIELDS = 3;

// Device counters of one run, whole batch.
struct Counters {
    unsigned long long fill_atomics;  // filter atomicOr issued
    unsigned long long query_probes;  // filter words loaded by the query
    // second-pass fields, cleared before every table attempt
    unsigned long long table_probes;  // slots visited by record + decision
    unsigned long long missing;       // candidate k-mers not found (must stay 0)
    unsigned long long pad[4];
};
constexpr uint32_t PASS2_OFFSET = 2;
constexpr uint32_t PASS2_FIELDS = 2;

struct SeqArgs {
    const uint64_t *seq;       // packed input as 64-bit words
    uint64_t seq_words;
    const DString *strings;
    uint32_t n_strings;
    uint32_t k;
    uint64_t n_tiles;
    uint32_t single;           // ordinary graph only (no reverse complements)
    uint32_t sketch;           // keep the distinct-count sketch (batches of one set)
    const uint32_t *tile_order;    // first-pass order: tiles grouped per XCD, slab by slab
    uint64_t xcd_start[NXCD + 1];  // tile_order range of each XCD
    const TileInfo *tiles;         // per tile, in memory order
    const SetDesc *sets;
    SetCounters *set_cnt;
    uint32_t n_sets;
    uint32_t classes;          // multiple rounds: only k-mers of the round's class count
    uint32_t pass2_slabs;      // bit 0 record, bit 1 decision: walk the first-pass order;
                               // bit 2 record in runs of RECORD_RUN entries of it
    uint32_t fill_dedup;       // blocked fill: skip filter effects the workgroup has sent
    uint32_t chunk;            // tiles a workgroup takes per visit of a tile walk
    uint32_t parts_log2;       // nonzero: few tiles, each cut in 2^parts_log2 parts and every
                               // part a workgroup (memory order)
    unsigned int *queue;       // tile queue of this launch (NXCD zeroed counters), or
                               // null: the walk's static chunk schedule
};

enum KernelId { K_FILL = 0, K_QUERY = 1, K_RECORD = 2, K_DECIDE = 3, K_COUNT = 4 };

// Sentinel k-mers: per set an open-addressing table of the normalised first
// and last k-mers of its strings (home slot by hash, linear probing, empty
// slots all ones -- never a k-mer value), plus two bit prefilters for all
// sets (by table hash, then by the middles' hashes), kept in LDS.
struct SentArgs {
    const void *table;         // sentinel-table pool: W words per slot
    uint32_t n;                // sentinel k-mers (2 per string)
    uint32_t pf_log2;          // a prefilter's size, log2 bits
    const uint32_t *prefilter; // both, one after the other
};
__host__ __device__ constexpr uint32_t prefilter_words(uint32_t pf_log2) {
    return (1u << pf_log2) / 32;
}
constexpr uint32_t SENT_TAB_MIN_LOG2 = 4;

struct BloomArgs {
    uint32_t *words;           // bit i: bit (i & 31) of words[i >> 5] (pool, or a set's region)
    uint64_t mask;             // bits - 1 (bits a power of two)
    uint32_t h;                // hash functions
    uint32_t blocked;          // blocked layout: 64-bit blocks keyed by the middle (k-1)-mer
};

// Exact-table slot words, one 64-bit word per slot:
//   packed     (k <= 27): key << 8 | in/out mask
//   reference  (k >= 28): hash tag | position << 8 | in/out mask, the position
//              (global base index) being where the sequence reads the key
// keys is the pools' base; a tile's set shifts it by table_off.
struct TableArgs {
    unsigned long long *keys;     // slot words
    uint64_t lomask;              // (1 << cap_e) - 1 (a set's; filled per tile)
    uint32_t cap_m, cap_e;        // a set's capacity: cap_m << cap_e home slots
    uint32_t packed;
    uint32_t ref_shift;           // reference words: the tag starts at this bit
    uint32_t pow2;                // table mode: every set's capacity is 2^cap_e (cap_m = 1)
    uint32_t pad;
};
constexpr uint32_t PACKED_MAX_K = 27;  // 2k + 8 <= 62 bits
struct OutArgs {
    uint64_t *pos;             // genome coordinate per junction
    uint64_t *vertex;          // W words per junction
    uint8_t *strand;
    uint64_t *joff;            // n_genomes + 1
    void *edges;               // tp_edge per edge
    const uint64_t *gbase;     // per genome
    uint32_t n_genomes;
    uint32_t pad;
};

// -------------------------------------------------------------- launchers
// Resident workgroups per CU of a tile kernel (sizes its persistent grid):
// pass1_occupancy for K_FILL / K_QUERY, pass2_occupancy for K_RECORD / K_DECIDE.
hipError_t pass1_occupancy(KernelId which, int W, bool blocked, bool fill_dedup, uint64_t n_tiles,
                           int *blocks_per_cu);
hipError_t pass2_occupancy(KernelId which, int W, int *blocks_per_cu);
// Several regions set to a repeated 32-bit value, or copied from memory that
// the device can read, in one launch (addresses multiples of 16 bytes; sizes
// too, a copy's rounded up).
struct ClearList {
    struct {
        void *p;
        const void *src;  // null: set to v
        uint64_t n16;
        uint32_t v;
    } r[10];
    uint32_t n;
    void add(void *p, uint64_t bytes, uint32_t v = 0) { put(p, nullptr, bytes / 16, v); }
    void copy(void *p, const void *src, uint64_t bytes) { put(p, src, (bytes + 15) / 16, 0); }
    void put(void *p, const void *src, uint64_t n16, uint32_t v) {
        if (n16)
            r[n].p = p, r[n].src = src, r[n].n16 = n16, r[n++].v = v;
    }
};
hipError_t launch_clear(const ClearList &c, hipStream_t s);

// What the host reads at its waits, written to memory that it can read (or to
// device memory for one copy) by one small kernel: counters, and of the
// sketch's registers (null: none) what its estimate needs.
struct SketchSum {
    double z;        // sum of 2^-register
    uint64_t zeros;  // empty registers
};
hipError_t launch_publish(const ClearList &copies, const uint32_t *hll, SketchSum *sketch,
                          hipStream_t s);
hipError_t launch_zero(void *p, uint64_t bytes, hipStream_t s);
hipError_t launch_fill_u64(uint64_t *p, uint64_t n, uint64_t v, hipStream_t s);

// a0: each set's sentinel table (normalised first and last k-mer of every
// string; tab_owner: a claim word per slot, tab_slots in all) and the sentinel
// prefilters, all cleared beforehand (clear_sentinels).
void clear_sentinels(ClearList &c, int W, const SentArgs &sa, uint32_t *tab_owner,
                     uint64_t tab_slots);
hipError_t launch_sentinels(int W, const SeqArgs &a, const SentArgs &sa, uint32_t *tab_owner,
                            hipStream_t s);
// a1: insert every normalised (k+1)-mer into its set's Bloom filter.
// Binned fill of a filter pool (the same bits as launch_fill; the pool zeroed
// beforehand): per chunk of tiles, every edge's filter effect (standard filter:
// every bit of it) becomes a 4-byte item of its bucket, the items of a bucket of several
// regions are split by region, and one workgroup per region ORs its items in
// LDS and writes the region back.
struct BinArgs {
    uint32_t *items_a;          // items by bucket
    uint32_t *items_b;          // items by region (buckets of several regions)
    unsigned long long *cursor; // per bucket, then (several regions) per region: items claimed
    const uint64_t *off;        // room: per bucket its first item in items_a, then the end
    const uint64_t *roff;       // per region its first item in items_b, then the end
    uint64_t t_lo, t_hi;        // the chunk: a range of the first-pass tile order
    uint64_t n_blocks;          // 64-bit blocks of the filter pool
    uint32_t n_buckets, bucket_log2, region_log2, n_regions;
    uint32_t slices;            // batches a bucket has room for (the split's grid)
    uint32_t n_cu;
    uint32_t cleared;           // the cursors are clear for the first chunk
    SetCounters *popcount;      // last chunk of a one-set pool: its filter popcount, else null
};
// Blocks of a bucket and of a region for a pool: one region per bucket where
// BIN_BUCKETS regions cover the pool (the larger regions only where they make
// that so: they leave one apply workgroup per CU instead of two), else about
// 256 buckets of up to 2^21 blocks, split by region afterwards (a batch's
// longer runs: 654 Mbp over 128 filters of 1.4 GB in all, k_bin_items 4.15 ms
// against 4.67 with 1024 buckets; 3.5 since).  Pools beyond 16 GiB need up to 2048
// buckets, for an item's block bits.
// The standard filter's items (h to an edge) go to 256 buckets at most:
// their claims (an atomic per bin and batch) would take as long as the sort.
inline void bin_shape(uint64_t n_blocks, bool blocked, uint32_t *bucket_log2,
                      uint32_t *region_log2) {
    const uint64_t last = n_blocks ? n_blocks - 1 : 0;
    *region_log2 = BIN_REGION_LOG2;
    // a small pool in smaller regions, up to one to a CU (2 MiB: 16.7 us in 32
    // regions, 12.5 in 256)
    while (*region_log2 > BIN_MIN_REGION_LOG2 && (last >> (*region_log2 - 1)) < BIN_BUCKETS / 4)
        --*region_log2;
    if (blocked && (last >> BIN_REGION_LOG2) >= BIN_BUCKETS && (last >> (BIN_REGION_LOG2 + 1)) < BIN_BUCKETS)
        ++*region_log2;
    *bucket_log2 = *region_log2;
    if ((last >> *region_log2) >= (blocked ? BIN_BUCKETS : BIN_BUCKETS / 4))
        while ((last >> *bucket_log2) >= BIN_BUCKETS / 4 && *bucket_log2 < BIN_LOCAL_LOG2)
            ++*bucket_log2;
}
hipError_t launch_fill_binned(int W, const SeqArgs &a, const BloomArgs &pool, Counters *cnt,
                              BinArgs b, uint32_t tiles_per_chunk, hipStream_t s);
hipError_t launch_fill(int W, const SeqArgs &a, const BloomArgs &pool, Counters *cnt,
                       uint32_t grid, hipStream_t s);
// a2: Bloom-queried neighbourhood of every k-mer position -> C1 bitmap,
// candidate counts and (one set) distinct-count sketch of candidate k-mers.
// With classes, only the round's k-mers are evaluated, and c1_union (when
// not null) collects the rounds' candidate bitmaps (overwritten in round 0).
hipError_t launch_query(int W, const SeqArgs &a, const BloomArgs &pool, const SentArgs &sa,
                        uint64_t *c1, uint64_t *c1_union, uint32_t round, Counters *cnt,
                        uint32_t *hll, uint32_t grid, hipStream_t s);
// Multiple rounds: per set, CLASS_Q counters of (k+1)-mer occurrences per
// class subrange of the two k-mers each contains (once per distinct one).
hipError_t launch_census(int W, const SeqArgs &a, unsigned long long *counters, uint32_t grid,
                         hipStream_t s);
// Filter popcount per set (bloom_starts: n_sets + 1 word offsets, device).
hipError_t launch_popcount(const uint32_t *pool, uint64_t n_words, const uint64_t *bloom_starts,
                           uint32_t n_sets, SetCounters *set_cnt, hipStream_t s);
// a3: exact in/out edge masks of every candidate k-mer.
hipError_t launch_record(int W, const SeqArgs &a, const uint64_t *c1, const TableArgs &pool,
                         Counters *cnt, uint32_t grid, hipStream_t s);

// Binned record (one set, packed one-word slots, home blocks of at most
// 2^TABLE_BLOCK_LOG2 slots): per pass, the candidates whose home block lies
// in [r_lo, r_hi) become items (their slot words), are partitioned by block
// and each block is built in LDS and written out whole.
constexpr uint32_t RBIN_MAX_PASSES = 64;
struct RecBinArgs {
    uint64_t *items_a;           // the pass's items by bucket
    uint64_t *items_b;           // the pass's items by block (buckets of several blocks)
    uint64_t *spill;             // items without room, of all passes
    unsigned long long *cursor;  // per bucket, then (several blocks) per block: items claimed
    unsigned long long *ctl;     // [0] items spilled, [1] nonzero: more than spill holds
    uint64_t room_a, room_b;     // items a bucket, a block has room for
    uint64_t spill_cap;
    uint64_t cursors;            // entries of cursor, rounded up to whole 16-byte pieces
    uint64_t r_lo, r_hi;         // the pass's home blocks
    uint32_t sub_log2;           // a bucket is 2^sub_log2 blocks
    uint32_t n_buckets;
    uint32_t n_cu;
};
// What a pass over `blocks` of a table's n_blocks home blocks takes.
struct RecBinShape {
    uint32_t sub_log2, n_buckets;
    uint64_t room_a, room_b, spill, bytes, cursors;
};
RecBinShape rbin_shape(uint64_t candidates, uint64_t n_blocks, uint64_t blocks, uint32_t genomes);
// table: set 0's table (keys, cap_m, cap_e, lomask, pow2 filled in).
hipError_t launch_record_binned(const SeqArgs &a, const uint64_t *c1, const TableArgs &table,
                                RecBinArgs rb, uint32_t passes, uint64_t n_blocks,
                                SetCounters *set_cnt, Counters *cnt, hipStream_t s);
// a4: junction decision for every candidate -> J bitmap and counts.
// With accumulate, junction words are ORed into jbits (rounds after the first).
hipError_t launch_decide(int W, const SeqArgs &a, const SentArgs &sa, const uint64_t *c1,
                         const TableArgs &pool, uint64_t *jbits, bool accumulate, Counters *cnt,
                         uint32_t grid, hipStream_t s);
// a5: ordered compaction of J and compacted edges.
hipError_t launch_compact(int W, const SeqArgs &a, const uint64_t *jbits, uint64_t nwords,
                          uint32_t *blockcnt, uint64_t *blockoff, const OutArgs &o,
                          uint64_t n_junctions, hipStream_t s);
// a5 with the junction count unknown on the host: the kernels always run,
// writing at most max_j junctions and max_e edges (joff holds true counts).
hipError_t launch_compact_bound(int W, const SeqArgs &a, const uint64_t *jbits, uint64_t nwords,
                                uint32_t *blockcnt, uint64_t *blockoff, const OutArgs &o,
                                uint64_t max_j, uint64_t max_e, hipStream_t s);

// Multiple rounds on the device: the greedy partition of every set's census
// (bounds: rounds + 1 per set), and the round's class bounds copied into the
// set descriptors.
hipError_t launch_partition(const unsigned long long *census, uint32_t n_sets, uint32_t rounds,
                            uint32_t *bounds, hipStream_t s);
hipError_t launch_set_round(SetDesc *sets, const uint32_t *bounds, uint32_t n_sets,
                            uint32_t rounds, uint32_t round, hipStream_t s);

// Counts of a caller-memory run, summed on the device (tp_ws_counts layout:
// status, positions, candidates, junctions, edges, table_keys, popcount).
struct FinalizeArgs {
    const SetCounters *set_cnt;
    const Counters *cnt;
    const uint64_t *blockoff;  // compaction scan: total at [nblocks]
    uint64_t nblocks;
    uint32_t n_sets;
    uint32_t pass2;            // second pass ran (table status is meaningful)
    uint64_t n_strings, positions, max_j;
    unsigned long long *out;   // 16 words
};
hipError_t launch_ws_finalize(const FinalizeArgs &f, hipStream_t s);

}  // namespace tp
