// Device helpers of the gfx950 junction-finding kernels: k-mer windows read
// from 2-bit packed sequence staged in LDS, normalised (canonical) k-mers,
// the Bloom/table hash specification, string (contig) lookup and the
// sentinel filter.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "layout.hpp"

namespace tp {

typedef unsigned __int128 u128;

// ---------------------------------------------------------------- hash spec
// mix64 is the SplitMix64 output function (Steele, Lea & Flood 2014).
// Bloom bit t of a normalised (k+1)-mer e: (H1 + t*H2) mod 2^64 mod b with
// H1 = mix64(fold(e) ^ S1), H2 = mix64(fold(e) ^ S2) | 1 (double hashing,
// Kirsch & Mitzenmacher 2006).  fold(e) = e for one-word values, else
// mix64(hi ^ S0) ^ lo.  Table slot of a normalised k-mer v:
// mix64(fold(v) ^ S3) mod capacity.  S0..S3 are hexadecimal digits of pi.
constexpr uint64_t kS0 = 0x243F6A8885A308D3ull;
constexpr uint64_t kS1 = 0x13198A2E03707344ull;
constexpr uint64_t kS2 = 0xA4093822299F31D0ull;
constexpr uint64_t kS3 = 0x082EFA98EC4E6C89ull;
constexpr uint64_t kS4 = 0x452821E638D01377ull;  // k-mer classes (multiple rounds)

__device__ __forceinline__ uint64_t mix64(uint64_t z) {
    z = (z ^ (z >> 30)) * 0xBF58476D1CE4E5B9ull;
    z = (z ^ (z >> 27)) * 0x94D049BB133111EBull;
    return z ^ (z >> 31);
}

// Reverse the order of the 2-bit groups of a 64-bit word.
__device__ __forceinline__ uint64_t rev2(uint64_t x) {
    uint64_t y = __builtin_bitreverse64(x);
    return ((y >> 1) & 0x5555555555555555ull) | ((y << 1) & 0xAAAAAAAAAAAAAAAAull);
}

// (lo >> sh) | (hi << (64 - sh)) for 0 <= sh < 64, without a branch.
__device__ __forceinline__ uint64_t funnel(uint64_t lo, uint64_t hi, uint32_t sh) {
    return (lo >> sh) | ((hi << 1) << (63 - sh));
}

// Four-word unsigned value (k <= 127: up to 128 bases), w0 least
// significant, with the operators the k-mer code uses.  Shifts by a variable
// count select words with conditional moves (no indexed register arrays).
struct u256 {
    uint64_t w0, w1, w2, w3;
    u256() = default;
    __host__ __device__ constexpr u256(uint64_t x) : w0(x), w1(0), w2(0), w3(0) {}
    __host__ __device__ constexpr u256(uint64_t a, uint64_t b, uint64_t c, uint64_t d)
        : w0(a), w1(b), w2(c), w3(d) {}
    __device__ __forceinline__ explicit operator uint64_t() const { return w0; }
    __device__ __forceinline__ explicit operator uint32_t() const { return (uint32_t)w0; }
};

__device__ __forceinline__ uint64_t u256_word(const u256 &a, uint32_t i) {
    return i == 0 ? a.w0 : i == 1 ? a.w1 : i == 2 ? a.w2 : i == 3 ? a.w3 : 0ull;
}
__device__ __forceinline__ u256 operator>>(const u256 &a, uint32_t n) {
    if (n >= 256)
        return u256(0);
    const uint32_t q = n >> 6, sh = n & 63;
    auto part = [&](uint32_t i) {
        const uint64_t lo = u256_word(a, i + q), hi = u256_word(a, i + q + 1);
        return sh ? (lo >> sh) | (hi << (64 - sh)) : lo;
    };
    return u256(part(0), part(1), part(2), part(3));
}
__device__ __forceinline__ u256 operator<<(const u256 &a, uint32_t n) {
    if (n >= 256)
        return u256(0);
    const uint32_t q = n >> 6, sh = n & 63;
    auto part = [&](uint32_t i) {
        const uint64_t hi = i >= q ? u256_word(a, i - q) : 0ull;
        const uint64_t lo = i >= q + 1 ? u256_word(a, i - q - 1) : 0ull;
        return sh ? (hi << sh) | (lo >> (64 - sh)) : hi;
    };
    return u256(part(0), part(1), part(2), part(3));
}
__device__ __forceinline__ u256 operator&(const u256 &a, const u256 &b) {
    return u256(a.w0 & b.w0, a.w1 & b.w1, a.w2 & b.w2, a.w3 & b.w3);
}
__device__ __forceinline__ u256 operator|(const u256 &a, const u256 &b) {
    return u256(a.w0 | b.w0, a.w1 | b.w1, a.w2 | b.w2, a.w3 | b.w3);
}
__device__ __forceinline__ u256 operator^(const u256 &a, const u256 &b) {
    return u256(a.w0 ^ b.w0, a.w1 ^ b.w1, a.w2 ^ b.w2, a.w3 ^ b.w3);
}
__device__ __forceinline__ u256 operator~(const u256 &a) {
    return u256(~a.w0, ~a.w1, ~a.w2, ~a.w3);
}
__device__ __forceinline__ bool operator==(const u256 &a, const u256 &b) {
    return ((a.w0 ^ b.w0) | (a.w1 ^ b.w1) | (a.w2 ^ b.w2) | (a.w3 ^ b.w3)) == 0;
}
__device__ __forceinline__ bool operator!=(const u256 &a, const u256 &b) { return !(a == b); }
__device__ __forceinline__ bool operator<(const u256 &a, const u256 &b) {
    if (a.w3 != b.w3)
        return a.w3 < b.w3;
    if (a.w2 != b.w2)
        return a.w2 < b.w2;
    if (a.w1 != b.w1)
        return a.w1 < b.w1;
    return a.w0 < b.w0;
}
__device__ __forceinline__ bool operator>(const u256 &a, const u256 &b) { return b < a; }
__device__ __forceinline__ bool operator<=(const u256 &a, const u256 &b) { return !(b < a); }
__device__ __forceinline__ bool operator>=(const u256 &a, const u256 &b) { return !(a < b); }

// Host-side dispatch on the k-mer width: f(tag) with a value of the k-mer
// type of W words (1: uint64_t, 2: u128, 4: u256).
template <class F> hipError_t by_width(int W, F &&f) {
    if (W == 1)
        return f(uint64_t{});
    if (W == 2)
        return f(u128{});
    return f(u256{});
}

// k-mer word traits: W = 1 (uint64_t, k <= 31), W = 2 (u128, k <= 63) or
// W = 4 (u256, k <= 127).  fold(x): the top word, then for each lower word
// f = mix64(f ^ S0) ^ word.
template <class T> struct KT;

template <> struct KT<uint64_t> {
    static constexpr int W = 1;
    __device__ static __forceinline__ uint64_t fold(uint64_t x) { return x; }
    // A word that depends on all of x (internal tables; not the hash spec).
    __device__ static __forceinline__ uint64_t mixed(uint64_t x) { return x ^ x >> 29; }
    __device__ static __forceinline__ uint64_t ones(uint32_t nbits) {
        return nbits >= 64 ? ~0ull : ((1ull << nbits) - 1);
    }
    // LSB-first window of L <= 32 bases starting at base index r of words w.
    __device__ static __forceinline__ uint64_t window(const uint64_t *w, uint32_t r, uint32_t L) {
        uint32_t q = r >> 5, sh = 2 * (r & 31);
        return funnel(w[q], w[q + 1], sh) & ones(2 * L);
    }
    // The 32 bases from base r of the 32-bit words w (LSB first).
    __device__ static __forceinline__ uint64_t win(const uint32_t *w, uint32_t r) {
        const uint32_t *p = w + (r >> 4), s = 2 * r;
        return (uint64_t)__builtin_amdgcn_alignbit(p[2], p[1], s) << 32 |
               __builtin_amdgcn_alignbit(p[1], p[0], s);
    }
    // val (first base most significant) of an LSB-first window of L bases.
    __device__ static __forceinline__ uint64_t val(uint64_t x, uint32_t L) {
        return rev2(x) >> (64 - 2 * L);
    }
    __device__ static __forceinline__ uint64_t word(uint64_t x, uint32_t) { return x; }
};

template <> struct KT<u128> {
    static constexpr int W = 2;
    __device__ static __forceinline__ uint64_t fold(u128 x) {
        return mix64((uint64_t)(x >> 64) ^ kS0) ^ (uint64_t)x;
    }
    __device__ static __forceinline__ uint64_t mixed(u128 x) {
        return KT<uint64_t>::mixed((uint64_t)x + (uint64_t)(x >> 64) * 0xD6E8FEB86659FD93ull);
    }
    __device__ static __forceinline__ u128 ones(uint32_t nbits) {
        return nbits >= 128 ? ~(u128)0 : (((u128)1 << nbits) - 1);
    }
    __device__ static __forceinline__ u128 window(const uint64_t *w, uint32_t r, uint32_t L) {
        uint32_t q = r >> 5, sh = 2 * (r & 31);
        uint64_t a = funnel(w[q], w[q + 1], sh);
        uint64_t b = funnel(w[q + 1], w[q + 2], sh);
        return (((u128)b << 64) | a) & ones(2 * L);
    }
    __device__ static __forceinline__ u128 win(const uint32_t *w, uint32_t r) {
        return (u128)KT<uint64_t>::win(w + 2, r) << 64 | KT<uint64_t>::win(w, r);
    }
    __device__ static __forceinline__ u128 val(u128 x, uint32_t L) {
        u128 r = ((u128)rev2((uint64_t)x) << 64) | rev2((uint64_t)(x >> 64));
        return r >> (128 - 2 * L);
    }
    __device__ static __forceinline__ uint64_t word(u128 x, uint32_t i) {
        return i == 0 ? (uint64_t)x : (uint64_t)(x >> 64);
    }
};

template <> struct KT<u256> {
    static constexpr int W = 4;
    __device__ static __forceinline__ uint64_t fold(const u256 &x) {
        uint64_t f = x.w3;
        f = mix64(f ^ kS0) ^ x.w2;
        f = mix64(f ^ kS0) ^ x.w1;
        return mix64(f ^ kS0) ^ x.w0;
    }
    __device__ static __forceinline__ uint64_t mixed(const u256 &x) {
        return KT<uint64_t>::mixed(x.w0 + x.w1 * 0xD6E8FEB86659FD93ull +
                                   (x.w2 + x.w3 * 0xD6E8FEB86659FD93ull) * 0xA0761D6478BD642Full);
    }
    __device__ static __forceinline__ u256 ones(uint32_t nbits) {
        auto part = [&](uint32_t i) -> uint64_t {
            const uint32_t lo = 64 * i;
            return nbits >= lo + 64 ? ~0ull : nbits <= lo ? 0ull : ((1ull << (nbits - lo)) - 1);
        };
        return u256(part(0), part(1), part(2), part(3));
    }
    // LSB-first window of L <= 128 bases starting at base index r of words w.
    __device__ static __forceinline__ u256 window(const uint64_t *w, uint32_t r, uint32_t L) {
        const uint32_t q = r >> 5, sh = 2 * (r & 31);
        const u256 x(funnel(w[q], w[q + 1], sh), funnel(w[q + 1], w[q + 2], sh),
                     funnel(w[q + 2], w[q + 3], sh), funnel(w[q + 3], w[q + 4], sh));
        return x & ones(2 * L);
    }
    __device__ static __forceinline__ u256 win(const uint32_t *w, uint32_t r) {
        return u256(KT<uint64_t>::win(w, r), KT<uint64_t>::win(w + 2, r),
                    KT<uint64_t>::win(w + 4, r), KT<uint64_t>::win(w + 6, r));
    }
    __device__ static __forceinline__ u256 val(const u256 &x, uint32_t L) {
        const u256 r(rev2(x.w3), rev2(x.w2), rev2(x.w1), rev2(x.w0));
        return r >> (256 - 2 * L);
    }
    __device__ static __forceinline__ uint64_t word(const u256 &x, uint32_t i) {
        return u256_word(x, i);
    }
};

// The value and reverse-complement value of an L-mer given its LSB-first
// window x: the reverse complement of base string s is sum (3-s[t]) 4^t over
// the LSB-first order, i.e. x with every 2-bit group complemented.
template <class T> struct Strands {
    T fwd, rc;
};

template <class T>
__device__ __forceinline__ Strands<T> strands(T x, uint32_t L) {
    Strands<T> s;
    s.fwd = KT<T>::val(x, L);
    s.rc = x ^ KT<T>::ones(2 * L);
    return s;
}

template <class T>
__device__ __forceinline__ T norm(const Strands<T> &s, bool single) {
    return (single || s.fwd <= s.rc) ? s.fwd : s.rc;
}

// ------------------------------------------------------------ staged tile
// A tile's packed words in LDS twice: as they are (f) and in reverse base
// order (b; base u of b is base STAGE_BASES - 1 - u of f).  A k-mer's value
// has its first base most significant, so it is a window of b, as its reverse
// complement's is the complement of a window of f: both strands of a k-mer
// are cut out with one funnel shift per 32-bit word, with no bit reversal and
// no shift by the k-mer's length (which for a four-word k-mer were more than
// half of the instructions; the tile kernels are bound by those).  Base index
// r of the stage is global base index tile * TILE - 32 + r.
constexpr uint32_t STAGE_BASES = STAGE_WORDS * 32;
struct Stage {
    uint64_t f[STAGE_WORDS];
    uint64_t b[STAGE_WORDS + 4];  // (the longest window reads past a short k-mer's last word)
};

__device__ __forceinline__ void stage_word(Stage &sg, uint32_t i, uint64_t x) {
    sg.f[i] = x;
    sg.b[STAGE_WORDS - 1 - i] = rev2(x);
}

// Bases from r upwards, and from r - 1 downwards, the first in the low bits.
template <class T> __device__ __forceinline__ T up_from(const Stage &sg, uint32_t r) {
    return KT<T>::win((const uint32_t *)sg.f, r);
}
template <class T> __device__ __forceinline__ T down_from(const Stage &sg, uint32_t r) {
    return KT<T>::win((const uint32_t *)sg.b, STAGE_BASES - r);
}

// The value and reverse-complement value of the L-mer at r.
template <class T>
__device__ __forceinline__ Strands<T> kmer_at(const Stage &sg, uint32_t r, uint32_t L) {
    const T ones = KT<T>::ones(2 * L);
    Strands<T> s;
    s.fwd = down_from<T>(sg, r + L) & ones;
    s.rc = ~up_from<T>(sg, r) & ones;
    return s;
}

// The k-mer at r with the bases before and after it.
template <class T>
__device__ __forceinline__ Strands<T> kmer_between(const Stage &sg, uint32_t r, uint32_t k,
                                                   uint32_t *before, uint32_t *after) {
    const T ones = KT<T>::ones(2 * k);
    const T u = up_from<T>(sg, r - 1), d = down_from<T>(sg, r + k + 1);
    *before = (uint32_t)u & 3u;
    *after = (uint32_t)d & 3u;
    Strands<T> s;
    s.fwd = (d >> 2) & ones;
    s.rc = ~(u >> 2) & ones;
    return s;
}

// A string relative to a tile: its first base and the one past its last, cut
// to what a position of the tile can tell apart (first: before the tile, -1).
// A position q of the tile starts a k-mer when gs <= q and q + k <= ge; it is
// the string's first when q == gs, its last when q + k == ge.
struct Span {
    int32_t gs, ge;
};

__device__ __forceinline__ Span span_of(const DString *S, uint32_t si, uint64_t t0) {
    const int64_t a = (int64_t)(S[si].gstart - t0), b = (int64_t)(S[si].gend - t0);
    return Span{(int32_t)(a < -1 ? -1 : a), (int32_t)(b > (1 << 20) ? (1 << 20) : b)};
}

// --------------------------------------------------------------- Bloom ops
struct BloomHash {
    uint64_t h1, h2;
};

template <class T>
__device__ __forceinline__ BloomHash bloom_hash(T e) {
    uint64_t f = KT<T>::fold(e);
    BloomHash bh;
    bh.h1 = mix64(f ^ kS1);
    bh.h2 = mix64(f ^ kS2) | 1ull;
    return bh;
}

// Blocked filter: all h bits of an edge x.m.y lie in the 64-bit block of its
// normalised middle (k-1)-mer mu: block = mix64(fold(mu) ^ S1) mod (b/64);
// with G = mix64(fold(mu) ^ S2), a = G & 63, d = ((G >> 6) & 63) | 1, the edge
// written in mu's orientation as (p, q) sets bits (a + (j*h + t)*d) mod 64,
// j = 4p + q, t < h.  orient: 0 middle read forward, 1 middle reversed,
// 2 palindromic middle (orientation of the normalised edge decides).
struct MiddleKey {
    uint64_t block;
    uint64_t g;  // G (also an orientation-free hash of the middle)
    uint32_t a, d, orient;
};

template <class T>
__device__ __forceinline__ MiddleKey middle_key(const T &mf, const T &mr, bool single,
                                                uint64_t nblock_mask) {
    MiddleKey key;
    const bool rev = !single && mr < mf;
    const T mu = rev ? mr : mf;
    key.orient = rev ? 1u : (!single && mr == mf) ? 2u : 0u;
    const uint64_t f = KT<T>::fold(mu);
    key.block = mix64(f ^ kS1) & nblock_mask;
    const uint64_t g = mix64(f ^ kS2);
    key.g = g;
    key.a = (uint32_t)(g & 63);
    key.d = (uint32_t)((g >> 6) & 63) | 1u;
    return key;
}

// Bits of edge pair j = 4p + q inside its block.
__device__ __forceinline__ uint64_t pair_mask(uint32_t a, uint32_t d, uint32_t j, uint32_t h) {
    uint64_t m = 0;
    for (uint32_t t = 0; t < h; ++t)
        m |= 1ull << ((a + (j * h + t) * d) & 63u);
    return m;
}

// Pair index of edge x.m.y in its middle's orientation.  With a palindromic
// middle the edge's value is at most its reverse complement's when x is at
// most 3 - y.
__device__ __forceinline__ uint32_t pair_index(uint32_t orient, uint32_t x, uint32_t y) {
    const bool flip = orient == 1 || (orient == 2 && x + y > 3);
    return flip ? 4 * (3 - y) + (3 - x) : 4 * x + y;
}

template <class T>
__device__ __forceinline__ uint64_t slot_hash(T v) {
    return mix64(KT<T>::fold(v) ^ kS3);
}

// Class subrange of a normalised k-mer for the multiple-rounds partition
// (Multiple Rounds section): the top CLASS_Q_LOG2 bits of mix64(fold(v) ^ S4).
template <class T>
__device__ __forceinline__ uint32_t class_subrange(T v) {
    return (uint32_t)(mix64(KT<T>::fold(v) ^ kS4) >> (64 - CLASS_Q_LOG2));
}

__device__ __forceinline__ bool in_class(uint32_t sub, uint32_t lo, uint32_t hi) {
    return sub >= lo && sub < hi;
}

// ---------------------------------------------------------- string lookup
// Strings (contigs) of length >= k, sorted by gstart, disjoint, in global
// base-index coordinates.  find the last string with gstart <= p among
// [lo, hi); returns hi when there is none.
__device__ __forceinline__ uint32_t find_string(const DString *S, uint32_t lo, uint32_t hi,
                                                uint64_t p) {
    uint32_t a = lo, b = hi;  // answer in [a-1, b)
    while (a < b) {
        uint32_t m = (a + b) >> 1;
        if (S[m].gstart <= p)
            a = m + 1;
        else
            b = m;
    }
    return a == lo ? hi : a - 1;
}

// The span of the string that holds position q of the tile at t0, among the
// tile's strings [lo, hi), or one that holds nothing.
__device__ __forceinline__ Span span_at(const DString *S, uint32_t lo, uint32_t hi, uint64_t t0,
                                        uint32_t q) {
    const uint32_t si = find_string(S, lo, hi, t0 + q);
    return si != hi ? span_of(S, si, t0) : Span{1 << 20, -1};
}

// ------------------------------------------------------- sentinel filter
// Sentinel k-mers (normalised first and last k-mer of every string): a bit
// prefilter kept in LDS, then the set's open-addressing sentinel table.
constexpr uint64_t kS6 = 0xC0AC29B7C97C50DDull;  // sentinel-table slots

// Two prefilters of the same sentinels, each by a hash that its kernels have at
// hand: the k-mer's table hash (the standard query and the decision), and the
// sum of the G values of its two middles (the blocked query; the same for both
// orientations).
__device__ __forceinline__ uint32_t prefilter_bit(uint64_t slot_hash, uint32_t log2bits) {
    return (uint32_t)(slot_hash >> 32) >> (32 - log2bits);
}
__device__ __forceinline__ uint32_t prefilter_bit_g(uint32_t ghi_sum, uint32_t log2bits) {
    return ghi_sum >> (32 - log2bits);
}

__device__ __forceinline__ bool prefilter_hit(const uint32_t *lds_pf, uint32_t bit) {
    return (lds_pf[bit >> 5] >> (bit & 31)) & 1u;
}

// Home slot of v in a sentinel table of 2^log2 slots.
template <class T>
__device__ __forceinline__ uint32_t sent_home(T v, uint32_t log2) {
    return (uint32_t)(mix64(KT<T>::fold(v) ^ kS6) >> (64 - log2));
}

// Whether v is in the sentinel table tab[0 .. 2^log2), probing from slot s
// whose value x has already been read.  The table is at most half full, so
// an empty slot ends every probe sequence.
template <class T>
__device__ __forceinline__ bool sent_probe_from(const T *tab, uint32_t log2, T v, uint32_t s, T x) {
    const uint32_t mask = (1u << log2) - 1;
    for (uint32_t i = 0; i <= mask; ++i) {
        if (i)
            x = tab[s];
        if (x == v)
            return true;
        if (x == ~T(0))
            return false;
        s = (s + 1) & mask;
    }
    return false;
}

// Membership in a set's sentinel table (tab: the set's first slot).
template <class T>
__device__ __forceinline__ bool in_sentinels(const T &v, const T *tab, uint32_t log2) {
    const uint32_t s = sent_home(v, log2);
    return sent_probe_from(tab, log2, v, s, tab[s]);
}

// A tile's set: its index, sentinel slice and filter region.
struct TileSet {
    uint32_t set;
    uint32_t sent_log2;
    uint64_t sent_off;
    uint32_t cls_lo, cls_hi;
    BloomArgs f;
};

__device__ __forceinline__ TileSet tile_set_of(const SeqArgs &a, const BloomArgs &pool,
                                               uint32_t set) {
    TileSet ts;
    ts.set = set;
    const SetDesc &d = a.sets[ts.set];
    ts.sent_log2 = d.sent_tab_log2;
    ts.sent_off = d.sent_tab_off;
    ts.cls_lo = d.cls_lo;
    ts.cls_hi = d.cls_hi;
    ts.f = pool;
    ts.f.words = pool.words + d.bloom_off;
    ts.f.mask = d.bloom_mask;
    return ts;
}

// Persistent-grid walks over a workgroup's tiles, in chunks of G
// consecutive entries (the chunk size, tp_config.chunk_tiles): workgroup i
// runs on XCD i mod NXCD (round-robin dispatch) and walks that XCD's share
// of the first-pass tile order (run_cursor), or the tiles in memory order
// (linear_run).  The grid is a multiple of NXCD.  Static schedule: every
// (grid/NXCD)-th chunk of the share, or every grid-th chunk in memory order.
// With a tile queue (SeqArgs.queue): a workgroup takes the next chunk from
// its share's counter (one per XCD; one in memory order) when it finishes
// one, and once that share is exhausted from the other XCDs' shares in
// turn, so the last chunks go to whichever workgroups are free.  The walk is
// the same for every thread of a workgroup; with a queue, every thread must
// call run_next (it synchronises the workgroup to share each claim).  Where
// there are too few tiles to go round, each is cut in parts instead
// (SeqArgs.parts_log2).
struct RunCursor {
    uint64_t c, end;
    uint32_t gi, G, step, ordered;
    uint32_t qx, qleft;  // queue: the share being walked, shares not yet exhausted
};

// One part of one tile: the workgroup's only entry.
__device__ __forceinline__ RunCursor part_cursor(const SeqArgs &a) {
    const uint64_t c = blockIdx.x >> a.parts_log2;
    return RunCursor{c, min(c + 1, a.n_tiles), 0, 1, gridDim.x, 0, 0, 0};
}

__device__ __forceinline__ RunCursor run_cursor(const SeqArgs &a, uint32_t G) {
    const uint32_t x = blockIdx.x % NXCD;
    if (a.parts_log2)
        return part_cursor(a);
    if (a.queue)  // nothing claimed yet: the first run_next claims
        return RunCursor{0, 0, G, G, 0, 1, x, NXCD};
    return RunCursor{a.xcd_start[x] + (uint64_t)(blockIdx.x / NXCD) * G, a.xcd_start[x + 1], 0,
                     G, gridDim.x / NXCD, 1, 0, 0};
}

__device__ __forceinline__ RunCursor linear_run(const SeqArgs &a, uint32_t G) {
    if (a.queue)
        return RunCursor{0, 0, G, G, 0, 0, 0, 1};
    return RunCursor{(uint64_t)blockIdx.x * G, a.n_tiles, 0, G, gridDim.x, 0, 0, 0};
}

// The workgroup's part of a tile, in eighths of it: steps [lo, hi).
struct Part {
    uint32_t lo, hi;
};
__device__ __forceinline__ Part tile_part(const SeqArgs &a) {
    static_assert(TILE / BLOCK == 8, "a tile is eight steps");
    const uint32_t n = 8u >> a.parts_log2, i = blockIdx.x & ((1u << a.parts_log2) - 1);
    return a.parts_log2 ? Part{i * n, i * n + n} : Part{0, 8};
}

// Next tile of the walk, or false at its end.
__device__ __forceinline__ bool run_next(const SeqArgs &a, RunCursor &rc, uint64_t *tile) {
    if (a.queue) {
        __shared__ uint32_t claimed;
        for (;;) {
            if (rc.gi < rc.G && rc.c + rc.gi < rc.end) {
                const uint64_t j = rc.c + rc.gi++;
                *tile = rc.ordered ? (uint64_t)a.tile_order[j] : j;
                return true;
            }
            if (!rc.qleft)
                return false;
            // claim the next chunk of share qx
            const uint64_t lo = rc.ordered ? a.xcd_start[rc.qx] : 0;
            const uint64_t hi = rc.ordered ? a.xcd_start[rc.qx + 1] : a.n_tiles;
            __syncthreads();  // every thread has read the last claim
            if (threadIdx.x == 0)
                claimed = atomicAdd(&a.queue[rc.qx], rc.G);
            __syncthreads();
            const uint64_t c = lo + claimed;
            if (c < hi) {
                rc.c = c;
                rc.end = hi;
                rc.gi = 0;
            } else {  // share exhausted: the next one
                rc.qx = rc.ordered ? (rc.qx + 1) % NXCD : 0;
                --rc.qleft;
                rc.gi = rc.G;
            }
        }
    }
    while (rc.c < rc.end) {
        if (rc.gi < rc.G && rc.c + rc.gi < rc.end) {
            const uint64_t j = rc.c + rc.gi++;
            *tile = rc.ordered ? (uint64_t)a.tile_order[j] : j;
            return true;
        }
        rc.c += (uint64_t)rc.step * rc.G;
        rc.gi = 0;
    }
    return false;
}

// Wave-wide ballot as a 64-bit mask (wave64).
__device__ __forceinline__ uint64_t ballot64(bool p) { return __ballot(p); }

// A per-set counter summed over the tiles a persistent workgroup walks.  Each
// thread keeps its part for the current set in a register; when the tile's
// set changes, and at the end, the workgroup adds the parts in LDS and issues
// one device atomic.  (Atomics on one address from every XCD serialise far
// from the CUs, so one per tile or per thread would dominate the kernel.)
// Every call must be reached by the whole workgroup with the same `set`.
struct SetSum {
    uint32_t set;
    unsigned long long v;
};

__device__ __forceinline__ SetSum setsum_begin() { return SetSum{~0u, 0ull}; }

__device__ __forceinline__ void setsum_flush(SetSum &s, unsigned long long *lds,
                                             unsigned long long *counter_of_set0,
                                             uint32_t stride_words) {
    if (s.set == ~0u)
        return;
    if (threadIdx.x == 0)
        *lds = 0;
    __syncthreads();
    if (s.v)
        atomicAdd(lds, s.v);
    __syncthreads();
    if (threadIdx.x == 0 && *lds)
        atomicAdd(counter_of_set0 + (uint64_t)s.set * stride_words, *lds);
    s.v = 0;
}

// Switch the sum to `set` (flushing the previous set's part when it differs).
__device__ __forceinline__ void setsum_switch(SetSum &s, uint32_t set, unsigned long long *lds,
                                              unsigned long long *counter_of_set0,
                                              uint32_t stride_words) {
    if (set != s.set) {
        setsum_flush(s, lds, counter_of_set0, stride_words);
        s.set = set;
    }
}

constexpr uint32_t SETCNT_STRIDE = sizeof(SetCounters) / sizeof(unsigned long long);

// ------------------------------------------------ binned schedules (LDS sort)

constexpr uint64_t BIN_NONE = ~0ull;  // no item (real items never have all bits set)

// Exclusive scan of the N counters cnt[] into start[] by NT threads
// (N / NT consecutive counters per thread, or one for the first N threads
// when N < NT); the total goes to *total.  Called by the whole workgroup;
// ends synchronised.
template <uint32_t N, uint32_t NT>
__device__ __forceinline__ void lds_scan(const uint32_t *cnt, uint32_t *start, uint32_t *wtot,
                                         uint32_t *total) {
    static_assert(NT % 64 == 0 && (N >= NT ? N % NT == 0 : NT % N == 0), "scan shape");
    constexpr uint32_t E = N >= NT ? N / NT : 1;
    const uint32_t t = threadIdx.x, lane = t & 63, wave = t >> 6;
    uint32_t c[E], sum = 0;
#pragma unroll
    for (uint32_t q = 0; q < E; ++q) {
        c[q] = t * E + q < N ? cnt[t * E + q] : 0;
        sum += c[q];
    }
    uint32_t x = sum;
#pragma unroll
    for (uint32_t d = 1; d < 64; d <<= 1) {
        const uint32_t y = __shfl_up(x, d, 64);
        if (lane >= d)
            x += y;
    }
    if (lane == 63)
        wtot[wave] = x;
    __syncthreads();
    uint32_t before = 0;
    for (uint32_t q = 0; q < wave; ++q)
        before += wtot[q];
    uint32_t e = before + x - sum;
#pragma unroll
    for (uint32_t q = 0; q < E; ++q) {
        if (t * E + q < N)
            start[t * E + q] = e;
        e += c[q];
    }
    if (t == NT - 1)
        *total = e;
    __syncthreads();
}

// Shared memory of a sort of NT * PER items into at most NB bins.
template <uint32_t NB, uint32_t NT, uint32_t PER, class I = uint32_t> struct BinSort {
    I srt[NT * PER];
    uint32_t cnt[NB];        // a bin's items of the batch, then its first place in the bin
    uint32_t start[NB + 1];  // a bin's first item in srt
    uint32_t wtot[NT / 64], total;
};

// Append a batch of items, PER per thread, to their bins: at[q] is bin << 14 |
// rank (the item's number in its bin, from an atomic add on sh.cnt), or ~0 for
// none.  The items are sorted by bin in LDS and a bin's items written as one
// run by a group of 2^lpb lanes; bin i has room for off(i+1) - off(i) items
// from out + off(i), of which cursor[i] are claimed.  direct(bin, item) takes
// an item without room, unless it equals the one before it in the run: items
// are idempotent, and a repetitive input's without room are mostly copies.
// sh.cnt is zero again on return.  Whole workgroup;
// ends synchronised.
template <uint32_t NB, uint32_t NT, uint32_t PER, class I, class Off, class Direct>
__device__ __forceinline__ void bin_append(BinSort<NB, NT, PER, I> &sh, const I (&item)[PER],
                                           const uint32_t (&at)[PER], uint32_t nb, uint32_t lpb,
                                           unsigned long long *cursor, Off off, I *out,
                                           Direct direct) {
    static_assert(NT * PER <= 1u << 14, "rank bits");
    constexpr uint32_t E = (NB + NT - 1) / NT;
    __syncthreads();  // every rank is taken
    // this thread's bins claim their room; the adds return while the scan runs
    uint64_t base[E];
#pragma unroll
    for (uint32_t e = 0; e < E; ++e) {
        const uint32_t bin = threadIdx.x * E + e, c = bin < nb ? sh.cnt[bin] : 0;
        base[e] = c ? atomicAdd(&cursor[bin], (unsigned long long)c) : 0;
    }
    lds_scan<NB, NT>(sh.cnt, sh.start, sh.wtot, &sh.total);
    if (threadIdx.x == 0)
        sh.start[NB] = sh.total;
#pragma unroll
    for (uint32_t e = 0; e < E; ++e)  // (a claim beyond 2^32 - 2^15 has no room anyhow)
        if (threadIdx.x * E + e < NB)
            sh.cnt[threadIdx.x * E + e] = (uint32_t)min(base[e], (uint64_t)0xFFFF7FFFu);
#pragma unroll
    for (uint32_t q = 0; q < PER; ++q)
        if (at[q] != ~0u)
            sh.srt[sh.start[at[q] >> 14] + (at[q] & 0x3FFFu)] = item[q];
    __syncthreads();
    const uint32_t l = threadIdx.x & ((1u << lpb) - 1);
    for (uint32_t bin = threadIdx.x >> lpb; bin < nb; bin += NT >> lpb) {
        const uint32_t s0 = sh.start[bin], n = sh.start[bin + 1] - s0, b0 = sh.cnt[bin];
        const uint64_t o = off(bin);
        const uint32_t room = (uint32_t)min(off(bin + 1) - o, (uint64_t)0xFFFF7FFFu);
        const uint32_t fit = b0 < room ? min(n, room - b0) : 0;
        for (uint32_t i = l; i < fit; i += 1u << lpb)
            out[o + b0 + i] = sh.srt[s0 + i];
        for (uint32_t i = fit + l; i < n; i += 1u << lpb)
            if (i == 0 || sh.srt[s0 + i - 1] != sh.srt[s0 + i])
                direct(bin, sh.srt[s0 + i]);
    }
    __syncthreads();
    for (uint32_t i = threadIdx.x; i < NB; i += NT)
        sh.cnt[i] = 0;
    __syncthreads();
}

// Lanes that write a bin's run: about as many as a batch has items per bin.
__device__ __forceinline__ uint32_t bin_lanes(uint32_t nb, uint32_t batch) {
    uint32_t lpb = 6;
    while (lpb > 3 && (nb << lpb) > batch)
        --lpb;
    return lpb;
}

}  // namespace tp
