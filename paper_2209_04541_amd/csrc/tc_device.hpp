// Device side of the block-list triangle count.
//
// PGAbB Section 3.6: for a block-list (A_ij, A_ik, A_jk) and each edge (u, v)
// of A_ij, the triangles closed inside the list are the common entries of
// row u of A_ik and row v of A_jk; the intersection may be list based or
// hash based.  Here one wavefront takes one work item of A_ij: a run of at
// most kSplitV entries v of a row u (stage A_ik[u], walk the A_jk[v]), or of
// entries u of a column v (stage A_jk[v], walk the A_ik[u]):
//   1. stage the shared list in the wave's LDS -- an open-addressing hash
//      table behind a bit filter, or a bitmap over stripe k's columns -- or
//      leave it in place for binary search when it is too long to stage;
//   2. walk the other lists as one flattened sequence: lane l takes element
//      base + l, so every 64-wide load is contiguous within a list and no
//      lane idles on short lists;
//   3. probe each element against the staged list and count hits in
//      registers; the caller reduces across the wave.
#pragma once

#include "graph.hpp"
#include "rules.hpp"
#include "wave.hpp"

namespace pgabb {

enum RowMode : int { kModeHash = 0, kModeSearch = 1, kModeBitmap = 2 };

// Hash and filter slots: Fibonacci hashing modulo 2^24.  A 24-bit multiply
// (full rate on CDNA, where 32-bit integer multiplies are quarter rate) by
// an odd constant near 0.618 * 2^24, keeping the top lg of its low 24 bits:
// slot = floor(frac(w * C / 2^24) * 2^lg).  Ids at or above 2^24 only
// collide more often (the table compares whole values).  __umul24 returns
// int here, so the product is taken as unsigned before the shift.
__device__ __forceinline__ uint32_t hash_slot(int32_t w, int shift, uint32_t mask) {
    return (static_cast<uint32_t>(__umul24(static_cast<uint32_t>(w), 0x9E3779u)) >> shift) & mask;
}

__device__ __forceinline__ uint32_t filter_slot(int32_t w, int fshift, uint32_t fmask) {
    return (static_cast<uint32_t>(__umul24(static_cast<uint32_t>(w), 0xC13FA9u)) >> fshift) & fmask;
}

// LDS split of a hash-mode wave region of LDS_WORDS words: a power-of-two
// table of kTableCap words and a membership filter of the rest.  The
// template sizes used are 320, 640, 1280, 2304 and 4352 words.
template <int LDS_WORDS>
struct HashLds {
    static constexpr int kTableCap = LDS_WORDS >= 4352 ? 4096
                                     : LDS_WORDS >= 2304 ? 2048
                                     : LDS_WORDS >= 1280 ? 1024
                                     : LDS_WORDS >= 640 ? 512
                                     : LDS_WORDS >= 320 ? 256 : 64;
    static constexpr int kFilterCap = LDS_WORDS - kTableCap;  // words
};

// How one item's staged list S is held, fixed before the walk.
struct Staging {
    int shift = 0, fshift = 0;  // hash and filter slot shifts (24 - lg)
    uint32_t tmask = 0;         // table size - 1
    uint32_t fmask = 0;         // filter bits - 1
    int words = 0, fwords = 0;  // table (or bitmap) and filter words
    int32_t *table = nullptr;   // hash table, after the filter
};

// Walked lists are read in segments of kSeg consecutive entries, one per lane
// and load: finding the list that holds an entry takes about 25 instructions
// per lane, which a segment shares among its entries, and the load is one 16
// byte access.  The last segment of a list may be partial; its load then
// reads past the list (at most kSeg - 1 words), so the arrays that lists lie
// in are allocated kSeg words longer.  Kernel ms, one entry per lane against
// segments (with the cut to `after` below): R-MAT scale 20 in 8 x 8 blocks
// 2.35 -> 1.75, in one block 4.48 -> 3.01, in 32 x 32 4.18 -> 2.79; scale 22
// in 8 x 8 13.8 -> 9.76; 777 small graphs 1.35 -> 0.94.  At 8 x 8 the vector
// units are then busy 56 % of the time and 10.7 GB cross from the fabric to
// the L2s (6 TB/s): the lists' lines bound it as much as the instructions.
typedef int32_t seg_t __attribute__((ext_vector_type(4), aligned(4)));

__device__ __forceinline__ int32_t segs_of(int32_t len) { return (len + kSeg - 1) / kSeg; }

// How many of the entries w (-1: none) are in the sorted list a[lo, hi), lo < hi.
// The entries' searches go side by side, so that their loads overlap: each step
// halves the range that an entry, if it is there, lies in.
__device__ __forceinline__ uint32_t sorted_hits(gptr<int32_t> a, int32_t lo, int32_t hi, const int32_t (&w)[kSeg]) {
    int32_t at[kSeg];
#pragma unroll
    for (int r = 0; r < kSeg; ++r) at[r] = lo;
    int32_t len = hi - lo;
    while (len > 1) {
        const int32_t half = len >> 1;
#pragma unroll
        for (int r = 0; r < kSeg; ++r) at[r] += a[at[r] + half - 1] < w[r] ? half : 0;
        len -= half;
    }
    uint32_t hits = 0;
#pragma unroll
    for (int r = 0; r < kSeg; ++r) hits += a[at[r]] == w[r] ? 1u : 0u;
    return hits;
}

// One load batch: UNROLL segments per lane, n[q] valid entries in each (none
// when n[q] <= 0).
template <int UNROLL>
struct SegBatch {
    seg_t v[UNROLL];
    int32_t n[UNROLL];
};

// Loads segments base + q * 64 + lane (q < UNROLL) of the flattened walk over
// the lists of one group of up to 64 lanes (lane l: wk_col[pb .. end), nseg
// segments from position pre of the walk), and for each the lane whose list
// holds it (src).  That lane is found without a search: every list that
// starts inside the batch writes its lane + 1 at its first position in `own`
// (64 * UNROLL words of the wave's LDS, zero between calls, and left zero),
// and a running maximum over the lanes fills the positions in between;
// `carry` (lane + 1 of the list holding the segment before the batch) starts
// at 0 for a new group.  Every call issues exactly UNROLL loads (past the
// end, of the first words of wk_col, which exist whenever a walk does), so
// the compiler can wait for one batch while the next is in flight; the
// entries past a list's end are masked when they are probed, not here, for
// the same reason.
template <int UNROLL>
__device__ __forceinline__ void walk_load(SegBatch<UNROLL> &B, int (&src)[UNROLL], int32_t base, int32_t total,
                                          int32_t pre, int32_t nseg, int32_t pb, int32_t end, uint32_t &carry,
                                          int32_t *__restrict__ own, gptr<int32_t> wk_col, int lane) {
    const int32_t p = pre - base;
    if (nseg > 0 && p >= 0 && p < UNROLL * kWave) own[p] = lane + 1;
    wave_lds_sync();
    uint32_t o[UNROLL];
#pragma unroll
    for (int q = 0; q < UNROLL; ++q) {
        o[q] = static_cast<uint32_t>(own[q * kWave + lane]);
        own[q * kWave + lane] = 0;
    }
    wave_lds_sync();
    const int32_t rel = pb - kSeg * pre;  // segment s of the walk starts at wk_col[rel + kSeg s] for the lane's list
#pragma unroll
    for (int q = 0; q < UNROLL; ++q) {
        const uint32_t sl = max(wave_max_scan_dpp(o[q]), carry);
        carry = __builtin_amdgcn_readlane(sl, kWave - 1);
        const int32_t s = base + q * kWave + lane;
        src[q] = static_cast<int>(sl) - 1;
        const int32_t at = __shfl(rel, src[q]) + kSeg * s;
        const int32_t left = __shfl(end, src[q]) - at;
        const bool inb = s < total;
        B.n[q] = inb ? left : 0;
        B.v[q] = *reinterpret_cast<const __attribute__((address_space(1))) seg_t *>(wk_col + (inb ? at : 0));
    }
}

// Items whose staged list has at most this many entries are walked together
// (tiny_items).
constexpr int kTinyCap = 4;

// Counts the items of the lanes in `m` (one task or graph, staged lists of
// at most kTinyCap entries; lane l: ids[b .. e) are its walked lists' ids and
// st_col[sb .. se) its staged list) in one walk instead of one after
// another.  The items' walked lists are flattened over the lanes 64 at a
// time, each list lane finding its item with the scattered lookup and taking
// the item's staged entries (held in registers, -2 padding no element
// matches); the lists' elements are then flattened over the lanes again and
// each is compared with its list's staged entries.  On hypersparse blocks an
// item walks a handful of entries, which a wave walking one item at a time
// spreads over a few of its lanes.
template <int UNROLL>
__device__ __forceinline__ uint32_t tiny_items(uint64_t m, int32_t b, int32_t e, int32_t sb, int32_t se,
                                               const int32_t *st_col_, const int32_t *ids_,
                                               const int32_t *wk_rptr_, const int32_t *wk_col_, int32_t *own,
                                               int lane) {
    const gptr<int32_t> st_col = as_global(st_col_), ids = as_global(ids_);
    const gptr<int32_t> wk_rptr = as_global(wk_rptr_), wk_col = as_global(wk_col_);
    const bool in = (m >> lane) & 1ull;
    int32_t s[kTinyCap];
#pragma unroll
    for (int t = 0; t < kTinyCap; ++t) s[t] = (in && t < se - sb) ? st_col[sb + t] : -2;
    const int32_t nl = in ? e - b : 0;  // walked lists of the lane's item
    const int32_t incl1 = wave_inclusive_scan(nl);
    const int32_t pre1 = incl1 - nl;
    const int32_t nlists = __builtin_amdgcn_readlane(incl1, kWave - 1);
    const int32_t idbase = b - pre1;  // list slot j of the item is ids[idbase + j]
    uint32_t cnt = 0;
    uint32_t carry1 = 0;
    for (int32_t j0 = 0; j0 < nlists; j0 += kWave) {
        // the item of list slot j0 + lane
        const int32_t p = pre1 - j0;
        if (nl > 0 && p >= 0 && p < kWave) own[p] = lane + 1;
        wave_lds_sync();
        const uint32_t o = static_cast<uint32_t>(own[lane]);
        own[lane] = 0;
        wave_lds_sync();
        const uint32_t il1 = max(wave_max_scan_dpp(o), carry1);
        carry1 = __builtin_amdgcn_readlane(il1, kWave - 1);
        const int il = static_cast<int>(il1) - 1;
        const int32_t j = j0 + lane;
        const int32_t ib = __shfl(idbase, il);
        int32_t ls[kTinyCap];
#pragma unroll
        for (int t = 0; t < kTinyCap; ++t) ls[t] = __shfl(s[t], il);
        int32_t pb = 0, len = 0;
        if (j < nlists) {
            const int32_t id = ids[ib + j];
            pb = wk_rptr[id];
            len = wk_rptr[id + 1] - pb;
        }
        // the segments of these lists, flattened over the lanes
        const int32_t nseg = segs_of(len);
        const int32_t incl = wave_inclusive_scan(nseg);
        const int32_t pre = incl - nseg;
        const int32_t total = __builtin_amdgcn_readlane(incl, kWave - 1);
        uint32_t carry = 0;
        for (int32_t base = 0; base < total; base += UNROLL * kWave) {
            SegBatch<UNROLL> B;
            int src[UNROLL];
            walk_load<UNROLL>(B, src, base, total, pre, nseg, pb, pb + len, carry, own, wk_col, lane);
#pragma unroll
            for (int q = 0; q < UNROLL; ++q) {
                int32_t sv[kTinyCap];
#pragma unroll
                for (int x = 0; x < kTinyCap; ++x) sv[x] = __shfl(ls[x], src[q]);
#pragma unroll
                for (int r = 0; r < kSeg; ++r) {
                    if (__ballot(r < B.n[q]) == 0) break;  // lists of a few entries
                    bool hit = false;
#pragma unroll
                    for (int x = 0; x < kTinyCap; ++x) hit |= B.v[q][r] == sv[x];
                    cnt += (hit && r < B.n[q]) ? 1u : 0u;
                }
            }
        }
    }
    return cnt;
}

// Items with small staged lists and few walked lists are walked together
// too (packed_items): staged lists of at most kPackS entries, at most
// kPackLists walked lists.
constexpr int kPackS = 64;
constexpr int kPackLists = 8;

// Staged entries that a pack may hold in a region of LDS_WORDS words (table
// load <= 1/2).
template <int LDS_WORDS>
constexpr int kPackEntries = HashLds<LDS_WORDS>::kTableCap / 2;

// Items of one pack over a stripe of `width` columns: the item's number and
// the entry share a 32-bit key.
__device__ __forceinline__ int pack_items(int32_t width) {
    return width < (1 << 26) ? kWave : 1 << (__clz(width) > 0 ? __clz(width) : 0);
}

// Counts the items of the lanes in `m` (one task; lane l: ids[b .. e) are
// its walked lists' ids, st_col[sb .. se) its staged list) in one walk: the
// items' staged lists go into one open-addressing table in the wave's LDS
// region behind a bit filter, as in tc_item_core, each entry keyed with its
// item's number (lane - first lane of m, below pack_items(width_k)); the
// walked lists are then flattened as in tiny_items and each entry probes with
// its list's item.  A key is never 0, the empty slot.  The used part of the
// region is zeroed: before the pack when hash staging left it (MODE hash),
// after it where bitmap staging expects zeros.
template <int MODE, int UNROLL, int LDS_WORDS>
__device__ __forceinline__ uint32_t packed_items(uint64_t m, int32_t b, int32_t e, int32_t sb, int32_t se,
                                                 const int32_t *st_col_, const int32_t *ids_,
                                                 const int32_t *wk_rptr_, const int32_t *wk_col_, int32_t width_k,
                                                 int32_t *__restrict__ lds, int32_t *own, int lane) {
    constexpr int FC = HashLds<LDS_WORDS>::kFilterCap;
    uint32_t *table = reinterpret_cast<uint32_t *>(lds) + FC;
    uint32_t *filter = reinterpret_cast<uint32_t *>(lds);
    const gptr<int32_t> st_col = as_global(st_col_), ids = as_global(ids_);
    const gptr<int32_t> wk_rptr = as_global(wk_rptr_), wk_col = as_global(wk_col_);
    const bool in = (m >> lane) & 1ull;
    const int first = __builtin_ctzll(m);
    const int kshift = width_k < (1 << 26) ? 26 : 32 - __clz(width_k);
    // ---- stage every item's list
    const int32_t ns = in ? se - sb : 0;
    const int32_t incls = wave_inclusive_scan(ns);
    const int32_t pres = incls - ns;
    const int32_t nsum = __builtin_amdgcn_readlane(incls, kWave - 1);
    int lg = 6;
    while ((1 << lg) < 2 * nsum) ++lg;  // at most kTableCap (nsum <= kPackEntries)
    int flg = 8;
    while ((1 << flg) < 16 * nsum && (1 << flg) < 32 * FC) ++flg;
    while ((1 << flg) > 32 * FC) --flg;
    const uint32_t tmask = (1u << lg) - 1u, fmask = (1u << flg) - 1u;
    const int shift = 24 - lg, fshift = 24 - flg;
    auto clear = [&]() {
        wave_lds_sync();
        for (int q = lane; q < (1 << lg); q += kWave) table[q] = 0u;
        for (int q = lane; q < (1 << flg) / 32; q += kWave) filter[q] = 0u;
        wave_lds_sync();
    };
    if (MODE != kModeBitmap) clear();
    const int32_t sbase = sb - pres;  // staged entry k of the item is st_col[sbase + k]
    uint32_t carry0 = 0;
    for (int32_t k0 = 0; k0 < nsum; k0 += kWave) {
        const int32_t p = pres - k0;
        if (ns > 0 && p >= 0 && p < kWave) own[p] = lane + 1;
        wave_lds_sync();
        const uint32_t o = static_cast<uint32_t>(own[lane]);
        own[lane] = 0;
        wave_lds_sync();
        const uint32_t il1 = max(wave_max_scan_dpp(o), carry0);
        carry0 = __builtin_amdgcn_readlane(il1, kWave - 1);
        const int il = static_cast<int>(il1) - 1;
        const int32_t k = k0 + lane;
        const int32_t base_k = __shfl(sbase, il);
        if (k < nsum) {
            const int32_t v = st_col[base_k + k];
            const uint32_t item = static_cast<uint32_t>(il - first);
            const uint32_t key = ((item << kshift) | static_cast<uint32_t>(v)) + 1u;
            const int32_t hv = v + static_cast<int32_t>(item) * 0x3C6EF35;  // the item enters the hash
            const uint32_t f = filter_slot(hv, fshift, fmask);
            atomicOr(&filter[f >> 5], 1u << (f & 31));
            uint32_t h = hash_slot(hv, shift, tmask);
            while (atomicCAS(&table[h], 0u, key) != 0u) h = (h + 1) & tmask;
        }
    }
    wave_lds_sync();
    // ---- the walked lists, flattened as in tiny_items
    const int32_t nl = in ? e - b : 0;
    const int32_t incl1 = wave_inclusive_scan(nl);
    const int32_t pre1 = incl1 - nl;
    const int32_t nlists = __builtin_amdgcn_readlane(incl1, kWave - 1);
    const int32_t idbase = b - pre1;
    uint32_t cnt = 0;
    uint32_t carry1 = 0;
    for (int32_t j0 = 0; j0 < nlists; j0 += kWave) {
        const int32_t p = pre1 - j0;
        if (nl > 0 && p >= 0 && p < kWave) own[p] = lane + 1;
        wave_lds_sync();
        const uint32_t o = static_cast<uint32_t>(own[lane]);
        own[lane] = 0;
        wave_lds_sync();
        const uint32_t il1 = max(wave_max_scan_dpp(o), carry1);
        carry1 = __builtin_amdgcn_readlane(il1, kWave - 1);
        const int il = static_cast<int>(il1) - 1;  // the item of list slot j0 + lane
        const int32_t j = j0 + lane;
        const int32_t ib = __shfl(idbase, il);
        int32_t pb = 0, len = 0;
        if (j < nlists) {
            const int32_t id = ids[ib + j];
            pb = wk_rptr[id];
            len = wk_rptr[id + 1] - pb;
        }
        const int32_t nseg = segs_of(len);
        const int32_t incl = wave_inclusive_scan(nseg);
        const int32_t pre = incl - nseg;
        const int32_t total = __builtin_amdgcn_readlane(incl, kWave - 1);
        uint32_t carry = 0;
        for (int32_t base = 0; base < total; base += UNROLL * kWave) {
            SegBatch<UNROLL> B;
            int src[UNROLL];
            walk_load<UNROLL>(B, src, base, total, pre, nseg, pb, pb + len, carry, own, wk_col, lane);
#pragma unroll
            for (int q = 0; q < UNROLL; ++q) {
                const uint32_t item = static_cast<uint32_t>(__shfl(il, src[q]) - first);  // the segment's item
                const int32_t mix = static_cast<int32_t>(item) * 0x3C6EF35;
                bool maybe[kSeg];
#pragma unroll
                for (int r = 0; r < kSeg; ++r) {
                    const uint32_t f = filter_slot(B.v[q][r] + mix, fshift, fmask);
                    maybe[r] = r < B.n[q] && ((filter[f >> 5] >> (f & 31)) & 1u) != 0u;
                }
#pragma unroll
                for (int r = 0; r < kSeg; ++r) {
                    bool go = maybe[r];
                    const uint32_t key = ((item << kshift) | static_cast<uint32_t>(B.v[q][r])) + 1u;
                    uint32_t h = hash_slot(B.v[q][r] + mix, shift, tmask);
                    while (__ballot(go) != 0) {
                        const uint32_t sv = table[h];
                        cnt += (go && sv == key) ? 1u : 0u;
                        go = go && sv != 0u && sv != key;
                        h = (h + 1) & tmask;
                    }
                }
            }
        }
    }
    if (MODE == kModeBitmap) clear();
    return cnt;
}

// Adds to cnt the hits of the entries of batch B against S.  Hash probes are
// predicated: a wave-uniform loop runs while any lane is still searching,
// with no per-lane branches.  `own` (see walk_load) holds zeros here: a
// bitmap probe of an entry past its list's end reads own[0] instead, which
// saves masking its result.
template <int PM, int UNROLL>
__device__ __forceinline__ void probe_batch(const SegBatch<UNROLL> &B, uint32_t &cnt,
                                            int32_t *__restrict__ lds, const Staging &sg, gptr<int32_t> st_col,
                                            int32_t sb, int32_t se, int32_t wbase, int32_t own_bit, int lane) {
#pragma unroll
    for (int q = 0; q < UNROLL; ++q) {
        if (PM == kModeBitmap) {
#pragma unroll
            for (int r = 0; r < kSeg; ++r) {
                const int32_t wl = r < B.n[q] ? B.v[q][r] - wbase : own_bit;
                cnt += (static_cast<uint32_t>(lds[wl >> 5]) >> (wl & 31)) & 1u;
            }
        } else if (PM == kModeHash) {
            int32_t w[kSeg];
            uint32_t bit[kSeg];
#pragma unroll
            for (int r = 0; r < kSeg; ++r) {
                w[r] = r < B.n[q] ? B.v[q][r] : -1;
                const uint32_t f = filter_slot(w[r], sg.fshift, sg.fmask);  // in range for any w
                bit[r] = (static_cast<uint32_t>(lds[f >> 5]) >> (f & 31)) & 1u;
            }
#pragma unroll
            for (int r = 0; r < kSeg; ++r) {
                bool go = (w[r] >= 0) & (bit[r] != 0u);
                uint32_t h = hash_slot(w[r], sg.shift, sg.tmask);
                uint32_t hit = 0;
                while (__ballot(go) != 0) {
                    const int32_t sv = sg.table[h];
                    hit |= (go && sv == w[r]) ? 1u : 0u;
                    go = go && sv >= 0 && sv != w[r];
                    h = (h + 1) & sg.tmask;
                }
                cnt += hit;
            }
        } else {
            // the segments' entries dealt one per lane again, through the region
            // (no list is staged there): neighbouring lanes then search for
            // neighbouring entries and read the same lines (eight complete
            // graphs of 900 vertices, staged rows searched, row walk: 5.4 ms with
            // a segment's searches one after the other, 5.2 side by side, 2.8
            // with this; one entry per lane 4.3)
            wave_lds_sync();
#pragma unroll
            for (int r = 0; r < kSeg; ++r) lds[kSeg * lane + r] = r < B.n[q] ? B.v[q][r] : -1;
            wave_lds_sync();
            int32_t w[kSeg];
#pragma unroll
            for (int r = 0; r < kSeg; ++r) w[r] = lds[r * kWave + lane];
            cnt += sorted_hits(st_col, sb, se, w);
        }
    }
}

// A group's lists are cut to their entries above `after` when they have at
// least this many segments each on average: half of the walk goes, for a
// search of about ten dependent loads per group.  (R-MAT scale 20, kernel ms
// at 3 / 6 / 12 segments: 8 x 8 blocks 1.79 / 1.78 / 1.77, one block 3.68 /
// 3.75 / 3.83.)
constexpr int32_t kAfterSegs = 6;

// The walk of one item once the staging kind PM is known: groups of up to 64
// walked lists; for the first group the first batch is loaded before S is
// staged, and every later batch loads while the previous one is probed.
// S is staged when the first non-empty group comes (`staged` tells the
// caller whether it was), so an item whose lists are all empty stages
// nothing.  after >= 0: no entry up to `after` is in S (see tc_item_core).
template <int PM, int UNROLL>
__device__ __forceinline__ uint32_t walk_item(Staging stg, gptr<int32_t> st_col, int32_t sb,
                                              int32_t se, gptr<int32_t> wk_rptr,
                                              gptr<int32_t> wk_col, gptr<int32_t> ids, int32_t ib,
                                              int32_t ie, int32_t g0, int32_t gn, int32_t id,
                                              int32_t *__restrict__ lds, int32_t wbase, int lane,
                                              bool &staged, int32_t *__restrict__ own, int32_t own_bit,
                                              int32_t after) {
    uint32_t cnt = 0;
    for (;;) {  // groups of up to 64 walked lists
        int32_t pb = 0, end = 0;
        if (lane < gn) {
            pb = wk_rptr[id];
            end = wk_rptr[id + 1];
        }
        int32_t nseg = segs_of(end - pb);
        int32_t incl = wave_inclusive_scan(nseg);
        int32_t total = __builtin_amdgcn_readlane(incl, kWave - 1);
        if (after >= 0 && total >= kAfterSegs * gn) {
            int32_t hi = end;
            while (__ballot(pb < hi) != 0) {  // pb: first entry above after
                const int32_t mid = halfway(pb, hi);
                if (pb < hi) {
                    if (wk_col[mid] <= after) pb = mid + 1;
                    else hi = mid;
                }
            }
            nseg = segs_of(end - pb);
            incl = wave_inclusive_scan(nseg);
            total = __builtin_amdgcn_readlane(incl, kWave - 1);
        }
        const int32_t pre = incl - nseg;
        uint32_t carry = 0;
        SegBatch<UNROLL> B;
        int src[UNROLL];
        walk_load<UNROLL>(B, src, 0, total, pre, nseg, pb, end, carry, own, wk_col, lane);

        if (!staged && total > 0) {
            staged = true;
            if (PM == kModeHash) {
                for (int q = lane; q < stg.words; q += kWave) stg.table[q] = -1;
                for (int q = lane; q < stg.fwords; q += kWave) lds[q] = 0;
                wave_lds_sync();
                for (int32_t idx = sb + lane; idx < se; idx += kWave) {
                    const int32_t x = st_col[idx];
                    const uint32_t f = filter_slot(x, stg.fshift, stg.fmask);
                    atomicOr(reinterpret_cast<uint32_t *>(&lds[f >> 5]), 1u << (f & 31));
                    uint32_t h = hash_slot(x, stg.shift, stg.tmask);
                    while (atomicCAS(&stg.table[h], -1, x) != -1) h = (h + 1) & stg.tmask;
                }
                wave_lds_sync();
            } else if (PM == kModeBitmap) {
                for (int32_t idx = sb + lane; idx < se; idx += kWave) {
                    const int32_t x = st_col[idx] - wbase;
                    atomicOr(reinterpret_cast<uint32_t *>(&lds[x >> 5]), 1u << (x & 31));
                }
                wave_lds_sync();
            }
        }

        // the last batch is probed after the loop, with no further one loading
        for (int32_t base = UNROLL * kWave; base < total; base += UNROLL * kWave) {
            SegBatch<UNROLL> Bn;
            walk_load<UNROLL>(Bn, src, base, total, pre, nseg, pb, end, carry, own, wk_col, lane);
            probe_batch<PM, UNROLL>(B, cnt, lds, stg, st_col, sb, se, wbase, own_bit, lane);
            B = Bn;
        }
        if (total > 0) probe_batch<PM, UNROLL>(B, cnt, lds, stg, st_col, sb, se, wbase, own_bit, lane);

        g0 += kWave;
        if (g0 >= ie) break;
        gn = min(ie - g0, kWave);
        id = lane < gn ? ids[g0 + lane] : 0;
    }
    return cnt;
}

// One work item of a block-list: the staged list S = st_col[sb .. se) (the
// row srow of the staging block) and the walked lists L_x = wk_col[wk_rptr[x] ..
// wk_rptr[x + 1]) for the ids x in ids[ib .. ie).  Returns, per lane, part of
// sum_x |S & L_x| (the sum over lanes is the item's count).  With the edge
// block walked by rows this is S = A_ik[u], L_v = A_jk[v] for v in A_ij[u];
// walked by columns, S = A_jk[v], L_u = A_ik[u] for u with (u, v) in A_ij.
// `lds` holds LDS_WORDS int32 words private to the wave, followed by 64 *
// UNROLL more, zero on entry and left zero (the walk's list positions).
// Column ids of both lists lie in [wbase, wbase + width_k).  after >= 0: every
// entry of S exceeds `after`, so the lists' entries up to it may be skipped.
// Every lane of the wave must call this with the same arguments.
//
// Hash staging: S goes into an open-addressing table (load <= 2/3) and into
// a bit filter with about eight bits per entry; a probe reads the filter
// first, so most misses -- nine in ten probes on skewed graphs -- cost one
// LDS read.
//
// The walk issues many instructions per element, so its code keeps the
// instruction count low: the staging kind is fixed per item outside the
// element loop, hash probes are predicated, and loads go through global
// views.  It is also latency bound per item (each step's addresses come from
// the previous step's loads), so independent loads are issued together: the
// ids of the walked lists with the bounds of S, the first chunks of the walk
// before S is staged, and every later chunk before the previous one is
// probed.
template <int MODE, int LDS_WORDS, int UNROLL = 1>
__device__ __forceinline__ uint32_t tc_item_core(const int32_t *__restrict__ st_col_, int32_t sb, int32_t se,
                                                 const int32_t *__restrict__ wk_rptr_,
                                                 const int32_t *__restrict__ wk_col_,
                                                 const int32_t *__restrict__ ids_, int32_t ib, int32_t ie,
                                                 int32_t width_k, int32_t *__restrict__ lds, int32_t wbase = 0,
                                                 int32_t after = -1) {
    const int lane = lane_id();
    static_assert(LDS_WORDS >= kSeg * kWave, "a batch's entries fit the region");
    int32_t *own = lds + LDS_WORDS;
    constexpr int32_t own_bit = 32 * LDS_WORDS;
    if (ib >= ie) return 0u;
    const gptr<int32_t> st_col = as_global(st_col_);
    const gptr<int32_t> wk_rptr = as_global(wk_rptr_), wk_col = as_global(wk_col_);
    const gptr<int32_t> ids = as_global(ids_);
    const int32_t gn = min(ie - ib, kWave);
    const int32_t id = lane < gn ? ids[ib + lane] : 0;
    const int32_t slen = se - sb;
    if (slen == 0) return 0u;

    // ---- choose how S is held
    int mode = MODE;
    Staging stg;
    if (mode == kModeBitmap) {
        stg.words = (width_k + 31) >> 5;
        if (stg.words > LDS_WORDS) mode = kModeHash;
    }
    if (mode == kModeHash) {
        constexpr int TC = HashLds<LDS_WORDS>::kTableCap;
        constexpr int FC = HashLds<LDS_WORDS>::kFilterCap;
        int lg = 6;
        while ((1 << lg) * 2 < 3 * slen) ++lg;
        if ((1 << lg) > TC || FC < 2) {
            mode = kModeSearch;
        } else {
            stg.words = 1 << lg;
            stg.shift = 24 - lg;
            stg.tmask = static_cast<uint32_t>(stg.words - 1);
            int flg = 8;  // filter bits: a power of two >= 8 * slen, >= 256
            while ((1 << flg) < 8 * slen && (1 << flg) < 32 * FC) ++flg;
            while ((1 << flg) > 32 * FC) --flg;
            stg.fwords = (1 << flg) >> 5;
            stg.fshift = 24 - flg;
            stg.fmask = static_cast<uint32_t>((1 << flg) - 1);
            stg.table = lds + FC;
        }
    }

    uint32_t cnt;
    bool staged = false;
    if (mode == kModeHash)
        cnt = walk_item<kModeHash, UNROLL>(stg, st_col, sb, se, wk_rptr, wk_col, ids, ib, ie, ib, gn, id,
                                           lds, wbase, lane, staged, own, own_bit, after);
    else if (mode == kModeBitmap)
        cnt = walk_item<kModeBitmap, UNROLL>(stg, st_col, sb, se, wk_rptr, wk_col, ids, ib, ie, ib, gn, id,
                                             lds, wbase, lane, staged, own, own_bit, after);
    else
        cnt = walk_item<kModeSearch, UNROLL>(stg, st_col, sb, se, wk_rptr, wk_col, ids, ib, ie, ib, gn, id,
                                             lds, wbase, lane, staged, own, own_bit, after);

    // ---- leave the LDS clean for the next row of this wave
    if (!staged) return cnt;
    if (mode == kModeBitmap) {
        wave_lds_sync();
        for (int32_t idx = sb + lane; idx < se; idx += kWave) lds[(st_col[idx] - wbase) >> 5] = 0;
        wave_lds_sync();
    } else if (mode == kModeHash) {
        wave_lds_sync();
        if (MODE == kModeBitmap) {
            // a bitmap kernel expects zeroed LDS between rows: clear the
            // filter and table words this item used
            constexpr int FC = HashLds<LDS_WORDS>::kFilterCap;
            for (int q = lane; q < stg.fwords; q += kWave) lds[q] = 0;
            for (int q = lane; q < stg.words; q += kWave) lds[FC + q] = 0;
            wave_lds_sync();
        }
    } else if (MODE == kModeBitmap) {
        wave_lds_sync();
        for (int q = lane; q < kSeg * kWave; q += kWave) lds[q] = 0;  // (the searched entries)
        wave_lds_sync();
    }
    return cnt;
}

}  // namespace pgabb
