// Partition phase: symmetric rectilinear 2-D cut of the oriented CSR into a
// p x p grid of blocks, block storage, and the block-list (task) table.
//
// PGAbB Section 4.3 (symmetric two-dimensional partitioning: one cut vector
// for rows and columns; block ids in row-major order; per-block CSR with
// rearranged local ids) and Section 3.6 (block-lists (A_ij, A_ik, A_jk) of
// the two-dimensional triangle count).  With vertices ranked in ascending
// degree and edges oriented from lower to higher rank, only blocks with
// i <= j hold entries, and a triangle with ranks a < b < c lies in the task
// (stripe(a), stripe(b), stripe(c)), so the tasks are the triples
// i <= j <= k whose three blocks are non-empty.  Tasks are weighted by their
// edge count (the paper's default estimate) and sorted heaviest first
// (Section 4.1).
#include <algorithm>
#include <chrono>
#include <numeric>

#include "common.hpp"
#include "graph.hpp"
#include "wave.hpp"

namespace pgabb {

namespace {

constexpr int B = 256;
constexpr int kMaxP = 64;

struct CutTable {
    int32_t p;
    int32_t c[kMaxP + 1];
    int32_t base[kMaxP];
};

// The cut table of nnz-balanced cuts, built on the device (one workgroup):
// cut s is the first row x whose CSR offset reaches s * m' / p, and stripe
// s's dense row range starts at max(cut s, lowest) (clamped to the stripe).
__global__ __launch_bounds__(B) void k_nnz_cut_table(const int64_t *__restrict__ row_off, int32_t n,
                                                     int64_t m, int32_t p, int32_t lowest,
                                                     CutTable *__restrict__ ct) {
    __shared__ int32_t s_c[kMaxP + 1];
    for (int32_t s = threadIdx.x; s <= p; s += B) {
        int32_t c;
        if (s == 0) {
            c = 0;
        } else if (s == p) {
            c = n;
        } else {
            // smallest x in [0, n] with row_off[x] * p >= s * m
            int64_t lo = 0, hi = n;
            const int64_t target = static_cast<int64_t>(s) * m;  // < 2^38 for m' < 2^32
            while (lo < hi) {
                const int64_t mid = (lo + hi) >> 1;
                if (row_off[mid] * p >= target) hi = mid;
                else lo = mid + 1;
            }
            c = static_cast<int32_t>(lo);
        }
        s_c[s] = c;
        ct->c[s] = c;
    }
    __syncthreads();
    for (int32_t s = threadIdx.x; s < p; s += B) ct->base[s] = min(max(s_c[s], lowest), s_c[s + 1]);
    if (threadIdx.x == 0) ct->p = p;
}

// First index in [lo, hi) whose column is >= c (hi when none).
__device__ __forceinline__ int64_t first_at_least(const int32_t *__restrict__ col, int64_t lo,
                                                  int64_t hi, int32_t c) {
    while (lo < hi) {
        const int64_t mid = (lo + hi) >> 1;
        if (col[mid] < c) lo = mid + 1;
        else hi = mid;
    }
    return lo;
}

// Stripe of x from cuts held in LDS (largest s < p with c[s] <= x).
__device__ __forceinline__ int32_t stripe_lds(int32_t x, const int32_t *c, int32_t p) {
    int32_t lo = 0, hi = p - 1;
    while (lo < hi) {
        const int32_t mid = (lo + hi + 1) >> 1;
        if (c[mid] <= x) lo = mid;
        else hi = mid - 1;
    }
    return lo;
}

// Last row in [lo, hi) that starts at or before entry e (row_off[lo] <= e).
__device__ __forceinline__ int32_t row_search(const int64_t *__restrict__ row_off, int32_t lo, int32_t hi, int64_t e) {
    while (hi - lo > 1) {
        const int32_t mid = lo + ((hi - lo) >> 1);
        if (row_off[mid] <= e) lo = mid;
        else hi = mid;
    }
    return lo;
}

// The same over all n rows, 64 samples a step, by the whole wave.
__device__ __forceinline__ int32_t row_search_wave(const int64_t *__restrict__ row_off, int32_t n, int64_t e) {
    int32_t lo = 0, hi = n;
    while (hi - lo > 1) {
        const int32_t step = (hi - lo - 1) / kWave + 1;
        const int64_t at = lo + static_cast<int64_t>(lane_id()) * step;
        const uint64_t below = __ballot(at < hi && row_off[at < hi ? at : lo] <= e);
        lo += (__popcll(below) - 1) * step;
        if (step < hi - lo) hi = lo + step;
    }
    return lo;
}

// The passes over the entries give every workgroup the same number of
// consecutive entries, whatever the rows' lengths: a row a thread or a wave
// waits for the longest one, which took two launches (short rows flattened 64
// to a wave, rows over 64 entries in pieces) of 30 to 80 us each, also where
// the graph was small.  Partition into 8 x 8 blocks, before and now: R-MAT scale
// 12 490 -> 310 us, 16 550 -> 400, 20 1460 -> 1245, 21 2540 -> 2280;
// Erdos-Renyi, 300 K vertices of even rows, 580 -> 585 (into 4 x 4 545 -> 575).
// Tiles of 4 B / 8 B / 16 B entries: scale 16 365 / 400 / 515 us, scale 21 2615
// / 2270 / 2325.
constexpr int kTile = 8 * B;  // entries of a workgroup
// Up to this many rows are marked at their first entries; a tile that spans
// more (a stretch of empty rows) looks its entries' rows up.
constexpr int32_t kMarkRows = 4 * kTile;

struct Tile {
    int64_t t0;        // entries [t0, t0 + count)
    int32_t count;
    int32_t r0;        // row of the first entry
    bool starts, ends; // the first entry starts its row, the last one ends its own
};

// first[t]: the row of tile t's first entry; one more for the last entry.  A
// wave finds each.  Passes over more than kTableTiles tiles, whose workgroups
// come in several rounds, take them from there; in smaller ones two waves of
// each workgroup search (partition of R-MAT scale 16 / 20 / 21, 430 / 7,700 /
// 15,400 tiles, into 8 x 8 blocks: 419 / 1249 / 2287 us with the table, 400 /
// 1289 / 2465 without).
constexpr unsigned kTableTiles = 2048;
__global__ __launch_bounds__(B) void k_tile_first(const int64_t *__restrict__ row_off, int32_t n, int64_t m,
                                                  int64_t tiles, int32_t *__restrict__ first) {
    const int64_t t = (static_cast<int64_t>(blockIdx.x) * B + threadIdx.x) / kWave;
    if (t > tiles) return;
    const int32_t r = row_search_wave(row_off, n, min(t * kTile, m - 1));
    if (lane_id() == 0) first[t] = r;
}

// The rows of tile number `tile`: rows[i] is the row of entry t0 + i, relative
// to r0.  Every thread of the workgroup calls it; without `first`, two waves
// search.
__device__ __forceinline__ Tile tile_rows(const int64_t *__restrict__ row_off, int32_t n, int64_t m, int64_t tile,
                                          const int32_t *__restrict__ first, int32_t *rows) {
    __shared__ int32_t s_row[2];
    __shared__ uint32_t s_max[B / kWave];
    const int tid = threadIdx.x, w = tid / kWave, lane = lane_id();
    Tile t;
    t.t0 = tile * kTile;
    t.count = static_cast<int32_t>(min(m - t.t0, static_cast<int64_t>(kTile)));
    if (!first && w < 2) {
        const int32_t r = row_search_wave(row_off, n, min(t.t0 + w * kTile, m - 1));
        if (lane == 0) s_row[w] = r;
    }
    for (int i = tid; i < kTile; i += B) rows[i] = 0;
    __syncthreads();
    // (r1: the row of the entry after the tile)
    t.r0 = first ? first[tile] : s_row[0];
    const int32_t r1 = first ? first[tile + 1] : s_row[1], nr = r1 - t.r0;
    t.starts = row_off[t.r0] == t.t0;
    if (nr <= kMarkRows) {
        for (int32_t q = 1 + tid; q <= nr; q += B) {
            const int64_t e0 = row_off[t.r0 + q];
            // (empty rows share a start)
            if (row_off[t.r0 + q + 1] > e0 && e0 - t.t0 < t.count) rows[e0 - t.t0] = q;
        }
        __syncthreads();
        // every entry belongs to the last row marked at or before it
        uint32_t v[kTile / B], top = 0;
#pragma unroll
        for (int i = 0; i < kTile / B; ++i) {
            top = max(top, static_cast<uint32_t>(rows[tid * (kTile / B) + i]));
            v[i] = top;
        }
        const uint32_t incl = wave_max_scan_dpp(top);
        const uint32_t up = __shfl_up(incl, 1);
        if (lane == kWave - 1) s_max[w] = incl;
        __syncthreads();
        uint32_t before = lane ? up : 0u;
        for (int q = 0; q < w; ++q) before = max(before, s_max[q]);
#pragma unroll
        for (int i = 0; i < kTile / B; ++i) rows[tid * (kTile / B) + i] = static_cast<int32_t>(max(v[i], before));
    } else {
        int32_t r = t.r0;
        for (int i = tid * (kTile / B); i < min((tid + 1) * (kTile / B), t.count); ++i) {
            r = row_search(row_off, r, r1 + 1, t.t0 + i);
            rows[i] = r - t.r0;
        }
    }
    __syncthreads();
    t.ends = row_off[t.r0 + rows[t.count - 1] + 1] == t.t0 + t.count;
    return t;
}

// Calls f(x, e, y) for every entry e = (x, y) of the workgroup's tile.
template <class F>
__device__ __forceinline__ void for_entries(const int64_t *__restrict__ row_off, const int32_t *__restrict__ col,
                                            int32_t n, int64_t m, const int32_t *__restrict__ first, F f) {
    __shared__ int32_t rows[kTile];
    const Tile t = tile_rows(row_off, n, m, blockIdx.x, first, rows);
    for (int i = threadIdx.x; i < t.count; i += B) f(t.r0 + rows[i], t.t0 + i, col[t.t0 + i]);
}

// Stripe look-up of many entries: seven thresholds in registers split the
// stripes into eight groups; more than eight stripes leave up to three steps of
// search in LDS.  (With all steps in LDS, and the entries' neighbours read
// there, a pass over R-MAT scale 20 in 8 x 8 blocks took 88 us instead of 73;
// what is left is bound by instructions, some 100 for 64 entries.)
struct Stripes {
    const int32_t *c;
    int32_t p, per;  // stripes of a group
    int32_t t[7];
    __device__ __forceinline__ Stripes(const int32_t *cuts, int32_t np) : c(cuts), p(np), per((np + 7) / 8) {
#pragma unroll
        for (int k = 0; k < 7; ++k)
            t[k] = __builtin_amdgcn_readfirstlane((k + 1) * per < np ? cuts[(k + 1) * per] : INT32_MAX);
    }
    __device__ __forceinline__ int32_t of(int32_t y) const {
        int32_t g = 0;
#pragma unroll
        for (int k = 0; k < 7; ++k) g += y >= t[k];
        if (per == 1) return g;
        int32_t lo = g * per, hi = min(lo + per, p) - 1;
        while (lo < hi) {
            const int32_t mid = (lo + hi + 1) >> 1;
            if (c[mid] <= y) lo = mid;
            else hi = mid - 1;
        }
        return lo;
    }
};

// x of the lane before (wave_shr:1); lane 0 takes `first`.
__device__ __forceinline__ int32_t lane_before(int32_t x, int32_t first) {
    return __builtin_amdgcn_update_dpp(first, x, 0x138, 0xf, 0xf, false);
}

// Calls f(x, si, j, e, y, at, last) for every entry e = (x, y) of the
// workgroup's tiles: si and j are the stripes of x and y, at the place of e in
// its run (row x, column stripe j), last whether e ends the run.  Every lane
// calls it; c: the cuts, in LDS.  A wave takes 512 consecutive entries, 64 at
// a time, and marks in one ballot the entries that begin a run, up to and
// including the one after the 64: an entry's run began at the mark before it,
// in the 64 or earlier ones, or, once per wave, where a search of the row finds
// it, and an entry ends its run if a mark follows.
template <class F>
__device__ __forceinline__ void for_runs(const int64_t *__restrict__ row_off, const int32_t *__restrict__ col,
                                         int32_t n, int64_t m, const int32_t *__restrict__ first, const int32_t *c,
                                         int32_t p, F f) {
    __shared__ int32_t rows[kTile];
    const int lane = lane_id();
    const uint64_t le_mask = ~0ull >> (kWave - 1 - lane);
    constexpr int kPart = kTile / (B / kWave);
    const Stripes stripes(c, p);
    for (int64_t tile = blockIdx.x; tile * kTile < m; tile += gridDim.x) {
        const Tile t = tile_rows(row_off, n, m, tile, first, rows);
        const int i0 = static_cast<int>(threadIdx.x / kWave) * kPart, i1 = min(i0 + kPart, t.count);
        // rows of one stripe, as nearly everywhere: no look-up per entry
        const int32_t si0 = stripes.of(t.r0), r_end = rows[t.count - 1];
        const bool same = t.r0 + r_end < c[si0 + 1];
        // row and column stripe of entry t0 + i, the one after the tile included
        // (row -1: it begins a row, whatever its number)
        auto row_of = [&](int i) { return i < t.count ? rows[i] : t.ends ? -1 : r_end; };
        auto col_of = [&](int i) { return i <= i1 && t.t0 + i < m ? col[t.t0 + i] : 0; };
        if (i0 < i1) {
            // the entry before the wave's first
            int32_t rp = i0 ? rows[i0 - 1] : t.starts ? -1 : 0;
            int32_t jp = t.t0 + i0 ? stripes.of(col[t.t0 + i0 - 1]) : 0;
            int32_t y = col_of(i0 + lane), r = row_of(min(i0 + lane, i1)), j = stripes.of(y);
            // first entry of the run that the 64 begin in, relative to t0
            int32_t carry = INT32_MAX;
            for (int base = i0; base < i1; base += kWave) {
                const int i = base + lane;
                const int32_t yn = col_of(i + kWave), rn = row_of(min(i + kWave, i1)), jn = stripes.of(yn);
                const int32_t rb = lane_before(r, rp), jb = lane_before(j, jp);  // (on every lane)
                const uint64_t marks = __ballot((rb != r) | (jb != j));
                rp = __builtin_amdgcn_readlane(r, kWave - 1);
                jp = __builtin_amdgcn_readlane(j, kWave - 1);
                const bool more = __builtin_amdgcn_readlane(rn, 0) != rp || __builtin_amdgcn_readlane(jn, 0) != jp;
                const uint64_t ends = (marks >> 1) | (static_cast<uint64_t>(more) << (kWave - 1));
                if (carry == INT32_MAX && !(marks & 1)) {  // the wave's first entry lies inside a run
                    const int32_t j0 = __builtin_amdgcn_readfirstlane(j);
                    carry = static_cast<int32_t>(
                        first_at_least(col, row_off[t.r0 + rows[i0]], t.t0 + i0, c[j0]) - t.t0);
                }
                const uint64_t mine = marks & le_mask;
                const int32_t lo = mine ? base + (63 - __clzll(static_cast<long long>(mine))) : carry;
                if (i < i1) {
                    const int32_t x = t.r0 + r;
                    f(x, same ? si0 : stripes.of(x), j, t.t0 + i, y, i - lo, ((ends >> lane) & 1) != 0);
                }
                if (marks) carry = base + (63 - __clzll(static_cast<long long>(marks)));
                y = yn;
                r = rn;
                j = jn;
            }
        }
        __syncthreads();  // before the next tile's rows are marked
    }
}

// Index of the stripe pair {a, b} among the p (p + 1) / 2 unordered pairs.
__device__ __forceinline__ int pair_index(int a, int b, int p) {
    const int lo = min(a, b), hi = max(a, b);
    return lo * (2 * p - lo + 1) / 2 + (hi - lo);
}

// Words that the workgroups of k_block_sizes add their walked entries to, and
// their number: additions to one word take some 25 ns each.
constexpr int kWalkWords = 64;
constexpr unsigned kSizesGrid = 4096;

// Per block (i, j): number of entries, of non-empty rows and of work items
// (each row's run split into pieces of at most kSplitV entries).  A pass
// sees blocks on one side of the diagonal only (upper: i <= j, the oriented
// graph; else i >= j, its transpose), so each workgroup accumulates per
// unordered stripe pair in LDS and flushes its non-zero counters to the
// p x p arrays.
__global__ __launch_bounds__(B) void k_block_sizes(const int64_t *__restrict__ row_off,
                                                   const int32_t *__restrict__ col, int32_t n, int64_t m,
                                                   const int32_t *__restrict__ first,
                                                   const CutTable *__restrict__ ctp, bool upper,
                                                   unsigned long long *__restrict__ nnz,
                                                   unsigned int *__restrict__ items,
                                                   unsigned int *__restrict__ rows,
                                                   unsigned long long *__restrict__ walk,
                                                   unsigned int *__restrict__ maxrun) {
    // per stripe pair: rows (high word) and items, then entries, then the
    // longest run
    extern __shared__ unsigned long long s_cnt[];
    __shared__ int32_t s_c[kMaxP + 1];
    __shared__ unsigned long long s_walk;
    const int p = ctp->p;
    const int pp = p * p;
    const int npairs = p * (p + 1) / 2;
    unsigned int *s_nnz = reinterpret_cast<unsigned int *>(s_cnt + npairs), *s_max = s_nnz + npairs;
    for (int q = threadIdx.x; q < npairs; q += B) {
        s_cnt[q] = 0;
        s_nnz[q] = 0;
        s_max[q] = 0;
    }
    for (int q = threadIdx.x; q <= p; q += B) s_c[q] = ctp->c[q];
    if (threadIdx.x == 0) s_walk = 0;
    __syncthreads();
    // Walked entries when the kernel reads A_ik[x] for every entry (x, y) of
    // A_ij and every k >= j: the run of stripe j has (hi - lo) entries, each
    // walking the (e1 - lo) entries of stripes j and above.
    unsigned long long my_walk = 0;
    for_runs(row_off, col, n, m, first, s_c, p,
             [&](int32_t x, int32_t si, int32_t j, int64_t e, int32_t, int32_t at, bool last) {
                 if (!last) return;
                 const unsigned int cnt = static_cast<unsigned int>(at) + 1;
                 const int t = pair_index(si, j, p);
                 atomicAdd(&s_cnt[t], (1ull << 32) + (cnt + kSplitV - 1) / kSplitV);
                 atomicAdd(&s_nnz[t], cnt);
                 if (cnt > s_max[t]) atomicMax(&s_max[t], cnt);
                 if (walk) my_walk += cnt * static_cast<unsigned long long>(row_off[x + 1] - e + at);
             });
    if (walk) {
        my_walk = wave_sum(my_walk);
        if (lane_id() == 0 && my_walk) atomicAdd(&s_walk, my_walk);
    }
    __syncthreads();
    for (int q = threadIdx.x; q < pp; q += B) {
        const int a = q / p, b = q - a * p;
        if (upper ? a > b : a < b) continue;
        const int t = pair_index(a, b, p);
        if (s_cnt[t]) {
            atomicAdd(&nnz[q], static_cast<unsigned long long>(s_nnz[t]));
            atomicAdd(&items[q], static_cast<unsigned int>(s_cnt[t]));
            atomicAdd(&rows[q], static_cast<unsigned int>(s_cnt[t] >> 32));
            if (maxrun) atomicMax(&maxrun[q], s_max[t]);
        }
    }
    if (walk && threadIdx.x == 0 && s_walk) atomicAdd(&walk[blockIdx.x % kWalkWords], s_walk);
}

// Per-row entry counts of every block the row touches, written at the row's
// slot of the block's dense row range (slot_base indexed by (row stripe,
// column stripe)).
__global__ __launch_bounds__(B) void k_row_slot_counts(const int64_t *__restrict__ row_off,
                                                       const int32_t *__restrict__ col, int32_t n, int64_t m,
                                                       const int32_t *__restrict__ first,
                                                       const CutTable *__restrict__ ctp,
                                                       const int64_t *__restrict__ slot_base,
                                                       uint32_t *__restrict__ slots) {
    __shared__ int32_t s_c[kMaxP + 1];
    __shared__ int32_t s_base[kMaxP];
    const int p = ctp->p;
    for (int q = threadIdx.x; q <= p; q += B) s_c[q] = ctp->c[q];
    for (int q = threadIdx.x; q < p; q += B) s_base[q] = ctp->base[q];
    __syncthreads();
    for_runs(row_off, col, n, m, first, s_c, p,
             [&](int32_t x, int32_t si, int32_t j, int64_t, int32_t, int32_t at, bool last) {
                 if (last) slots[slot_base[si * p + j] + (x - s_base[si])] = static_cast<uint32_t>(at) + 1;
             });
}

// Block of slot q: the last block whose slot range starts at or before q.
__device__ __forceinline__ int32_t block_of_slot(int64_t q, const int64_t *sb, int32_t nb) {
    int32_t lo = 0, hi = nb - 1;
    while (lo < hi) {
        const int32_t mid = (lo + hi + 1) >> 1;
        if (sb[mid] <= q) lo = mid;
        else hi = mid - 1;
    }
    return lo;
}

// Dense row offsets of every block from the scanned slot counts, and the
// number of work items of every row (for the item-list compaction).  The
// region offsets are absolute int32-word offsets in the arena.
__global__ __launch_bounds__(B) void k_fill_rptr(const uint32_t *__restrict__ scanned,
                                                 int64_t nslots,
                                                 const int64_t *__restrict__ slot_base_dense,
                                                 const int64_t *__restrict__ rptr_off,
                                                 const int32_t *__restrict__ width, int32_t nblk,
                                                 int32_t *__restrict__ rbase,
                                                 uint32_t *__restrict__ flags) {
    extern __shared__ int64_t s_sb[];
    for (int q = threadIdx.x; q < nblk; q += B) s_sb[q] = slot_base_dense[q];
    __syncthreads();
    if (blockIdx.x == 0 && threadIdx.x == 0) flags[nslots] = 0u;
    for (int64_t q = blockIdx.x * int64_t(B) + threadIdx.x; q < nslots; q += int64_t(gridDim.x) * B) {
        const int32_t b = block_of_slot(q, s_sb, nblk);
        const int64_t r = q - s_sb[b];
        const uint32_t v = scanned[q] - scanned[s_sb[b]];
        rbase[rptr_off[b] + r] = static_cast<int32_t>(v);
        flags[q] = r < width[b] ? (scanned[q + 1] - scanned[q] + kSplitV - 1) / kSplitV : 0u;
    }
}

__global__ __launch_bounds__(B) void k_fill_items(const uint32_t *__restrict__ flags,
                                                  const uint32_t *__restrict__ pos, int64_t nslots,
                                                  const int64_t *__restrict__ slot_base_dense,
                                                  const int64_t *__restrict__ items_off,
                                                  const int64_t *__restrict__ rptr_off,
                                                  int32_t nblk, const int32_t *__restrict__ rbase,
                                                  int32_t *__restrict__ arena) {
    extern __shared__ int64_t s_sb[];
    for (int q = threadIdx.x; q < nblk; q += B) s_sb[q] = slot_base_dense[q];
    __syncthreads();
    for (int64_t q = blockIdx.x * int64_t(B) + threadIdx.x; q < nslots; q += int64_t(gridDim.x) * B) {
        const uint32_t f = flags[q];
        if (!f) continue;
        const int32_t b = block_of_slot(q, s_sb, nblk);
        const int64_t r = q - s_sb[b];
        const uint32_t at = pos[q] - pos[s_sb[b]];
        // the row's entries [start, end) (its dense offsets, written by
        // k_fill_rptr), cut into runs of at most kSplitV
        const int32_t start = rbase[rptr_off[b] + r], end = rbase[rptr_off[b] + r + 1];
        int32_t *it = arena + items_off[b] + kItemWords * static_cast<int64_t>(at);
        for (uint32_t c = 0; c < f; ++c) {
            const int32_t rb = start + static_cast<int32_t>(c) * kSplitV;
            it[kItemWords * c] = static_cast<int32_t>(r);
            it[kItemWords * c + 1] = rb;
            it[kItemWords * c + 2] = min(rb + kSplitV, end);
        }
    }
}

// Entries: row x's run in stripe j goes to the block of (stripe(x), j) at the
// row's dense offset, as local column ids (rptr_off, col_off: by stripe pair).
__global__ __launch_bounds__(B) void k_fill_cols(const int64_t *__restrict__ row_off,
                                                 const int32_t *__restrict__ col, int32_t n, int64_t m,
                                                 const int32_t *__restrict__ first,
                                                 const CutTable *__restrict__ ctp,
                                                 const int64_t *__restrict__ rptr_off,
                                                 const int64_t *__restrict__ col_off,
                                                 const int32_t *__restrict__ rbase,
                                                 int32_t *__restrict__ arena) {
    __shared__ int32_t s_c[kMaxP + 1];
    __shared__ int32_t s_base[kMaxP];
    const int p = ctp->p;
    for (int q = threadIdx.x; q <= p; q += B) s_c[q] = ctp->c[q];
    for (int q = threadIdx.x; q < p; q += B) s_base[q] = ctp->base[q];
    __syncthreads();
    for_runs(row_off, col, n, m, first, s_c, p,
             [&](int32_t x, int32_t si, int32_t j, int64_t, int32_t y, int32_t at, bool) {
                 const int b = si * p + j;
                 arena[col_off[b] + rbase[rptr_off[b] + (x - s_base[si])] + at] = y - s_base[j];
             });
}

// Reversed oriented graph: for every entry (x, y), the key y and the value x.
__global__ __launch_bounds__(B) void k_rev_pairs(const int64_t *__restrict__ row_off,
                                                 const int32_t *__restrict__ col, int32_t n, int64_t m,
                                                 const int32_t *__restrict__ first, uint32_t *__restrict__ ky,
                                                 uint32_t *__restrict__ vx) {
    for_entries(row_off, col, n, m, first, [&](int32_t x, int64_t e, int32_t y) {
        ky[e] = static_cast<uint32_t>(y);
        vx[e] = static_cast<uint32_t>(x);
    });
}

// ---- one block (p = 1): the block is the oriented graph over the ranks from
// `lo` on, its sizes are known from the build, and one pass over the rows
// writes its columns and the pairs its transpose is sorted from.

// The pairs of the transpose (higher end; lower end as a local id) and the
// block's local columns.
__global__ __launch_bounds__(B) void k_one_pairs(const int64_t *__restrict__ row_off, const int32_t *__restrict__ col,
                                                 int32_t n, int64_t m, int32_t lo, uint32_t *__restrict__ ky,
                                                 uint32_t *__restrict__ vx, int32_t *__restrict__ out_col) {
    for_entries(row_off, col, n, m, nullptr, [&](int32_t x, int64_t e, int32_t y) {
        ky[e] = static_cast<uint32_t>(y);
        vx[e] = static_cast<uint32_t>(x - lo);
        out_col[e] = y - lo;
    });
}

// Work items per row, then per column, and the local row offsets.
__global__ __launch_bounds__(B) void k_one_counts(const int64_t *__restrict__ row_off,
                                                  const int32_t *__restrict__ outdeg,
                                                  const int32_t *__restrict__ indeg, int32_t lo, int32_t width,
                                                  int32_t *__restrict__ rptr, uint32_t *__restrict__ counts) {
    for (int64_t r = blockIdx.x * int64_t(B) + threadIdx.x; r <= width; r += int64_t(gridDim.x) * B) {
        rptr[r] = static_cast<int32_t>(row_off[lo + r]);
        if (r == width) break;
        counts[r] = (outdeg[lo + r] + kSplitV - 1) / kSplitV;
        counts[width + r] = (indeg[lo + r] + kSplitV - 1) / kSplitV;
    }
}

__global__ __launch_bounds__(B) void k_one_items(const int64_t *__restrict__ row_off,
                                                 const int64_t *__restrict__ rev_off,
                                                 const uint32_t *__restrict__ pos, uint32_t row_items, int32_t lo,
                                                 int32_t width, int32_t *__restrict__ items,
                                                 int32_t *__restrict__ citems) {
    for (int64_t q = blockIdx.x * int64_t(B) + threadIdx.x; q < 2 * static_cast<int64_t>(width);
         q += int64_t(gridDim.x) * B) {
        const bool column = q >= width;
        const int32_t r = static_cast<int32_t>(column ? q - width : q);
        const int64_t *off = column ? rev_off : row_off;
        const int32_t b = static_cast<int32_t>(off[lo + r]), e = static_cast<int32_t>(off[lo + r + 1]);
        int32_t *it = column ? citems + kItemWords * static_cast<int64_t>(pos[q] - row_items)
                             : items + kItemWords * static_cast<int64_t>(pos[q]);
        for (int32_t s = b; s < e; s += kSplitV, it += kItemWords) {
            it[0] = r;
            it[1] = s;
            it[2] = min(s + kSplitV, e);
        }
    }
}

unsigned cap_grid(int64_t work) {
    unsigned g = grid_for(work, B);
    return g > 65536u ? 65536u : g;
}

// Workgroups of a pass over m > 0 entries.
unsigned tiles_of(int64_t m) { return static_cast<unsigned>((m + kTile - 1) / kTile); }

// The partition of a non-empty graph into one block.  No sizes have to come
// back from the device, so it is a dozen launches and no round trip, where the
// general path takes four passes over the rows and four over the columns
// (Erdos-Renyi, 4,096 vertices: 340 -> 85 us; R-MAT scale 20: 1.54 -> 0.61
// ms).
void partition_one_block(pgabb_graph *g, int32_t lowest) {
    hipStream_t s = g->stream;
    const int32_t n = g->n;
    const int64_t m = g->m;
    g->cuts = {0, n};
    g->base = {std::min(std::max(0, lowest), n)};
    const int32_t lo = g->base[0], width = n - lo;
    BlockInfo bi;
    bi.width = bi.cwidth = width;
    bi.nitems = static_cast<int32_t>(g->stat[kStatRowItems]);
    bi.ncitems = static_cast<int32_t>(g->stat[kStatColItems]);
    bi.nnz = m;
    bi.max_row = g->max_out;
    bi.nrows = static_cast<int32_t>(g->stat[kStatRows]);
    bi.ncols = static_cast<int32_t>(g->stat[kStatCols]);
    bi.chunk_off = 0;
    bi.chunk_len = bi.end();
    g->arena_words = bi.chunk_len;
    g->block_of[0] = 0;
    g->blocks.push_back(bi);
    g->tasks.push_back(Task{0, 0, 0, 0, 0, 0, 3 * m});
    g->probe_work_col = g->stat[kStatRowSquares];
    // (walked lists are read in segments, which may reach past the last list)
    g->arena.reset(static_cast<size_t>(g->arena_words) + kSeg, s);
    int32_t *arena = g->arena.get();

    const int passes = (g->nb + 7) / 8;
    DArray<uint32_t> ky(m, s), ky_alt(m, s), vx(m, s);
    // the sort's last pass writes the transposed entries in place
    uint32_t *crow = reinterpret_cast<uint32_t *>(arena + bi.off_crow());
    uint32_t *v0 = passes % 2 ? vx.get() : crow, *v1 = passes % 2 ? crow : vx.get();
    k_one_pairs<<<tiles_of(m), B, 0, s>>>(g->row_off.get(), g->col.get(), n, m, lo, ky.get(), v0,
                                          arena + bi.off_col());
    PGABB_HIP(hipGetLastError());
    const bool alt = radix_sort_u32(ky.get(), ky_alt.get(), v0, v1, m, g->nb, s);
    if (alt != (passes % 2 == 1))  // one edge: nothing was sorted
        PGABB_HIP(hipMemcpyAsync(crow, alt ? v1 : v0, sizeof(uint32_t) * m, hipMemcpyDeviceToDevice, s));
    DArray<int64_t> rev_off(static_cast<size_t>(n) + 1, s);
    scan_exclusive_i32(g->indeg.get(), rev_off.get(), n, rev_off.get() + n, s);
    DArray<uint32_t> counts(2 * static_cast<size_t>(width), s), pos(2 * static_cast<size_t>(width), s);
    k_one_counts<<<cap_grid(static_cast<int64_t>(width) + 1), B, 0, s>>>(g->row_off.get(), g->outdeg.get(),
                                                                        g->indeg.get(), lo, width,
                                                                        arena + bi.off_rptr(), counts.get());
    PGABB_HIP(hipGetLastError());
    scan_exclusive_u32(counts.get(), pos.get(), 2 * static_cast<int64_t>(width), nullptr, s);
    k_one_items<<<cap_grid(2 * static_cast<int64_t>(width)), B, 0, s>>>(g->row_off.get(), rev_off.get(), pos.get(),
                                                                       static_cast<uint32_t>(bi.nitems), lo, width,
                                                                       arena + bi.off_items(),
                                                                       arena + bi.off_citems());
    PGABB_HIP(hipGetLastError());
}

void partition_blocks(pgabb_graph *g, int32_t p, int32_t cut_mode, const int32_t *cuts_host) {
    hipStream_t s = g->stream;
    const int32_t n = g->n;
    if (!g->part_timer) g->part_timer = std::make_unique<StreamTimer>();
    g->part_timer->start(s);

    // ---- cut table, on the device.  Ranks below `lowest` own no edge
    // (isolated vertices rank first under the degree order), so each
    // stripe's dense row range starts at or after it.  The host reads the
    // table back with the block sizes, in one round trip.
    const int32_t lowest = (g->flags & PGABB_ORDER_BY_ID) ? 0 : static_cast<int32_t>(g->isolated);
    const bool one = p == 1 && g->m > 0;  // (cuts 0, n, whatever the mode)
    DArray<CutTable> dct(1, s);
    if (one) {
    } else if (cuts_host || cut_mode == PGABB_CUT_UNIFORM) {
        Staged<CutTable> hct(1, s);
        CutTable &ct = hct[0];
        ct = CutTable{};
        ct.p = p;
        for (int32_t i = 0; i <= p; ++i)
            ct.c[i] = cuts_host ? cuts_host[i] : static_cast<int32_t>((static_cast<int64_t>(i) * n) / p);
        for (int32_t i = 0; i < p; ++i) ct.base[i] = std::min(std::max(ct.c[i], lowest), ct.c[i + 1]);
        PGABB_HIP(hipMemcpyAsync(dct.get(), hct.get(), sizeof(CutTable), hipMemcpyHostToDevice, s));
    } else {
        k_nnz_cut_table<<<1, B, 0, s>>>(g->row_off.get(), n, g->m, p, lowest, dct.get());
        PGABB_HIP(hipGetLastError());
    }
    const CutTable *ctp = dct.get();
    Staged<CutTable> hct(1, s);
    auto take_cuts = [&]() {
        // after the round trip: the host copy of the cut table
        std::vector<int32_t> cuts(hct[0].c, hct[0].c + p + 1), base(hct[0].base, hct[0].base + p);
        g->cuts = cuts;
        g->base = base;
    };

    // drop any previous partition
    g->arena.release();
    g->host_arena.release();
    g->blocks_on_host = false;
    g->blocks.clear();
    g->tasks.clear();
    g->task_counts.clear();
    g->block_of.assign(static_cast<size_t>(p) * p, -1);
    g->p = 0;  // until every table and the arena are there
    g->cut_mode = cuts_host ? -1 : cut_mode;
    g->arena_words = 0;
    g->probe_work_col = 0;

    if (one) {
        partition_one_block(g, lowest);
    } else if (g->m > 0) {
        const size_t pp = static_cast<size_t>(p) * p;
        const unsigned tiles = tiles_of(g->m);
        const bool table = tiles > kTableTiles;
        DArray<int32_t> first_f(table ? static_cast<size_t>(tiles) + 1 : 0, s);
        DArray<int32_t> first_r(table ? static_cast<size_t>(tiles) + 1 : 0, s);
        const unsigned fgrid = tiles / (B / kWave) + 1;
        if (table) k_tile_first<<<fgrid, B, 0, s>>>(g->row_off.get(), n, g->m, tiles, first_f.get());
        PGABB_HIP(hipGetLastError());

        // one buffer cleared at once: block sizes -- nnz[pp] nnz_r[pp] (u64) |
        // items[pp] items_r[pp] (u32) | walked entries of column walks (u64s) |
        // longest row run per block, non-empty rows, non-empty rows of the
        // transposes (u32 each) -- which are copied back
        const size_t nsz = 3 * pp + kWalkWords + (3 * pp + 1) / 2;
        DArray<unsigned long long> dsz(nsz, s);
        PGABB_HIP(hipMemsetAsync(dsz.get(), 0, nsz * sizeof(unsigned long long), s));

        // ---- reversed oriented graph (in-edges, sorted by (y, x)): its blocks
        // are the transposes of the forward blocks
        // (row offsets: the scanned in-degrees from the build)
        DArray<int64_t> rev_off(static_cast<size_t>(n) + 1, s);
        DArray<uint32_t> vx(g->m, s), vx_alt(g->m, s);
        const int32_t *rev_col = nullptr;
        {
            DArray<uint32_t> ky(g->m, s), ky_alt(g->m, s);
            k_rev_pairs<<<tiles, B, 0, s>>>(g->row_off.get(), g->col.get(), n, g->m, first_f.get(), ky.get(), vx.get());
            PGABB_HIP(hipGetLastError());
            // pairs come in CSR order, ascending in x within each y, so a
            // stable sort on y orders them by (y, x)
            const bool alt = radix_sort_u32(ky.get(), ky_alt.get(), vx.get(), vx_alt.get(), g->m, g->nb, s);
            rev_col = reinterpret_cast<const int32_t *>(alt ? vx_alt.get() : vx.get());
            (alt ? vx : vx_alt).release();
            scan_exclusive_i32(g->indeg.get(), rev_off.get(), n, rev_off.get() + n, s);
        }
        if (table) k_tile_first<<<fgrid, B, 0, s>>>(rev_off.get(), n, g->m, tiles, first_r.get());
        PGABB_HIP(hipGetLastError());

        // ---- block sizes, forward (entries, row items) and reversed (column items)
        unsigned long long *dnnz = dsz.get(), *dnnz_r = dnnz + pp, *dwalk = dsz.get() + 3 * pp;
        unsigned int *ditems = reinterpret_cast<unsigned int *>(dnnz_r + pp), *ditems_r = ditems + pp;
        unsigned int *dmax = reinterpret_cast<unsigned int *>(dwalk + kWalkWords);
        unsigned int *drows = dmax + pp, *drows_r = drows + pp;
        const unsigned sgrid = std::min(tiles, kSizesGrid);
        const size_t slds = 4 * sizeof(unsigned int) * static_cast<size_t>(p) * (p + 1) / 2;
        k_block_sizes<<<sgrid, B, slds, s>>>(g->row_off.get(), g->col.get(), n, g->m, first_f.get(), ctp, true, dnnz,
                                             ditems, drows, dwalk, dmax);
        k_block_sizes<<<sgrid, B, slds, s>>>(rev_off.get(), rev_col, n, g->m, first_r.get(), ctp, false, dnnz_r,
                                             ditems_r, drows_r, nullptr, nullptr);
        PGABB_HIP(hipGetLastError());
        Staged<unsigned long long> hsz(nsz, s);
        PGABB_HIP(hipMemcpyAsync(hsz.get(), dsz.get(), hsz.bytes(), hipMemcpyDeviceToHost, s));
        PGABB_HIP(hipMemcpyAsync(hct.get(), dct.get(), sizeof(CutTable), hipMemcpyDeviceToHost, s));
        PGABB_HIP(hipStreamSynchronize(s));
        take_cuts();
        const std::vector<int32_t> &cuts = g->cuts, &base = g->base;
        const unsigned long long *hnnz = hsz.get();
        const unsigned int *hitems = reinterpret_cast<const unsigned int *>(hsz.get() + 2 * pp);
        const unsigned int *hitems_r = hitems + pp;
        const unsigned int *hmax = reinterpret_cast<const unsigned int *>(hsz.get() + 3 * pp + kWalkWords);
        const unsigned int *hrows = hmax + pp, *hrows_r = hrows + pp;
        for (int q = 0; q < kWalkWords; ++q) g->probe_work_col += hsz[3 * pp + q];

        // ---- block table (row-major block order) and chunk layout
        for (int32_t i = 0; i < p; ++i) {
            for (int32_t j = 0; j < p; ++j) {
                const size_t q = static_cast<size_t>(i) * p + j;
                if (!hnnz[q]) continue;
                PGABB_REQUIRE(i <= j, PGABB_EDEVICE, "entry below the diagonal in block (%d, %d)", i, j);
                BlockInfo bi;
                bi.i = i;
                bi.j = j;
                bi.width = cuts[i + 1] - base[i];
                bi.cwidth = cuts[j + 1] - base[j];
                bi.nitems = static_cast<int32_t>(hitems[q]);
                bi.ncitems = static_cast<int32_t>(hitems_r[static_cast<size_t>(j) * p + i]);
                bi.nnz = static_cast<int64_t>(hnnz[q]);
                bi.max_row = static_cast<int32_t>(hmax[q]);
                bi.nrows = static_cast<int32_t>(hrows[q]);
                bi.ncols = static_cast<int32_t>(hrows_r[static_cast<size_t>(j) * p + i]);
                bi.chunk_off = g->arena_words;
                bi.chunk_len = bi.end() - bi.chunk_off;
                g->arena_words += bi.chunk_len;
                g->block_of[q] = static_cast<int32_t>(g->blocks.size());
                g->blocks.push_back(bi);
            }
        }
        const int32_t nblk = static_cast<int32_t>(g->blocks.size());
        // (walked lists are read in segments, which may reach past the last list)
        g->arena.reset(static_cast<size_t>(g->arena_words) + kSeg, s);
        // the transposes' dense column offsets, needed only while the chunks
        // are filled
        std::vector<int64_t> coff(static_cast<size_t>(nblk) + 1, 0);
        for (int32_t b = 0; b < nblk; ++b) coff[b + 1] = coff[b] + g->blocks[b].cwidth + 1;
        DArray<int32_t> ctmp(static_cast<size_t>(std::max<int64_t>(coff[nblk], 1)), s);

        // Both passes run the same machinery: per-row run counts at dense
        // slots, one scan (row offsets), per-row item counts, one scan (item
        // lists), then the entries.  The reversed pass fills the transposes.
        // Per-block tables of each pass travel in one pinned host buffer
        // (int64 tables, then int32 tables) and one copy.
        for (int pass = 0; pass < 2; ++pass) {
            const bool rev = pass == 1;
            const int64_t *off = rev ? rev_off.get() : g->row_off.get();
            const int32_t *cl = rev ? rev_col : g->col.get();
            const int32_t *first = rev ? first_r.get() : first_f.get();
            // layout: sb_pp[pp] ro_pp[pp] co_pp[pp] (by stripe pair, of non-empty
            // blocks) sb_dense[nblk] rptr_off[nblk] items_off[nblk] |
            // width[nblk] (int32)
            const size_t n64 = 3 * pp + 3 * static_cast<size_t>(nblk);
            const size_t n32 = static_cast<size_t>(nblk);
            Staged<int64_t> tab(n64 + (n32 + 1) / 2, s);
            int64_t *sb_pp = tab.get(), *ro_pp = sb_pp + pp, *co_pp = ro_pp + pp;
            int64_t *sb_dense = co_pp + pp, *rptr_off = sb_dense + nblk, *items_off = rptr_off + nblk;
            int32_t *width = reinterpret_cast<int32_t *>(tab.get() + n64);
            std::fill(sb_pp, sb_pp + 3 * pp, int64_t(-1));
            int64_t nslots = 0;
            for (int32_t b = 0; b < nblk; ++b) {
                const BlockInfo &bi = g->blocks[b];
                // forward: rows in stripe i, columns in stripe j; reversed: the
                // transpose, rows in stripe j, columns in stripe i
                const size_t q = rev ? static_cast<size_t>(bi.j) * p + bi.i : static_cast<size_t>(bi.i) * p + bi.j;
                sb_pp[q] = nslots;
                sb_dense[b] = nslots;
                width[b] = rev ? bi.cwidth : bi.width;
                rptr_off[b] = rev ? coff[b] : bi.off_rptr();
                items_off[b] = rev ? bi.off_citems() : bi.off_items();
                ro_pp[q] = rptr_off[b];
                co_pp[q] = rev ? bi.off_crow() : bi.off_col();
                nslots += static_cast<int64_t>(width[b]) + 1;
            }
            DArray<int64_t> dtab(tab.size(), s);
            PGABB_HIP(hipMemcpyAsync(dtab.get(), tab.get(), tab.bytes(), hipMemcpyHostToDevice, s));
            const int64_t *d_sb_pp = dtab.get(), *d_ro_pp = d_sb_pp + pp, *d_co_pp = d_ro_pp + pp;
            const int64_t *d_sb = d_co_pp + pp, *d_ro = d_sb + nblk, *d_io = d_ro + nblk;
            const int32_t *d_w = reinterpret_cast<const int32_t *>(dtab.get() + n64);

            DArray<uint32_t> slots(static_cast<size_t>(nslots) + 1, s), flags(static_cast<size_t>(nslots) + 1, s);
            PGABB_HIP(hipMemsetAsync(slots.get(), 0, (nslots + 1) * sizeof(uint32_t), s));
            k_row_slot_counts<<<tiles, B, 0, s>>>(off, cl, n, g->m, first, ctp, d_sb_pp, slots.get());
            PGABB_HIP(hipGetLastError());
            scan_exclusive_u32(slots.get(), slots.get(), nslots + 1, nullptr, s);
            const size_t lds = static_cast<size_t>(nblk) * sizeof(int64_t);
            int32_t *rbase = rev ? ctmp.get() : g->arena.get();
            k_fill_rptr<<<cap_grid(nslots), B, lds, s>>>(slots.get(), nslots, d_sb, d_ro, d_w, nblk, rbase,
                                                         flags.get());
            PGABB_HIP(hipGetLastError());
            scan_exclusive_u32(flags.get(), slots.get(), nslots + 1, nullptr, s);  // slots now item positions
            k_fill_items<<<cap_grid(nslots), B, lds, s>>>(flags.get(), slots.get(), nslots, d_sb, d_io, d_ro,
                                                          nblk, rbase, g->arena.get());
            PGABB_HIP(hipGetLastError());
            k_fill_cols<<<tiles, B, 0, s>>>(off, cl, n, g->m, first, ctp, d_ro_pp, d_co_pp, rbase, g->arena.get());
            PGABB_HIP(hipGetLastError());
        }

        // ---- tasks: i <= j <= k with three non-empty blocks
        for (int32_t i = 0; i < p; ++i)
            for (int32_t j = i; j < p; ++j) {
                const int32_t bij = g->block_of[static_cast<size_t>(i) * p + j];
                if (bij < 0) continue;
                for (int32_t k = j; k < p; ++k) {
                    const int32_t bik = g->block_of[static_cast<size_t>(i) * p + k];
                    const int32_t bjk = g->block_of[static_cast<size_t>(j) * p + k];
                    if (bik < 0 || bjk < 0) continue;
                    Task t{i, j, k, bij, bik, bjk,
                           g->blocks[bij].nnz + g->blocks[bik].nnz + g->blocks[bjk].nnz};
                    g->tasks.push_back(t);
                }
            }
        std::stable_sort(g->tasks.begin(), g->tasks.end(),
                         [](const Task &a, const Task &b) { return a.weight > b.weight; });
        // no wait here: the fills run on while the caller goes on; later
        // work on the stream is ordered after them, and the scratch freed
        // above is reused only after its free's event
    } else {
        PGABB_HIP(hipMemcpyAsync(hct.get(), dct.get(), sizeof(CutTable), hipMemcpyDeviceToHost, s));
        PGABB_HIP(hipStreamSynchronize(s));
        take_cuts();
    }
    g->task_counts.assign(g->tasks.size(), 0);
    g->part_timer->stop(s);
    g->part_time_pending = true;
    g->p = p;
}

}  // namespace

void partition_graph(pgabb_graph *g, int32_t p, int32_t cut_mode, const int32_t *cuts_host) {
    try {
        partition_blocks(g, p, cut_mode, cuts_host);
    } catch (...) {
        // Block and task tables are filled in before the arena they point into
        // is allocated.  A partition that ends early leaves none of them, so
        // that no later call follows them into memory that is not there: the
        // graph is as if it had never been partitioned.  (p > 0: it ended
        // before the previous partition was dropped.)
        if (g->p == 0) {
            g->arena.release();
            g->blocks.clear();
            g->tasks.clear();
            g->task_counts.clear();
            g->block_of.clear();
            g->cuts.clear();
            g->base.clear();
            g->arena_words = 0;
            g->probe_work_col = 0;
            g->part_time_pending = false;
        }
        throw;
    }
}

}  // namespace pgabb
