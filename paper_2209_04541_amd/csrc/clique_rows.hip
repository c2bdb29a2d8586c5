// 4-cliques of a graph in device memory, from the oriented CSR: one vertex at
// a time instead of one (4-list, edge) at a time (PGAbB Section 3.2's
// multi-block pattern mode; the per-4-list counts of kclique.hip come from
// the stripes of the clique's vertices).
//
// Each 4-clique with ranks a < b < c < d is a triangle of the subgraph that
// a's out-neighbours N+(a) induce.  For a vertex a with members c_0 < c_1 <
// ... of N+(a):
//   1. the induced subgraph is written as a bit matrix M in LDS (bit y of row
//      x, x < y, when (c_x, c_y) is an edge): lane l tests pair (x, 64 q + l)
//      and one ballot is the 64-bit word q of row x;
//   2. its triangles x < y < z are counted as bits of M[x] & M[y] over the
//      edges (x, y): lane l holds a word of row y = 64 q + l, the row of x is
//      broadcast.
// A pair is tested with one load in a bit matrix of the kHubRanks highest
// ranks ("hubs", which hold most of the members on skewed graphs), or, when
// c_x is no hub, by a binary search of N+(c_x).
//
// This tests sum_a d+(a) (d+(a) - 1) / 2 pairs and reads no list per (a, b);
// the kernel over block 4-lists walks A_kl[c] for every (a, b, c), 67.6 G
// entries on R-MAT scale 20 against 1.2 G pairs here (155 -> 4.3 ms in one
// block, 187 -> 4.9 ms over 8 x 8; scale 18 over 4 x 4 26.8 -> 1.0 ms).
// Bound by the pair tests' loads (step 1) on skewed graphs: on R-MAT scale 20
// two thirds of their requests miss L2 (105 M lines, 3.1 TB/s) and the waves
// wait 63 % of their cycles, the LDS is active 18 % and the VALU 45 %.  Step 2
// issues about 12 instructions per 64 words of z's.
//
// Vertices with kWaveRow < d+ <= kGroupRow are taken by whole workgroups
// (their matrix needs up to 128 KB of LDS), then those with 3 <= d+ <=
// kWaveRow by single waves (8 KB of LDS each): sixteen waves per workgroup, one
// workgroup per CU.
#include <hip/hip_runtime.h>

#include <algorithm>

#include "common.hpp"
#include "graph.hpp"
#include "wave.hpp"

namespace pgabb {

namespace {

constexpr int kRB = 256;
constexpr int kRowWaves = 16;
constexpr int kRowThreads = kRowWaves * kWave;
constexpr int kWaveRow = 256;              // longest row one wave takes
constexpr int kGroupRow = kQuadRowCap;     // longest row a workgroup takes
constexpr int kWaveWords = kWaveRow * (kWaveRow / 64);     // 64-bit words of a wave's matrix
constexpr int kGroupWords = kGroupRow * (kGroupRow / 64);  // and of a workgroup's
static_assert(kWaveWords * kRowWaves == kGroupWords, "both layouts share the LDS");
// Per-4-list counters kept in LDS up to this grid (a workgroup adds them to
// the device counters once); larger grids spread their additions over enough
// device counters.
constexpr int kLdsGrid = 12;
constexpr int kLdsLists = kLdsGrid * (kLdsGrid + 1) * (kLdsGrid + 2) * (kLdsGrid + 3) / 24;
constexpr int kMaxStripes = 64;
// Ranks of the hub matrix.  A skewed graph (some row longer than a wave):
// 32,768 of them, 128 MB; R-MAT scale 20 takes 11.2 / 6.9 / 5.2 / 4.3 ms of
// kernels with 4096 / 8192 / 16384 / 32768, scale 18 1.26 / 1.15 / 1.04 /
// 0.92 ms: every pair below them costs a binary search.  Without such rows a
// hub is any vertex and the matrix does not pay (Erdos-Renyi, n = 100,001, m
// = 1.6 M: 233 / 243 / 261 / 274 us).
constexpr int kHubRanks = 32768;
constexpr int kHubRanksShort = 4096;
// When device memory is short the matrix is halved, down to this many ranks,
// and then left out: every pair is then searched.
constexpr int kHubRanksLeast = 512;
constexpr int kRowQueues = 8;        // work counters of the single-wave vertices
constexpr int kRowQueueStride = 32;  // words apart
constexpr int kRowGrab = 4;          // vertices per grab

// Position of (i, j, k, l), i <= j <= k <= l, among all such four.
__host__ __device__ __forceinline__ int32_t quad_index(int32_t i, int32_t j, int32_t k, int32_t l) {
    return i + j * (j + 1) / 2 + k * (k + 1) * (k + 2) / 6 +
           static_cast<int32_t>(static_cast<int64_t>(l) * (l + 1) * (l + 2) * (l + 3) / 24);
}

// Bit matrix of the hub ranks [lo, n): bit (w - lo) of row (v - lo) for every
// edge (v, w), v a hub (w > v is one too); `words` 32-bit words per row.  One
// wave per row: the row is gathered in LDS and written once.
__global__ __launch_bounds__(kRB) void k_hub_rows(const int64_t *__restrict__ row_off, const int32_t *__restrict__ col,
                                                  int32_t lo, int32_t n, int32_t words, uint32_t *__restrict__ hub) {
    __shared__ uint32_t s_row[kRB / kWave][kHubRanks / 32];
    uint32_t *row = s_row[threadIdx.x / kWave];
    const int lane = lane_id();
    const int32_t nw = static_cast<int32_t>(gridDim.x) * (kRB / kWave);
    for (int32_t v = lo + static_cast<int32_t>(blockIdx.x) * (kRB / kWave) + static_cast<int32_t>(threadIdx.x / kWave);
         v < n; v += nw) {
        for (int32_t q = lane; q < words; q += kWave) row[q] = 0u;
        wave_lds_sync();
        const int64_t e1 = row_off[v + 1];
        for (int64_t e = row_off[v] + lane; e < e1; e += kWave) {
            const int32_t w = col[e] - lo;
            atomicOr(&row[w >> 5], 1u << (w & 31));
        }
        wave_lds_sync();
        uint32_t *dst = hub + static_cast<int64_t>(v - lo) * words;
        for (int32_t q = lane; q < words; q += kWave) dst[q] = row[q];
        wave_lds_sync();
    }
}

// The vertices of the two classes, highest rank first as far as the
// workgroups' order goes: num[0] of big (a workgroup each), num[1] of small.
__global__ __launch_bounds__(kRB) void k_row_classes(const int64_t *__restrict__ row_off, int32_t n,
                                                     int32_t *__restrict__ big, int32_t *__restrict__ small,
                                                     unsigned int *__restrict__ num) {
    __shared__ unsigned int s_n[2], s_at[2];
    if (threadIdx.x < 2) s_n[threadIdx.x] = 0;
    __syncthreads();
    constexpr int kPer = 4;
    const int64_t base = blockIdx.x * static_cast<int64_t>(kRB) * kPer;
    int cls[kPer];
    unsigned int at[kPer];
#pragma unroll
    for (int q = 0; q < kPer; ++q) {
        const int64_t r = base + q * kRB + threadIdx.x;
        cls[q] = -1;
        at[q] = 0;
        if (r < n) {
            const int64_t v = n - 1 - r;
            const int64_t d = row_off[v + 1] - row_off[v];
            if (d >= 3 && d <= kGroupRow) cls[q] = d > kWaveRow ? 0 : 1;
        }
        if (cls[q] >= 0) at[q] = atomicAdd(&s_n[cls[q]], 1u);
    }
    __syncthreads();
    if (threadIdx.x < 2) s_at[threadIdx.x] = s_n[threadIdx.x] ? atomicAdd(&num[threadIdx.x], s_n[threadIdx.x]) : 0u;
    __syncthreads();
#pragma unroll
    for (int q = 0; q < kPer; ++q) {
        if (cls[q] < 0) continue;
        const int32_t v = static_cast<int32_t>(n - 1 - (base + q * kRB + threadIdx.x));
        (cls[q] == 0 ? big : small)[s_at[cls[q]] + at[q]] = v;
    }
}

struct RowArgs {
    const int64_t *row_off;
    const int32_t *col;
    const uint32_t *hub;  // bit matrix of the ranks >= hub_lo
    const int32_t *big, *small;
    const unsigned int *num;
    unsigned long long *next;    // big's counter, then kRowQueues of small's, kRowQueueStride apart
    unsigned long long *counts;  // by quad_index
    const int32_t *cuts;         // p + 1
    int32_t hub_lo, hub_words;
    int32_t p;
};

// Whether w is an entry of the sorted list col[lo, hi).
__device__ __forceinline__ bool row_has(gptr<int32_t> col, int64_t lo, int64_t hi, int32_t w) {
    int32_t len = static_cast<int32_t>(hi - lo);
    if (len <= 0) return false;
    gptr<int32_t> x = col + lo;
    while (len > 1) {  // the last entry <= w, if any, stays in x[0, len)
        const int32_t half = len >> 1;
        x = x[half] <= w ? x + half : x;
        len -= half;
    }
    return x[0] == w;
}

// The bit matrix of one vertex's members mem[0, d), NB words a row, by the
// NW waves of its team (this one: wv).  Every word at or right of a row's
// diagonal word is written.
template <int NW>
__device__ __forceinline__ void induced_bits(const RowArgs &a, const int32_t *mem, int32_t d, int32_t NB,
                                             uint64_t *__restrict__ M, int wv, int lane) {
    const gptr<int64_t> ro = as_global(a.row_off);
    const gptr<int32_t> col = as_global(a.col);
    const gptr<uint32_t> hub = as_global(a.hub);
    // hubs are the members from xc on (members ascend)
    int32_t xc = 0;
    {
        int32_t hi = d;
        while (xc < hi) {
            const int32_t mid = (xc + hi) >> 1;
            if (mem[mid] < a.hub_lo) xc = mid + 1;
            else hi = mid;
        }
        xc = __builtin_amdgcn_readfirstlane(xc);
    }
    constexpr int32_t kRun = 16;  // rows per unit of work
    int32_t u = 0;
    for (int32_t yb = 0; yb < NB; ++yb) {
        const int32_t y = yb * kWave + lane;
        const int32_t cy = y < d ? mem[y] : -1;
        const int32_t h = cy - a.hub_lo;  // a hub when some x before it is
        const int32_t hw = h >= 0 ? h >> 5 : 0;
        const uint32_t hb = static_cast<uint32_t>(h & 31);
        const int32_t xend = min(d, yb * kWave + kWave);
        for (int32_t x0 = 0; x0 < xend; x0 += kRun, ++u) {
            if (NW > 1 && u % NW != wv) continue;
            const int32_t x1 = min(x0 + kRun, xend);
            int32_t x = x0;
            for (; x < min(x1, xc); ++x) {  // no hub: search N+(c_x)
                const int32_t cx = __builtin_amdgcn_readfirstlane(mem[x]);
                const int64_t r0 = ro[cx], r1 = ro[cx + 1];
                const bool in = y > x && y < d && row_has(col, r0, r1, cy);
                const uint64_t bits = __ballot(in);
                if (lane == 0) M[x * NB + yb] = bits;
            }
            for (; x + 4 <= x1; x += 4) {  // four rows' loads in flight
                uint32_t wd[4];
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    const int32_t cx = __builtin_amdgcn_readfirstlane(mem[x + q]);
                    wd[q] = hub[static_cast<int64_t>(cx - a.hub_lo) * a.hub_words + hw];
                }
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    const uint64_t bits = __ballot(((wd[q] >> hb) & 1u) != 0u && y > x + q && y < d);
                    if (lane == 0) M[(x + q) * NB + yb] = bits;
                }
            }
            for (; x < x1; ++x) {
                const int32_t cx = __builtin_amdgcn_readfirstlane(mem[x]);
                const uint32_t wd = hub[static_cast<int64_t>(cx - a.hub_lo) * a.hub_words + hw];
                const uint64_t bits = __ballot(((wd >> hb) & 1u) != 0u && y > x && y < d);
                if (lane == 0) M[x * NB + yb] = bits;
            }
        }
    }
}

// The same for at most 64 members, by one wave: the pairs x < y are flattened
// over the lanes (a short row would leave most lanes idle above).
__device__ __forceinline__ void induced_bits_short(const RowArgs &a, const int32_t *mem, int32_t d,
                                                   uint64_t *__restrict__ M, int lane) {
    const gptr<int64_t> ro = as_global(a.row_off);
    const gptr<int32_t> col = as_global(a.col);
    const gptr<uint32_t> hub = as_global(a.hub);
    M[lane] = 0ull;
    wave_lds_sync();
    const int32_t np = d * (d - 1) / 2;
    for (int32_t t = lane; t < np; t += kWave) {
        // pair t: y (y - 1) / 2 <= t < y (y + 1) / 2, x = t - y (y - 1) / 2
        int32_t y = static_cast<int32_t>((1.0f + sqrtf(1.0f + 8.0f * static_cast<float>(t))) * 0.5f);
        if (y * (y - 1) / 2 > t) --y;
        if ((y + 1) * y / 2 <= t) ++y;
        const int32_t x = t - y * (y - 1) / 2;
        const int32_t cx = mem[x], cy = mem[y];
        bool in;
        if (cx >= a.hub_lo) {
            const int32_t h = cy - a.hub_lo;
            in = (hub[static_cast<int64_t>(cx - a.hub_lo) * a.hub_words + (h >> 5)] >> (h & 31)) & 1u;
        } else {
            in = row_has(col, ro[cx], ro[cx + 1], cy);
        }
        if (in) atomicOr(reinterpret_cast<uint32_t *>(M) + 2 * x + (y >> 5), 1u << (y & 31));
    }
    wave_lds_sync();
}

// Bits [a, b) of a 64-bit word whose bit 0 is position `at`.
__device__ __forceinline__ uint64_t range_mask(int32_t a, int32_t b, int32_t at) {
    const int32_t lo = max(a - at, 0), hi = min(b - at, 64);
    if (lo >= hi) return 0ull;
    const uint64_t upto = hi == 64 ? ~0ull : ((1ull << hi) - 1ull);
    return upto & (~0ull << lo);
}

// Triangles x < y < z of the induced subgraph, by the NW waves of its team.
// A unit of work is a block of 64 rows x, a block of 64 rows y (one per lane)
// and a word of z's.  With one stripe the lanes' sums stay in acc; else a
// unit's sums go to the counter of their stripes: sst[s] is the stripe of the
// members [seg[s], seg[s + 1]).
template <int NW, bool BLOCKS, class Add>
__device__ __forceinline__ void induced_triangles(const uint64_t *__restrict__ M, int32_t d, int32_t NB, int32_t ns,
                                                  const uint16_t *seg, const uint8_t *sst, int wv, int lane,
                                                  unsigned long long &acc, Add add) {
    const uint32_t *M32 = reinterpret_cast<const uint32_t *>(M);
    int32_t u = 0;
    for (int32_t yb = 0; yb < NB; ++yb) {
        const int32_t y = yb * kWave + lane;
        for (int32_t w = yb; w < NB; ++w) {
            const uint64_t my = y < d ? M[y * NB + w] : 0ull;
            for (int32_t xb = 0; xb <= yb; ++xb, ++u) {
                if (NW > 1 && u % NW != wv) continue;
                const int32_t xa = xb * kWave, xz = min(xa + kWave, d);
                auto rows = [&](int32_t x0, int32_t x1, uint64_t row_y) {
                    uint32_t cnt = 0;
                    const uint32_t y0 = static_cast<uint32_t>(row_y), y1 = static_cast<uint32_t>(row_y >> 32);
                    const int32_t sel = 2 * yb + (lane >> 5);
#pragma unroll 4
                    for (int32_t x = x0; x < x1; ++x) {
                        const uint64_t mx = M[x * NB + w];
                        // all ones where (x, y) is an edge
                        const uint32_t edge = static_cast<uint32_t>(
                            -static_cast<int32_t>((M32[2 * (x * NB) + sel] >> (lane & 31)) & 1u));
                        cnt += (__popc(static_cast<uint32_t>(mx) & y0) + __popc(static_cast<uint32_t>(mx >> 32) & y1)) &
                               edge;
                    }
                    return cnt;
                };
                if (!BLOCKS || ns == 1) {
                    acc += rows(xa, xz, my);
                    continue;
                }
                for (int32_t l = 0; l < ns; ++l) {
                    const uint64_t ml = my & range_mask(seg[l], seg[l + 1], w * kWave);
                    if (__ballot(ml != 0ull) == 0) continue;
                    for (int32_t j = 0; j <= l; ++j) {
                        const int32_t x0 = max(xa, static_cast<int32_t>(seg[j]));
                        const int32_t x1 = min(xz, static_cast<int32_t>(seg[j + 1]));
                        if (x0 >= x1) continue;
                        const uint32_t cnt = rows(x0, x1, ml);
                        if (__ballot(cnt != 0u) == 0) continue;
                        for (int32_t k = j; k <= l; ++k) {
                            const bool mine = y >= seg[k] && y < seg[k + 1];
                            if (__ballot(mine && cnt != 0u) == 0) continue;
                            const uint32_t sum = wave_sum(mine ? cnt : 0u);
                            if (lane == 0) add(sst[j], sst[k], sst[l], sum);
                        }
                    }
                }
            }
        }
    }
}

// The stripes of the members: ns segments (first member, stripe), by one wave.
__device__ __forceinline__ int32_t member_stripes(const RowArgs &a, const int32_t *s_cuts, const int32_t *mem,
                                                  int32_t d, uint16_t *seg, uint8_t *sst, int lane) {
    int32_t ns = 0, prev_last = -1;
    const uint64_t below = lane ? (~0ull >> (64 - lane)) : 0ull;
    for (int32_t y0 = 0; y0 < d; y0 += kWave) {
        const int32_t y = y0 + lane;
        int32_t st = 0;
        if (y < d) {
            const int32_t c = mem[y];
            int32_t lo = 0, hi = a.p - 1;
            while (lo < hi) {
                const int32_t mid = (lo + hi + 1) >> 1;
                if (s_cuts[mid] <= c) lo = mid;
                else hi = mid - 1;
            }
            st = lo;
        }
        int32_t prev = __shfl_up(st, 1);
        if (lane == 0) prev = prev_last;
        const bool start = y < d && st != prev;
        const uint64_t starts = __ballot(start);
        if (start) {
            const int32_t at = ns + __popcll(starts & below);
            seg[at] = static_cast<uint16_t>(y);
            sst[at] = static_cast<uint8_t>(st);
        }
        ns += __popcll(starts);
        prev_last = __builtin_amdgcn_readlane(st, kWave - 1);
    }
    if (lane == 0) seg[ns] = static_cast<uint16_t>(d);
    return ns;
}

template <bool BLOCKS>
__global__ __launch_bounds__(kRowThreads) void k_quad_rows(RowArgs a) {
    __shared__ uint64_t s_m[kGroupWords];
    __shared__ int32_t s_mem[kRowWaves * kWaveRow];
    __shared__ uint16_t s_seg[kRowWaves][kMaxStripes + 2];
    __shared__ uint8_t s_sst[kRowWaves][kMaxStripes];
    __shared__ int32_t s_cuts[kMaxStripes + 1];
    __shared__ int32_t s_take, s_ns;
    __shared__ unsigned long long s_counts[BLOCKS ? kLdsLists : 1];
    const int lane = lane_id();
    const int wv = __builtin_amdgcn_readfirstlane(static_cast<int>(threadIdx.x / kWave));
    const int32_t nlists = quad_index(0, 0, 0, a.p);  // first index past the grid's
    const bool lds_counts = BLOCKS && a.p <= kLdsGrid;
    if (BLOCKS) {
        for (int32_t q = threadIdx.x; q <= a.p; q += kRowThreads) s_cuts[q] = a.cuts[q];
        if (lds_counts)
            for (int32_t q = threadIdx.x; q < nlists; q += kRowThreads) s_counts[q] = 0ull;
    }
    __syncthreads();
    const gptr<int64_t> ro = as_global(a.row_off);
    const gptr<int32_t> col = as_global(a.col);
    unsigned long long acc = 0;  // one stripe: this lane's sum over all vertices
    auto stripe_of = [&](int32_t v) {
        int32_t lo = 0, hi = a.p - 1;
        while (lo < hi) {
            const int32_t mid = (lo + hi + 1) >> 1;
            if (s_cuts[mid] <= v) lo = mid;
            else hi = mid - 1;
        }
        return lo;
    };
    auto adder = [&](int32_t i) {
        return [&, i](int32_t j, int32_t k, int32_t l, uint32_t sum) {
            const int32_t q = quad_index(i, j, k, l);
            if (lds_counts) atomicAdd(&s_counts[q], static_cast<unsigned long long>(sum));
            else atomicAdd(&a.counts[q], static_cast<unsigned long long>(sum));
        };
    };
    // members of one stripe: the lanes' sums of this vertex to its counter
    auto flush_one = [&](int32_t i, int32_t jkl, unsigned long long part) {
        const unsigned long long sum = wave_sum(part);
        if (lane == 0 && sum) {
            const int32_t q = quad_index(i, jkl, jkl, jkl);
            if (lds_counts) atomicAdd(&s_counts[q], sum);
            else atomicAdd(&a.counts[q], sum);
        }
    };

    // ---- long rows: the whole workgroup
    const int32_t nbig = static_cast<int32_t>(a.num[0]);
    for (;;) {
        if (threadIdx.x == 0)
            s_take = static_cast<int32_t>(min(atomicAdd(&a.next[0], 1ull), static_cast<unsigned long long>(nbig)));
        __syncthreads();
        const int32_t take = s_take;
        if (take >= nbig) break;
        const int32_t v = a.big[take];
        const int64_t e0 = ro[v];
        const int32_t d = static_cast<int32_t>(ro[v + 1] - e0);
        const int32_t NB = (d + kWave - 1) / kWave;
        for (int32_t y = threadIdx.x; y < d; y += kRowThreads) s_mem[y] = col[e0 + y];
        __syncthreads();
        induced_bits<kRowWaves>(a, s_mem, d, NB, s_m, wv, lane);
        if (BLOCKS && wv == 0) {
            const int32_t ns = member_stripes(a, s_cuts, s_mem, d, s_seg[0], s_sst[0], lane);
            if (lane == 0) s_ns = ns;
        }
        __syncthreads();
        const int32_t ns = BLOCKS ? s_ns : 1;
        const int32_t i = BLOCKS ? stripe_of(v) : 0;
        unsigned long long part = 0;
        induced_triangles<kRowWaves, BLOCKS>(s_m, d, NB, ns, s_seg[0], s_sst[0], wv, lane, part, adder(i));
        if (!BLOCKS) acc += part;
        else if (ns == 1) flush_one(i, s_sst[0][0], part);
        __syncthreads();  // before the next vertex overwrites the matrix
    }

    // ---- short rows: a wave each
    const int64_t nsmall = static_cast<int64_t>(a.num[1]);
    uint64_t *M = s_m + wv * kWaveWords;
    int32_t *mem = s_mem + wv * kWaveRow;
    const int64_t nchunks = (nsmall + kRowGrab - 1) / kRowGrab;
    UnitTaker<kRowQueues, kRowQueueStride> taker(a.next + kRowQueueStride, nchunks,
                                                 static_cast<int64_t>(gridDim.x) * kRowWaves,
                                                 static_cast<int64_t>(blockIdx.x) * kRowWaves + wv);
    for (int64_t c; (c = taker.take(lane)) >= 0;) {
        const int64_t t1 = min((c + 1) * kRowGrab, nsmall);
        for (int64_t t = c * kRowGrab; t < t1; ++t) {
            const int32_t v = __builtin_amdgcn_readfirstlane(a.small[t]);
            const int64_t e0 = ro[v];
            const int32_t d = __builtin_amdgcn_readfirstlane(static_cast<int32_t>(ro[v + 1] - e0));
            const int32_t NB = (d + kWave - 1) / kWave;
            for (int32_t y = lane; y < d; y += kWave) mem[y] = col[e0 + y];
            wave_lds_sync();
            if (d <= kWave) induced_bits_short(a, mem, d, M, lane);
            else induced_bits<1>(a, mem, d, NB, M, 0, lane);
            int32_t ns = 1, i = 0;
            if (BLOCKS) {
                ns = member_stripes(a, s_cuts, mem, d, s_seg[wv], s_sst[wv], lane);
                i = stripe_of(v);
            }
            wave_lds_sync();
            unsigned long long part = 0;
            induced_triangles<1, BLOCKS>(M, d, NB, ns, s_seg[wv], s_sst[wv], 0, lane, part, adder(i));
            if (!BLOCKS) acc += part;
            else if (ns == 1) flush_one(i, s_sst[wv][0], part);
            wave_lds_sync();  // before the next vertex overwrites the matrix
        }
    }
    if (!BLOCKS) {
        const unsigned long long sum = group_sum(acc);
        if (threadIdx.x == 0 && sum) atomicAdd(&a.counts[0], sum);
        return;
    }
    __syncthreads();
    if (lds_counts)
        for (int32_t q = threadIdx.x; q < nlists; q += kRowThreads)
            if (s_counts[q]) atomicAdd(&a.counts[q], s_counts[q]);
}

__global__ __launch_bounds__(kRB) void k_clear_u64(unsigned long long *p, int64_t n) {
    for (int64_t q = blockIdx.x * int64_t(kRB) + threadIdx.x; q < n; q += int64_t(gridDim.x) * kRB) p[q] = 0ull;
}

}  // namespace

double quad_rows(pgabb_graph *g, std::vector<uint64_t> &per_list) {
    hipStream_t s = g->stream;
    const int32_t n = g->n, p = g->p;
    const int32_t nlists = quad_index(0, 0, 0, p);
    per_list.assign(static_cast<size_t>(nlists), 0);
    RowArgs a;
    a.row_off = g->row_off.get();
    a.col = g->col.get();
    a.p = p;
    // the hub matrix: rows padded to whole 64-bit words
    int32_t hubs = std::min(n, g->max_out > kWave ? kHubRanks : kHubRanksShort);
    DArray<uint32_t> hub;
    for (;; hubs = hubs > kHubRanksLeast ? hubs / 2 : 0) {
        a.hub_words = (hubs + 63) / 64 * 2;
        try {
            hub.reset(static_cast<size_t>(hubs) * a.hub_words, s);
            break;
        } catch (const Error &e) {
            if (e.status != PGABB_ENOMEM || hubs == 0) throw;
        }
    }
    a.hub_lo = n - hubs;
    a.hub = hub.get();
    DArray<int32_t> lists(static_cast<size_t>(n) + static_cast<size_t>(g->m / kWaveRow) + 1, s);
    a.small = lists.get();
    a.big = lists.get() + n;  // at most m' / kWaveRow rows are longer than kWaveRow
    constexpr int32_t kCtr = (1 + kRowQueues) * kRowQueueStride;
    DArray<unsigned long long> ctr(static_cast<size_t>(nlists) + kCtr + 1, s);  // counts, counters, class sizes
    k_clear_u64<<<std::min(grid_for(nlists + kCtr + 1, kRB), 1024u), kRB, 0, s>>>(ctr.get(), nlists + kCtr + 1);
    a.counts = ctr.get();
    a.next = ctr.get() + nlists;
    unsigned int *num = reinterpret_cast<unsigned int *>(ctr.get() + nlists + kCtr);
    a.num = num;
    DArray<int32_t> dcuts(static_cast<size_t>(p) + 1, s);
    Staged<int32_t> hcuts(static_cast<size_t>(p) + 1, s);
    std::copy(g->cuts.begin(), g->cuts.end(), hcuts.get());
    PGABB_HIP(hipMemcpyAsync(dcuts.get(), hcuts.get(), hcuts.bytes(), hipMemcpyHostToDevice, s));
    a.cuts = dcuts.get();
    StreamTimer tm;
    tm.start(s);
    if (hubs)
        k_hub_rows<<<std::min(grid_for(hubs, kRB / kWave), 4096u), kRB, 0, s>>>(a.row_off, a.col, a.hub_lo, n,
                                                                                a.hub_words, hub.get());
    k_row_classes<<<grid_for(n, 4 * kRB), kRB, 0, s>>>(a.row_off, n, lists.get() + n, lists.get(), num);
    if (p == 1) k_quad_rows<false><<<256, kRowThreads, 0, s>>>(a);
    else k_quad_rows<true><<<256, kRowThreads, 0, s>>>(a);
    PGABB_HIP(hipGetLastError());
    tm.stop(s);
    Staged<unsigned long long> h(static_cast<size_t>(nlists), s);
    PGABB_HIP(hipMemcpyAsync(h.get(), a.counts, h.bytes(), hipMemcpyDeviceToHost, s));
    PGABB_HIP(hipStreamSynchronize(s));
    std::copy(h.get(), h.get() + nlists, per_list.begin());
    return tm.ms();
}

uint64_t quad_rows_count(const std::vector<uint64_t> &per_list, const std::array<int32_t, 4> &q) {
    return per_list[static_cast<size_t>(quad_index(q[0], q[1], q[2], q[3]))];
}

}  // namespace pgabb
