// Build phase: edge list -> cleaned, degree-ranked, oriented CSR on device.
//
// Steps (PGAbB Section 5.1: inputs made undirected and deduplicated;
// Section 5.4: degree-based vertex ordering, triangle counting needs only
// half of the edges):
//   1. pack each pair as key = min << nb | max, self-loops -> sentinel
//   2. radix sort the keys, keep the first of every run (dedupe)
//   3. deg[v] = number of distinct pairs touching v
//   4. rank = position in ascending (deg, id): a stable sort of the degrees
//      with the ids as values (ties keep id order)
//   5. relabel both ends to ranks, key = lo << nb | hi, radix sort again;
//      rows (lo) and sorted columns (hi) give the oriented CSR
#include <algorithm>

#include "common.hpp"
#include "graph.hpp"
#include "radix.hpp"
#include "rules.hpp"
#include "wave.hpp"

namespace pgabb {

namespace {

constexpr int B = 256;
constexpr uint64_t kSentinel = ~0ull;
// Up to this many pairs the high ends are counted with one atomic each (64 K
// of them take less than the launches of a sort); above they are sorted.
constexpr int64_t kHiAtomics = 65536;
// Up to this many dedupe tiles each adds up the counts before its own (64 KB
// from L2); above they are scanned first.
constexpr int64_t kUniqDirect = 16384;

// Key of pair e, stored in keys; an endpoint out of range sets *bad and gives
// the sentinel.
struct PairKeys {
    const int32_t *src, *dst;
    int32_t n;
    int nb;
    uint64_t *keys;
    uint32_t *bad;
    __device__ __forceinline__ uint64_t operator()(int64_t e) const {
        const int32_t a = src[e], b = dst[e];
        uint64_t key = kSentinel;
        if (a < 0 || b < 0 || a >= n || b >= n) {
            *bad = 1u;
        } else if (a != b) {
            const uint64_t lo = static_cast<uint32_t>(a < b ? a : b);
            const uint64_t hi = static_cast<uint32_t>(a < b ? b : a);
            key = (lo << nb) | hi;
        }
        keys[e] = key;
        return key;
    }
};

template <class Make>
__global__ void k_make_one(Make make) {
    make(0);
}

// Dedupe: a tile of UT keys per workgroup.  The first launch counts the keys
// that are the first of a run of equal valid keys; the second adds up the
// counts of the tiles before its own, places its first keys, and makes the
// degrees' parts on the way.  (Flags, a scan of them, a compaction and a pass
// over the result for the low ends' run lengths moved twice the bytes: 270 ->
// 125 us for the 16.8 M keys of R-MAT scale 20.)
constexpr int kUniqPer = 8;
constexpr int64_t UT = int64_t(B) * kUniqPer;

__global__ __launch_bounds__(B) void k_uniq_count(const uint64_t *__restrict__ keys, int64_t m, uint64_t valid_limit,
                                                  uint32_t *__restrict__ sums) {
    __shared__ uint32_t wt[B / 64];
    const int64_t base = blockIdx.x * UT;
    uint32_t c = 0;
#pragma unroll
    for (int q = 0; q < kUniqPer; ++q) {
        const int64_t e = base + q * B + threadIdx.x;
        if (e < m) {
            const uint64_t k = keys[e];
            c += (k < valid_limit && (e == 0 || keys[e - 1] != k)) ? 1u : 0u;
        }
    }
    c = wave_sum(c);
    if (lane_id() == 0) wt[threadIdx.x >> 6] = c;
    __syncthreads();
    if (threadIdx.x == 0) {
        uint32_t t = 0;
        for (int w = 0; w < B / 64; ++w) t += wt[w];
        sums[blockIdx.x] = t;
    }
}

// Distinct keys, in order, to out[0, m') (total: m').  They are sorted by (lo,
// hi), so the low ends form runs: start[lo] and end[lo] are the run's bounds
// (0, 0 without one).  The high ends go to his (to be sorted and counted: on
// large inputs scattered atomics on hub vertices would serialise), or, with
// his null, each adds one to deg_hi.
template <bool SCANNED>
__global__ __launch_bounds__(B) void k_uniq_write(const uint64_t *__restrict__ keys, int64_t m, uint64_t valid_limit,
                                                  int nb, const uint32_t *__restrict__ sums,
                                                  uint64_t *__restrict__ out, uint32_t *__restrict__ start,
                                                  uint32_t *__restrict__ end, uint32_t *__restrict__ his,
                                                  uint32_t *__restrict__ deg_hi, uint32_t *__restrict__ total) {
    __shared__ uint32_t wt[B / 64];
    const int w = threadIdx.x >> 6, lane = lane_id();
    const uint64_t mask = (1ull << nb) - 1;
    uint32_t at = 0;  // distinct keys before this tile
    if (SCANNED) {
        at = sums[blockIdx.x];
    } else {
        for (uint32_t q = threadIdx.x; q < blockIdx.x; q += B) at += sums[q];
        at = wave_sum(at);
        if (lane == 0) wt[w] = at;
        __syncthreads();
        at = 0;
        for (int q = 0; q < B / 64; ++q) at += wt[q];
        __syncthreads();
    }
    const int64_t base = blockIdx.x * UT;
    const uint64_t below = lane ? (~0ull >> (64 - lane)) : 0ull;
#pragma unroll
    for (int q = 0; q < kUniqPer; ++q) {
        const int64_t e = base + q * B + threadIdx.x;
        uint64_t k = ~0ull, prev = ~0ull;
        if (e < m) {
            k = keys[e];
            if (e > 0) prev = keys[e - 1];
        }
        const bool first = e < m && k < valid_limit && (e == 0 || prev != k);
        const uint64_t firsts = __ballot(first);
        if (lane == 0) wt[w] = static_cast<uint32_t>(__popcll(firsts));
        __syncthreads();
        uint32_t pos = at + static_cast<uint32_t>(__popcll(firsts & below));
        for (int x = 0; x < B / 64; ++x) {
            if (x < w) pos += wt[x];
            at += wt[x];
        }
        __syncthreads();
        // the run of the key before ends where a new low end (or the sentinels) begins
        const bool prev_valid = e < m && e > 0 && prev < valid_limit;
        if (prev_valid && (k >= valid_limit || (prev >> nb) != (k >> nb))) end[prev >> nb] = pos;
        if (first) {
            const uint32_t hi = static_cast<uint32_t>(k & mask);
            out[pos] = k;
            if (e == 0 || (prev >> nb) != (k >> nb)) start[k >> nb] = pos;
            if (his) his[pos] = hi;
            else atomicAdd(&deg_hi[hi], 1u);
        }
        if (e == m - 1) {
            const uint32_t after = pos + (first ? 1u : 0u);
            *total = after;
            if (k < valid_limit) end[k >> nb] = after;
        }
    }
}

// The high ends' counts from ends that are sorted by all but their low
// kLowBits bits: a workgroup counts the low bits of `tile` consecutive ends in
// LDS, one value of the high bits after the other, and adds what it found.  (A
// full sort and run lengths took three passes and 54 us for the 15.7 M ends
// of R-MAT scale 20, 316 us; one pass and this, 59 us, take 162.  Builds of
// scale 18 768 -> 718 us, 20 1938 -> 1778, 21 4205 -> 3911.  With 11 / 12 bits
// scale 20 takes 1896 / 1768, scale 21 4142 / 4138, for a second pass; 14 would
// leave two workgroups a CU.)
constexpr int kLowBits = 13;

__global__ __launch_bounds__(B) void k_degrees_hi(const uint32_t *__restrict__ his, int64_t m, int64_t tile,
                                                  uint32_t *__restrict__ deg_hi) {
    __shared__ uint32_t cnt[1 << kLowBits];
    const int64_t t1 = min((blockIdx.x + int64_t(1)) * tile, m);
    for (int64_t pos = blockIdx.x * tile; pos < t1;) {
        // [pos, end): the ends with pos's high bits
        const uint32_t high = his[pos] >> kLowBits;
        int64_t end = t1;
        if (his[t1 - 1] >> kLowBits != high) {
            int64_t lo = pos;  // last known in, end: first known out
            end = t1 - 1;
            while (end - lo > 1) {
                const int64_t mid = (lo + end) >> 1;
                if (his[mid] >> kLowBits == high) lo = mid;
                else end = mid;
            }
        }
        for (int q = threadIdx.x; q < 1 << kLowBits; q += B) cnt[q] = 0;
        __syncthreads();
#pragma unroll 8
        for (int64_t e = pos + threadIdx.x; e < end; e += B) atomicAdd(&cnt[his[e] & ((1u << kLowBits) - 1)], 1u);
        __syncthreads();
        for (int q = threadIdx.x; q < 1 << kLowBits; q += B)
            if (cnt[q]) atomicAdd(&deg_hi[(high << kLowBits) + q], cnt[q]);
        __syncthreads();
        pos = end;
    }
}

// The same from ends that are sorted by all bits: each run of equal ends adds
// its length once.
__global__ __launch_bounds__(B) void k_degrees_runs(const uint32_t *__restrict__ his, int64_t m,
                                                    int32_t *__restrict__ deg_hi) {
    const int64_t stride = int64_t(gridDim.x) * B;
    for (int64_t base = blockIdx.x * int64_t(B) + (threadIdx.x & ~63); base < m; base += stride) {
        const int64_t e = base + lane_id();
        const bool valid = e < m;
        add_run_lengths(valid, valid ? static_cast<int64_t>(his[e]) : 0, deg_hi);
    }
}

// Degree of vertex v, stored in deg.
struct Degrees {
    const uint32_t *start, *end, *deg_hi;
    int32_t *deg;
    __device__ __forceinline__ uint32_t operator()(int64_t v) const {
        const uint32_t d = end[v] - start[v] + deg_hi[v];
        deg[v] = static_cast<int32_t>(d);
        return d;
    }
};

// The rank sort's keys and values.
struct DegreeKeys {
    Degrees degree;
    uint32_t *dk, *dv;
    __device__ __forceinline__ uint32_t operator()(int64_t v) const {
        const uint32_t d = degree(v);
        dk[v] = d;
        dv[v] = static_cast<uint32_t>(v);
        return d;
    }
};

// The degrees, and ranks in id order.
__global__ void k_degrees_by_id(Degrees degree, int32_t n, int32_t *__restrict__ rank) {
    for (int64_t v = blockIdx.x * int64_t(B) + threadIdx.x; v < n; v += int64_t(gridDim.x) * B) {
        degree(v);
        rank[v] = static_cast<int32_t>(v);
    }
}

// Key of distinct pair e by the ends' ranks.
struct OrientedKeys {
    const uint64_t *ukeys;
    int nb;
    const int32_t *rank;
    uint64_t *okeys;
    __device__ __forceinline__ uint64_t operator()(int64_t e) const {
        const uint64_t k = ukeys[e];
        const uint32_t ra = static_cast<uint32_t>(rank[k >> nb]);
        const uint32_t rb = static_cast<uint32_t>(rank[k & ((1ull << nb) - 1)]);
        const uint64_t lo = ra < rb ? ra : rb, hi = ra < rb ? rb : ra;
        const uint64_t key = (lo << nb) | hi;
        okeys[e] = key;
        return key;
    }
};

__global__ void k_row_counts_and_cols(const uint64_t *__restrict__ okeys, int64_t m, int nb,
                                      int32_t *__restrict__ outdeg, int32_t *__restrict__ col) {
    const uint64_t mask = (1ull << nb) - 1;
    const int64_t stride = int64_t(gridDim.x) * B;
    for (int64_t base = blockIdx.x * int64_t(B) + (threadIdx.x & ~63); base < m; base += stride) {
        const int64_t e = base + lane_id();
        const bool valid = e < m;
        const uint64_t k = valid ? okeys[e] : 0ull;
        add_run_lengths(valid, static_cast<int64_t>(k >> nb), outdeg);
        if (valid) col[e] = static_cast<int32_t>(k & mask);
    }
}

// Workgroups of k_vertex_stats, each of which adds to the same nine words: with
// 128 / 256 / 512 / 1,024 of them builds of R-MAT scale 18 take 691 / 692 / 697
// / 721 us, scale 20 1788 / 1769 / 1741 / 1793.
constexpr unsigned kStatGrid = 512;

struct Stats {
    int32_t max_out;
    int32_t max_in;
    unsigned long long sum[kStatSums];  // by Stat
};

// Per vertex v (rank r): indeg[r] = deg[v] - outdeg[r], the edges of v
// whose other end ranks lower; and the statistics, reduced per workgroup
// (one atomic each; launched with a small grid): the longest row and column,
// the isolated vertices, the probe work W = sum over oriented edges (x, y) of
// outdeg[y] = sum over y of indeg[y] outdeg[y], and what a partition into one
// block needs to know of it.
__global__ __launch_bounds__(B) void k_vertex_stats(const int32_t *__restrict__ deg,
                                                    const int32_t *__restrict__ rank,
                                                    const int32_t *__restrict__ outdeg, int32_t n,
                                                    int32_t *__restrict__ indeg, Stats *st) {
    __shared__ int32_t s_mx[B / 64][2];
    __shared__ unsigned long long s_sum[B / 64][kStatSums];
    int32_t mo = 0, mi = 0;
    unsigned long long sum[kStatSums] = {};
    for (int64_t v = blockIdx.x * int64_t(B) + threadIdx.x; v < n; v += int64_t(gridDim.x) * B) {
        const int32_t r = rank[v];
        const int32_t o = outdeg[r], i = deg[v] - o;
        indeg[r] = i;
        mo = max(mo, o);
        mi = max(mi, i);
        sum[kStatIsolated] += deg[v] == 0;
        sum[kStatProbeWork] += static_cast<unsigned long long>(i) * static_cast<unsigned long long>(o);
        sum[kStatRowSquares] += static_cast<unsigned long long>(o) * static_cast<unsigned long long>(o);
        sum[kStatRows] += o > 0;
        sum[kStatCols] += i > 0;
        sum[kStatRowItems] += (o + kSplitV - 1) / kSplitV;
        sum[kStatColItems] += (i + kSplitV - 1) / kSplitV;
    }
#pragma unroll
    for (int d = 1; d < kWave; d <<= 1) {
        mo = max(mo, __shfl_xor(mo, d));
        mi = max(mi, __shfl_xor(mi, d));
    }
#pragma unroll
    for (int q = 0; q < kStatSums; ++q) sum[q] = wave_sum(sum[q]);
    if (lane_id() == 0) {
        s_mx[threadIdx.x >> 6][0] = mo;
        s_mx[threadIdx.x >> 6][1] = mi;
        for (int q = 0; q < kStatSums; ++q) s_sum[threadIdx.x >> 6][q] = sum[q];
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        for (int q = 1; q < B / 64; ++q) {
            mo = max(mo, s_mx[q][0]);
            mi = max(mi, s_mx[q][1]);
        }
        atomicMax(&st->max_out, mo);
        atomicMax(&st->max_in, mi);
    }
    if (threadIdx.x < kStatSums) {
        unsigned long long t = 0;
        for (int q = 0; q < B / 64; ++q) t += s_sum[q][threadIdx.x];
        if (t) atomicAdd(&st->sum[threadIdx.x], t);
    }
}

unsigned cap_grid(int64_t work) {
    unsigned g = grid_for(work, B);
    return g > 65536u ? 65536u : g;
}

}  // namespace

void build_graph(pgabb_graph *g, const int32_t *src, const int32_t *dst, int64_t m) {
    hipStream_t s = g->stream;
    const int32_t n = g->n;
    g->m_input = m;
    g->nb = std::max(1, bit_width_u64(n > 0 ? static_cast<uint64_t>(n - 1) : 0));
    const int nb = g->nb;

    g->rank.reset(static_cast<size_t>(n), s);
    g->outdeg.reset(static_cast<size_t>(n), s);
    g->indeg.reset(static_cast<size_t>(n), s);
    g->row_off.reset(static_cast<size_t>(n) + 1, s);
    if (n > 0) PGABB_HIP(hipMemsetAsync(g->outdeg.get(), 0, sizeof(int32_t) * n, s));
    else PGABB_HIP(hipMemsetAsync(g->row_off.get(), 0, sizeof(int64_t), s));  // (else written by the scan)

    DArray<int32_t> deg(static_cast<size_t>(n), s);
    g->m = 0;
    // what starts at zero, cleared at once: the statistics, two words (an
    // endpoint lay out of range; distinct edges), the low ends' run bounds and
    // the high ends' counts
    constexpr size_t kHead = (sizeof(Stats) + sizeof(uint32_t) - 1) / sizeof(uint32_t);
    const size_t nz = kHead + 2 + 3 * static_cast<size_t>(n);
    DArray<uint32_t> zeroed(nz, s);
    PGABB_HIP(hipMemsetAsync(zeroed.get(), 0, nz * sizeof(uint32_t), s));
    Stats *st = reinterpret_cast<Stats *>(zeroed.get());
    uint32_t *meta = zeroed.get() + kHead, *run_start = meta + 2, *run_end = run_start + n, *deg_hi = run_end + n;

    const Degrees degrees{run_start, run_end, deg_hi, deg.get()};
    if (m > 0) {
        DArray<uint64_t> keys(static_cast<size_t>(m), s), alt(static_cast<size_t>(m), s);
        // Out-of-range edges get the sentinel key, so sorting and compacting
        // them is harmless and one round trip reports both words.
        const PairKeys pairs{src, dst, n, nb, keys.get(), meta};

        // 1-2: sort and dedupe.  Valid keys are below (n-1) << nb | (n-1) + 1;
        // the sentinel has every low 2nb bit set, so it sorts after them.
        const int kbits = 2 * nb;
        uint64_t *k0 = keys.get(), *k1 = alt.get();
        if (m == 1) k_make_one<<<1, 1, 0, s>>>(pairs);
        else if (radix_sort_made<uint64_t>(pairs, k0, k1, nullptr, nullptr, nullptr, m, 0, kbits, s)) std::swap(k0, k1);
        PGABB_HIP(hipGetLastError());
        const uint64_t valid_limit = (static_cast<uint64_t>(n - 1) << nb) + static_cast<uint64_t>(n);
        DArray<uint32_t> his;
        if (m > kHiAtomics) his.reset(static_cast<size_t>(m), s);
        {
            const int64_t tiles = (m + UT - 1) / UT;
            DArray<uint32_t> sums(static_cast<size_t>(tiles), s);
            k_uniq_count<<<static_cast<unsigned>(tiles), B, 0, s>>>(k0, m, valid_limit, sums.get());
            PGABB_HIP(hipGetLastError());
            if (tiles > kUniqDirect) {
                scan_exclusive_u32(sums.get(), sums.get(), tiles, nullptr, s);
                k_uniq_write<true><<<static_cast<unsigned>(tiles), B, 0, s>>>(k0, m, valid_limit, nb, sums.get(), k1,
                                                                             run_start, run_end, his.get(), deg_hi,
                                                                             meta + 1);
            } else {
                k_uniq_write<false><<<static_cast<unsigned>(tiles), B, 0, s>>>(k0, m, valid_limit, nb, sums.get(), k1,
                                                                              run_start, run_end, his.get(), deg_hi,
                                                                              meta + 1);
            }
            PGABB_HIP(hipGetLastError());
            Staged<uint32_t> mh(2, s);
            PGABB_HIP(hipMemcpyAsync(mh.get(), meta, mh.bytes(), hipMemcpyDeviceToHost, s));
            PGABB_HIP(hipStreamSynchronize(s));
            PGABB_REQUIRE(!mh[0], PGABB_EINVAL, "an edge endpoint lies outside [0, %d)", n);
            g->m = mh[1];
        }
        std::swap(k0, k1);  // k0: distinct keys [0, m')
        const int64_t mu = g->m;

        // 3: the high ends' counts, where not added one by one
        if (mu > 0 && his.get()) {
            DArray<uint32_t> his_alt(static_cast<size_t>(mu), s);
            uint32_t *hs = his.get();
            const bool low = degrees_by_low_bits(mu, n, kLowBits);
            if (radix_sort_impl<uint32_t>(his.get(), his_alt.get(), nullptr, nullptr, mu, low ? kLowBits : 0, nb, s))
                hs = his_alt.get();
            // tiles for some 512 workgroups, long enough for their LDS to pay
            const int64_t tile = std::min<int64_t>(std::max<int64_t>(mu / 512, 8192), 65536);
            if (low) k_degrees_hi<<<static_cast<unsigned>((mu + tile - 1) / tile), B, 0, s>>>(hs, mu, tile, deg_hi);
            else k_degrees_runs<<<cap_grid(mu), B, 0, s>>>(hs, mu, reinterpret_cast<int32_t *>(deg_hi));
            PGABB_HIP(hipGetLastError());
        }
        // 4: degrees and ranks
        if ((g->flags & PGABB_ORDER_BY_ID) || n == 1) {
            k_degrees_by_id<<<cap_grid(n), B, 0, s>>>(degrees, n, g->rank.get());
            PGABB_HIP(hipGetLastError());
        } else {
            DArray<uint32_t> dk(n, s), dka(n, s), dv(n, s), dva(n, s);
            radix_sort_made<uint32_t>(DegreeKeys{degrees, dk.get(), dv.get()}, dk.get(), dka.get(), dv.get(), dva.get(),
                                      g->rank.get(), n, 0, nb, s);
        }

        // 5: orient and sort by (row, col)
        if (mu > 0) {
            const OrientedKeys oriented{k0, nb, g->rank.get(), k1};
            if (mu == 1) k_make_one<<<1, 1, 0, s>>>(oriented);
            else if (radix_sort_made<uint64_t>(oriented, k1, k0, nullptr, nullptr, nullptr, mu, 0, kbits, s))
                std::swap(k0, k1);
            PGABB_HIP(hipGetLastError());
            // sorted oriented keys now in k1
            // (rows are read in segments, which may reach past the last one)
            g->col.reset(static_cast<size_t>(mu) + kSeg, s);
            k_row_counts_and_cols<<<cap_grid(mu), B, 0, s>>>(k1, mu, nb, g->outdeg.get(), g->col.get());
            PGABB_HIP(hipGetLastError());
        }
    } else if (n > 0) {
        k_degrees_by_id<<<cap_grid(n), B, 0, s>>>(degrees, n, g->rank.get());  // every degree 0
        PGABB_HIP(hipGetLastError());
    }
    if (g->m == 0) g->col.release();

    // statistics for sizing kernels and stating algorithmic bytes
    if (n > 0) {
        scan_exclusive_i32(g->outdeg.get(), g->row_off.get(), n, g->row_off.get() + n, s);
        k_vertex_stats<<<std::min(cap_grid(n), kStatGrid), B, 0, s>>>(deg.get(), g->rank.get(), g->outdeg.get(), n,
                                                                  g->indeg.get(), st);
        PGABB_HIP(hipGetLastError());
    }
    Staged<Stats> hs(1, s);
    PGABB_HIP(hipMemcpyAsync(hs.get(), st, sizeof(Stats), hipMemcpyDeviceToHost, s));
    PGABB_HIP(hipStreamSynchronize(s));
    g->max_out = hs[0].max_out;
    g->max_in = hs[0].max_in;
    for (int q = 0; q < kStatSums; ++q) g->stat[q] = hs[0].sum[q];
    g->isolated = static_cast<int64_t>(g->stat[kStatIsolated]);
    g->probe_work = g->stat[kStatProbeWork];
}

}  // namespace pgabb
