// Triangles containing each edge (edge support): the per-edge quantity behind
// clustering coefficients (PGAbB Section 1) and the peeling of k-truss
// (Section 3.2), from the same intersections as the count (Section 3.6) with
// a different reduction.  The oriented graph is taken as one block (p = 1):
// every triangle r(a) < r(b) < r(c) is found once, as the common entry c of
// N+(a) and N+(b) for the edge (a, b), and adds one to each of its edges
// (a, b), (a, c) and (b, c).
//
// The edge is reached from its higher end: one wave owns a vertex b at a
// time, stages N+(b) in LDS with one counter per entry, and for every in-edge
// (a, b) walks the part of N+(a) after b (only c > b can lie in N+(b)) in
// segments of kSeg entries, one per lane and load, flattened over the lanes
// (tc_device.hpp), looking each walked entry up.  This reads sum_a d+(a)
// (d+(a) - 1) / 2 entries, against sum over edges (a, b) of d+(b) when every
// N+(b) is walked from the lower end (3.6 x more on R-MAT scale 20).  A hit
// counts (b, c) in LDS (flushed once per unit), (a, b) in a per-in-edge LDS
// counter (flushed once per unit) and (a, c), the walked entry, with a device
// atomic.
//
// N+(b) is staged as a bitmap of the kSupHubs highest ranks ("hubs", which
// hold most walked entries on skewed graphs) with the number of entries
// before each word, so an entry is found, and its position known, with no
// search.  A row with entries below the hubs goes to a hash table instead, all of
// it where it fits (kSupWideCap).  Held in one hash table (load up to 2/3, probed
// until the last of 64 lanes is done, one entry a lane) a chunk of 64 walked
// entries cost 105 vector and 97 scalar instructions and the pass was bound by
// them: R-MAT scale 20 7.15 ms with the walked-edge atomics, 6.50 without.  Now
// 4.25 ms, bound by the 424 M device atomics, which go past the L2s (2.8 ms of
// them; one segment per lane in each atomic instruction, touching four times the
// lines, took 9.8 ms).
//
// Work units are runs of at most 64 in-edges of one owner (one per lane), so
// an owner with many in-edges spreads over many waves (each stages N+(b) and
// flushes its own counters); units are listed from the highest rank down (the
// hubs, whose in-edges are many, start first), only for owners with both
// in-edges and a non-empty row, and dealt round-robin to eight work counters.
// Rows that do not fit the LDS region are searched and counted in device
// memory.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <chrono>
#include <cstddef>

#include "common.hpp"
#include "graph.hpp"
#include "tc_device.hpp"
#include "wave.hpp"

namespace pgabb {

namespace {

constexpr int kSupWaves = 4;
constexpr int kSupB = 256;
constexpr int kSupHubs = 8192;                // ranks of the bitmap: four words a lane
constexpr int kSupWords = kSupHubs / 32;
constexpr int kSupCap = 1024;                 // longest row staged in LDS
constexpr int kSupLowCap = 341;               // entries below the hubs that are (table load <= 2/3)
constexpr int kSupTableLg = 9;
// Rows with entries below the hubs, up to this length, take the whole LDS region
// for one table of all their entries, counted by slot: an entry is looked up
// once, not in the bitmap and then in a table, and dense graphs of more than
// kSupHubs vertices without skew keep their rows in LDS.  Kernel ms, every row in
// one hash table of 1,024 slots / bitmap and table, longer low rows searched in
// device memory / now: 64 complete graphs of 600 vertices 8.9 / 18.5 / 8.5; random
// geometric graphs of 20,011 vertices at degree 300 1.94 / 1.66 / 1.07, 600 5.6 /
// 7.8 / 4.0, 1000 14.4 / 14.4 / 12.6; Erdos-Renyi, 100,001 vertices at degree 100
// 0.92 / 0.68 / 0.39; R-MAT scale 20 7.1 / 4.96 / 4.25.
constexpr int kSupWideCap = 682;
constexpr int kSupWideLg = 10;
// A segment's entries take this many steps through the table together, so that
// their reads overlap; what is left of each then runs by itself, since together
// all wait for the longest of 256 (0 / 1 / 2 / all steps together: degree 1000
// 14.5 / 13.9 / 12.6 / 16.6, 600 4.0 / 4.1 / 4.0 / 4.4).
constexpr int kSupJoined = 2;
constexpr int kSupUnitEdges = kWave;  // in-edges per work unit (one per lane)
// Units per grab (random geometric graph, 200,003 vertices: 549 us at 1, 399
// at 2, 347 at 4, where a unit is a short chain of dependent loads).
constexpr int kSupGrab = 4;
constexpr int kSupQueues = 8;       // work counters, kSupQueueStride words apart
constexpr int kSupQueueStride = 32;

struct SupportLds {
    union {
        struct {
            int32_t key[1 << kSupTableLg];     // hash table of the entries below the hubs: entry, or -1
            uint16_t pos[1 << kSupTableLg];    // its position in the row
            uint32_t cnt[kSupCap / 4];         // triangles found on edge (b, row[x]), a byte each: a unit's
                                               // 64 in-edges find at most one each
            uint32_t bits[kSupWords + 1];      // N+(b)'s hubs; a zero word after them
            uint16_t before[kSupWords + 2];    // N+(b)'s hubs before each word
        };
        struct {  // rows up to kSupWideCap entries, some of them below the hubs
            int32_t wide_key[1 << kSupWideLg];       // hash table of all entries
            uint32_t wide_cnt[(1 << kSupWideLg) / 4];  // the triangles, by slot
        };
    };
    uint32_t own[kWave];               // list positions of the flattened walk
    uint32_t hits[kWave];              // triangles found on each in-edge of the unit
};
static_assert(offsetof(SupportLds, wide_cnt) + sizeof(SupportLds::wide_cnt) <=
                  offsetof(SupportLds, bits) + kSupWords * sizeof(uint32_t),
              "a wide row leaves the zero word");

// Entries after every CSR position in its row: the length of the walk an
// in-edge at that position starts.
__global__ __launch_bounds__(kSupB) void k_sup_rest(const int64_t *__restrict__ row_off, int32_t n,
                                                     int32_t *__restrict__ rest) {
    for_row_entries(row_off, n, [&](int32_t, int64_t e, int64_t e1) { rest[e] = static_cast<int32_t>(e1 - e - 1); });
}

// Work units of every owner, in processing order (rank n - 1 first): one per
// kSupUnitEdges in-edges when the owner has in-edges and a non-empty row.
__global__ __launch_bounds__(kSupB) void k_sup_unit_counts(const int64_t *__restrict__ row_off,
                                                            const int64_t *__restrict__ in_off, int32_t n,
                                                            int64_t *__restrict__ units) {
    for (int64_t r = blockIdx.x * static_cast<int64_t>(kSupB) + threadIdx.x; r < n;
         r += static_cast<int64_t>(gridDim.x) * kSupB) {
        const int64_t b = n - 1 - r;
        const int64_t d = row_off[b + 1] - row_off[b], nin = in_off[b + 1] - in_off[b];
        units[r] = (d > 0 && nin > 0) ? (nin + kSupUnitEdges - 1) / kSupUnitEdges : 0;
    }
}

// The unit list: (owner, first in-edge of the owner's unit).
__global__ __launch_bounds__(kSupB) void k_sup_unit_fill(const int64_t *__restrict__ upre, int32_t n,
                                                          int2 *__restrict__ units) {
    for (int64_t r = blockIdx.x * static_cast<int64_t>(kSupB) + threadIdx.x; r < n;
         r += static_cast<int64_t>(gridDim.x) * kSupB) {
        const int64_t u0 = upre[r], c = upre[r + 1] - u0;
        for (int64_t j = 0; j < c; ++j)
            units[u0 + j] = make_int2(static_cast<int32_t>(n - 1 - r), static_cast<int32_t>(j * kSupUnitEdges));
    }
}

// Sort keys (the higher end of each edge) and values (its CSR position).
__global__ __launch_bounds__(kSupB) void k_sup_pairs(const int32_t *__restrict__ col, int64_t m,
                                                      uint32_t *__restrict__ key, uint32_t *__restrict__ val) {
    for (int64_t e = blockIdx.x * static_cast<int64_t>(kSupB) + threadIdx.x; e < m;
         e += static_cast<int64_t>(gridDim.x) * kSupB) {
        key[e] = static_cast<uint32_t>(col[e]);
        val[e] = static_cast<uint32_t>(e);
    }
}

__global__ __launch_bounds__(kSupB) void k_sup_widen(const int32_t *__restrict__ in, int32_t n,
                                                      int64_t *__restrict__ out) {
    for (int64_t v = blockIdx.x * static_cast<int64_t>(kSupB) + threadIdx.x; v < n;
         v += static_cast<int64_t>(gridDim.x) * kSupB)
        out[v] = in[v];
}

// Six waves per SIMD, what the LDS leaves room for, at the price of four spilled
// registers (20 bytes of scratch a lane).  Left alone the compiler takes 94, five
// waves: R-MAT scale 20 4.39 ms against 4.27, Erdos-Renyi of degree 100 0.45
// against 0.39, a random geometric graph of degree 24 0.286 against 0.273; dense
// geometric graphs gain up to 6 % without (degree 500 2.64 against 2.80).
__global__ __launch_bounds__(kSupWaves *kWave) __attribute__((amdgpu_waves_per_eu(6)))
void k_edge_support(const int64_t *__restrict__ row_off,
                                                                    const int32_t *__restrict__ col,
                                                                    const int64_t *__restrict__ in_off,
                                                                    const uint32_t *__restrict__ in_pos,
                                                                    const int32_t *__restrict__ rest,
                                                                    const int2 *__restrict__ units,
                                                                    const int64_t *__restrict__ nunits_dev,
                                                                    int32_t hub_lo,
                                                                    uint32_t *__restrict__ support,
                                                                    unsigned long long *__restrict__ next,
                                                                    unsigned long long *__restrict__ total) {
    __shared__ SupportLds s_lds[kSupWaves];
    SupportLds &L = s_lds[threadIdx.x / kWave];
    const int lane = lane_id();
    const gptr<int64_t> ro = as_global(row_off);
    const gptr<int32_t> cl = as_global(col);
    const gptr<int64_t> io = as_global(in_off);
    const gptr<uint32_t> ip = as_global(in_pos);
    const gptr<int32_t> rs = as_global(rest);
    L.own[lane] = 0;
    if (lane == 0) L.bits[kSupWords] = 0u;
    wave_lds_sync();
    const gptr<int32_t> un = as_global(reinterpret_cast<const int32_t *>(units));  // (owner, first in-edge) pairs
    const int64_t nunits = *as_global(nunits_dev);
    unsigned long long found = 0;
    // units per grab: kSupGrab share their headers' round trips; one where that
    // would leave waves without units (R-MAT scale 12, 77 us: 96 at four)
    const int64_t waves = static_cast<int64_t>(gridDim.x) * kSupWaves;
    const int grab = static_cast<int>(max(min(nunits / (4 * waves), static_cast<int64_t>(kSupGrab)),
                                          static_cast<int64_t>(1)));
    UnitTaker<kSupQueues, kSupQueueStride> taker(next, (nunits + grab - 1) / grab, waves,
                                                 static_cast<int64_t>(blockIdx.x) * kSupWaves + threadIdx.x / kWave);
    for (int64_t g; (g = taker.take(lane)) >= 0;) {
        const int64_t u0 = g * grab;
        const int ng = static_cast<int>(min(nunits - u0, static_cast<int64_t>(grab)));
        // the units' headers, one per lane; then per unit its in-edges, one per
        // lane (position of (a, b) and its walk's length), and the first 64
        // entries of N+(b): four round trips for the whole grab
        int32_t hb = 0, hd = 0, hin = 0;
        int64_t hb0 = 0, hi0 = 0;
        if (lane < ng) {
            hb = un[2 * (u0 + lane)];
            const int32_t i = un[2 * (u0 + lane) + 1];
            hb0 = ro[hb];
            hd = static_cast<int32_t>(ro[hb + 1] - hb0);
            hi0 = io[hb] + i;
            hin = static_cast<int32_t>(min(io[hb + 1] - hi0, static_cast<int64_t>(kSupUnitEdges)));
        }
        uint32_t g_eab[kSupGrab];
        int32_t g_len[kSupGrab], g_v0[kSupGrab];
#pragma unroll
        for (int j = 0; j < kSupGrab; ++j) {  // (hin, hd: 0 past the grab's end)
            const int64_t i0 = shfl_t(hi0, j), b0 = shfl_t(hb0, j);  // (every lane shuffles)
            g_eab[j] = lane < __builtin_amdgcn_readlane(hin, j) ? ip[i0 + lane] : 0u;
            g_v0[j] = lane < __builtin_amdgcn_readlane(hd, j) ? cl[b0 + lane] : 0;
        }
#pragma unroll
        for (int j = 0; j < kSupGrab; ++j)
            g_len[j] = lane < __builtin_amdgcn_readlane(hin, j) ? rs[g_eab[j]] : 0;
#pragma unroll 1
        for (int j = 0; j < ng; ++j) {
        const int32_t d = __builtin_amdgcn_readlane(hd, j);
        const int32_t nin = __builtin_amdgcn_readlane(hin, j);
        const int64_t b0 = shfl_t(hb0, j);
        uint32_t eab = g_eab[0];
        int32_t len = g_len[0], v0 = g_v0[0];
#pragma unroll
        for (int q = 1; q < kSupGrab; ++q)
            if (j == q) {
                eab = g_eab[q];
                len = g_len[q];
                v0 = g_v0[q];
            }
        // ---- stage N+(b): its entries below the hubs are its first `low`
        int32_t low = __popcll(__ballot(lane < d && v0 < hub_lo));
        for (int32_t x0 = kWave; x0 < d && low == x0; x0 += kWave) {
            const int32_t x = x0 + lane;
            low += __popcll(__ballot(x < d && cl[b0 + x] < hub_lo));
        }
        const bool wide = low > 0 && d <= kSupWideCap;
        const bool staged = wide || (d <= kSupCap && low <= kSupLowCap);
        if (wide) low = d;
        const int32_t table_end = wide ? INT32_MAX : hub_lo;  // entries below it are in the table
        const bool hubs = d > low;
        int lg = 6;  // table of 2^lg >= 3 low slots, as far as they are there (1.5 low are)
        while ((1 << lg) < 3 * low && lg < (wide ? kSupWideLg : kSupTableLg)) ++lg;
        int32_t *const key = L.wide_key;  // (both tables start there)
        uint32_t *const cnt = wide ? L.wide_cnt : L.cnt;
        const uint32_t tmask = (1u << lg) - 1u;
        const int shift = 24 - lg;
        if (staged) {
            if (hubs) {
#pragma unroll
                for (int q = 0; q < kSupWords / kWave; ++q) L.bits[q * kWave + lane] = 0u;
            }
            for (int x = lane; x < (wide ? 1 << lg : d + 3) / 4; x += kWave) cnt[x] = 0u;
            if (low > 0)
                for (int x = lane; x < (1 << lg); x += kWave) key[x] = -1;
            wave_lds_sync();
            for (int x = lane; x < d; x += kWave) {
                const int32_t v = x < kWave ? v0 : cl[b0 + x];
                if (v >= table_end) {
                    const int32_t h = v - hub_lo;
                    atomicOr(&L.bits[h >> 5], 1u << (h & 31));
                } else {
                    uint32_t s = hash_slot(v, shift, tmask);
                    while (atomicCAS(&key[s], -1, v) != -1) s = (s + 1) & tmask;
                    if (!wide) L.pos[s] = static_cast<uint16_t>(x);
                }
            }
            wave_lds_sync();
            if (hubs) {  // lane l takes words 4 l .. 4 l + 3
                int32_t pc[4], sum = 0;
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    pc[q] = sum;
                    sum += __popc(L.bits[4 * lane + q]);
                }
                const int32_t base = low + wave_inclusive_scan(sum) - sum;
#pragma unroll
                for (int q = 0; q < 4; ++q) L.before[4 * lane + q] = static_cast<uint16_t>(base + pc[q]);
            }
        }
        L.hits[lane] = 0;
        wave_lds_sync();
        // ---- the walk
        const int32_t nseg = segs_of(len);
        const int32_t incl = wave_inclusive_scan(nseg);
        const int32_t pre = incl - nseg;
        const int32_t tot = __builtin_amdgcn_readlane(incl, kWave - 1);
        const uint32_t rel = eab + 1u - static_cast<uint32_t>(kSeg * pre);  // segment t starts at rel + kSeg t
        const int32_t end = len + kSeg * pre;                              // entries left at segment t: end - kSeg t
        uint32_t carry = 0;
        seg_t v, vn;
        int32_t n = 0, nn = 0, sl = 0, sn = 0;
        uint32_t ev = 0, en = 0;
        auto load = [&](int32_t base, seg_t &w, int32_t &cnt, int32_t &src, uint32_t &at) {
            const int32_t p = pre - base;
            if (nseg > 0 && p >= 0 && p < kWave) L.own[p] = static_cast<uint32_t>(lane + 1);
            wave_lds_sync();
            const uint32_t o = L.own[lane];
            L.own[lane] = 0;
            wave_lds_sync();
            const uint32_t s1 = max(wave_max_scan_dpp(o), carry);
            carry = __builtin_amdgcn_readlane(s1, kWave - 1);
            const int32_t t = base + lane;
            src = static_cast<int32_t>(s1) - 1;
            at = __shfl(rel, src) + static_cast<uint32_t>(kSeg * t);
            const int32_t left = __shfl(end, src) - kSeg * t;
            const bool inb = t < tot;
            cnt = inb ? left : 0;
            w = *reinterpret_cast<const __attribute__((address_space(1))) seg_t *>(cl + (inb ? at : 0u));
        };
        int32_t acc_lo = 0;  // hits on a lane's current list gather in a register
        uint32_t acc = 0;
        auto probe = [&](int32_t segs) {  // segments in the batch
            uint32_t hits = 0;  // of the segment's entries, a bit each
            if (staged) {
                if (hubs) {
                    int32_t h[kSeg];
                    uint32_t word[kSeg];
#pragma unroll
                    for (int r = 0; r < kSeg; ++r) {
                        h[r] = v[r] - hub_lo;
                        word[r] = L.bits[r < n && h[r] >= 0 ? h[r] >> 5 : kSupWords];
                    }
#pragma unroll
                    for (int r = 0; r < kSeg; ++r) {
                        if (((word[r] >> (h[r] & 31)) & 1u) == 0u) continue;
                        const uint32_t at = L.before[h[r] >> 5] + __popc(word[r] & ((1u << (h[r] & 31)) - 1u));
                        atomicAdd(&cnt[at >> 2], 1u << (8 * (at & 3u)));
                        hits |= 1u << r;
                    }
                }
                if (low > 0) {
                    bool go[kSeg], any = false;
                    uint32_t s[kSeg];
#pragma unroll
                    for (int r = 0; r < kSeg; ++r) {
                        go[r] = r < n && v[r] < table_end;
                        s[r] = hash_slot(v[r], shift, tmask);
                        any |= go[r];
                    }
                    auto step = [&](int r) {
                        const int32_t kv = key[s[r]];
                        if (go[r] && kv == v[r]) {
                            const uint32_t at = wide ? s[r] : L.pos[s[r]];
                            atomicAdd(&cnt[at >> 2], 1u << (8 * (at & 3u)));
                            hits |= 1u << r;
                        }
                        go[r] = go[r] && kv != -1 && kv != v[r];
                        s[r] = (s[r] + 1) & tmask;
                    };
                    for (int z = 0; z < kSupJoined && __ballot(any) != 0; ++z) {
                        any = false;
#pragma unroll
                        for (int r = 0; r < kSeg; ++r) {
                            step(r);
                            any |= go[r];
                        }
                    }
#pragma unroll
                    for (int r = 0; r < kSeg; ++r)
                        while (__ballot(go[r]) != 0) step(r);
                }
            } else {
#pragma unroll
                for (int r = 0; r < kSeg; ++r) {
                    if (r >= n) continue;
                    int32_t lo = 0, hi = d;
                    while (lo < hi) {
                        const int32_t mid = (lo + hi) >> 1;
                        if (cl[b0 + mid] < v[r]) lo = mid + 1;
                        else hi = mid;
                    }
                    if (lo < d && cl[b0 + lo] == v[r]) {
                        atomicAdd(&support[b0 + lo], 1u);
                        hits |= 1u << r;
                    }
                }
            }
            // the walked edges: 16 segments at a time with one entry per lane, so
            // that an atomic instruction touches consecutive words (one segment
            // per lane would touch each line four times)
            if (__ballot(hits != 0u) == 0) return;
#pragma unroll
            for (int k = 0; k < kSeg; ++k) {
                if (k * (kWave / kSeg) >= segs) break;
                const int from = k * (kWave / kSeg) + lane / kSeg;
                const uint32_t hs = __shfl(hits, from);
                const uint32_t at = __shfl(ev, from) + static_cast<uint32_t>(lane % kSeg);
                if ((hs >> (lane % kSeg)) & 1u) atomicAdd(&support[at], 1u);
            }
            const uint32_t hit = __popc(hits);
            if (hit) {
                found += hit;
                if (sl != acc_lo) {
                    if (acc) atomicAdd(&L.hits[acc_lo], acc);
                    acc_lo = sl;
                    acc = 0;
                }
                acc += hit;
            }
        };
        if (tot > 0) {
            load(0, v, n, sl, ev);
            for (int32_t f = kWave; f < tot; f += kWave) {  // the next batch loads while one is probed
                load(f, vn, nn, sn, en);
                probe(kWave);
                v = vn;
                n = nn;
                sl = sn;
                ev = en;
            }
            probe((tot - 1) % kWave + 1);
        }
        if (acc) atomicAdd(&L.hits[acc_lo], acc);
        wave_lds_sync();
        if (lane < nin && L.hits[lane]) atomicAdd(&support[eab], L.hits[lane]);
        if (staged)
            for (int x = lane; x < d; x += kWave) {
                uint32_t at = x;
                if (wide) {  // (the entry is in the table)
                    const int32_t e = cl[b0 + x];
                    at = hash_slot(e, shift, tmask);
                    while (key[at] != e) at = (at + 1) & tmask;
                }
                const uint32_t c = (cnt[at >> 2] >> (8 * (at & 3))) & 0xffu;
                if (c) atomicAdd(&support[b0 + x], c);
            }
        wave_lds_sync();  // before the next unit is staged
        }
    }
    found = group_sum(found);
    if (threadIdx.x == 0 && found) atomicAdd(total, found);
}

}  // namespace

void in_edges(pgabb_graph *g, DArray<int64_t> &in_off, DArray<uint32_t> &in_pos) {
    hipStream_t s = g->stream;
    const int64_t m = g->m;
    const int32_t n = g->n;
    DArray<uint32_t> key(static_cast<size_t>(m), s), key_alt(static_cast<size_t>(m), s);
    DArray<uint32_t> pos(static_cast<size_t>(m), s), pos_alt(static_cast<size_t>(m), s);
    in_off.reset(static_cast<size_t>(n) + 1, s);
    k_sup_pairs<<<grid_for(m, kSupB), kSupB, 0, s>>>(g->col.get(), m, key.get(), pos.get());
    k_sup_widen<<<grid_for(n, kSupB), kSupB, 0, s>>>(g->indeg.get(), n, in_off.get());
    PGABB_HIP(hipGetLastError());
    scan_exclusive_i64(in_off.get(), in_off.get(), n, in_off.get() + n, s);
    const bool alt = radix_sort_u32(key.get(), key_alt.get(), pos.get(), pos_alt.get(), m, g->nb, s);
    in_pos = std::move(alt ? pos_alt : pos);
}

uint64_t edge_support(pgabb_graph *g, uint32_t *out, bool out_on_device, DArray<int64_t> *in_off_out,
                      DArray<uint32_t> *in_pos_out) {
    hipStream_t s = g->stream;
    const auto t0 = std::chrono::steady_clock::now();
    const int64_t m = g->m;
    const int32_t n = g->n;
    g->t_kernel_ms = 0;
    g->kernel_launches = 0;
    g->h2d_bytes = 0;
    uint64_t triangles = 0;
    if (m > 0) {
        PGABB_REQUIRE(m < (int64_t{1} << 32), PGABB_EINVAL, "edge support needs m' < 2^32 (m' = %lld)",
                      static_cast<long long>(m));
        DArray<uint32_t> own;
        uint32_t *sup = out;
        if (!out_on_device) {
            own.reset(static_cast<size_t>(m), s);
            sup = own.get();
        }
        // in-edges of every vertex: CSR positions sorted by the higher end
        // (stable, so ascending in the lower end), offsets from the kept
        // in-degrees; and the length of the walk that each starts
        DArray<int32_t> rest(static_cast<size_t>(m), s);
        k_sup_rest<<<std::min(grid_for(n, kSupB / 16), 16384u), kSupB, 0, s>>>(g->row_off.get(), n, rest.get());
        PGABB_HIP(hipGetLastError());
        DArray<int64_t> in_off;
        DArray<uint32_t> in_pos_arr;
        in_edges(g, in_off, in_pos_arr);
        const uint32_t *in_pos = in_pos_arr.get();
        // work units (at most one per owner plus one per kSupUnitEdges in-edges)
        DArray<int64_t> upre(static_cast<size_t>(n) + 1, s);
        const int64_t max_units = static_cast<int64_t>(n) + m / kSupUnitEdges + 1;
        DArray<int2> units(static_cast<size_t>(max_units), s);
        k_sup_unit_counts<<<grid_for(n, kSupB), kSupB, 0, s>>>(g->row_off.get(), in_off.get(), n, upre.get());
        PGABB_HIP(hipGetLastError());
        scan_exclusive_i64(upre.get(), upre.get(), n, upre.get() + n, s);
        k_sup_unit_fill<<<grid_for(n, kSupB), kSupB, 0, s>>>(upre.get(), n, units.get());
        PGABB_HIP(hipGetLastError());

        constexpr int kCtr = kSupQueues * kSupQueueStride + 1;  // work counters, triangles
        DArray<unsigned long long> ctr(kCtr, s);
        PGABB_HIP(hipMemsetAsync(ctr.get(), 0, kCtr * sizeof(unsigned long long), s));
        PGABB_HIP(hipMemsetAsync(sup, 0, sizeof(uint32_t) * static_cast<size_t>(m), s));
        // six workgroups of four waves fit a CU's LDS
        const int64_t want = (max_units + kSupWaves - 1) / kSupWaves;
        const int grid = static_cast<int>(std::max<int64_t>(1, std::min<int64_t>(want, 256 * 6)));
        StreamTimer tm;
        tm.start(s);
        k_edge_support<<<grid, kSupWaves * kWave, 0, s>>>(g->row_off.get(), g->col.get(), in_off.get(), in_pos,
                                                           rest.get(), units.get(), upre.get() + n,
                                                           std::max(0, n - kSupHubs), sup, ctr.get(),
                                                           ctr.get() + kCtr - 1);
        PGABB_HIP(hipGetLastError());
        tm.stop(s);
        Staged<unsigned long long> h(1, s);
        PGABB_HIP(hipMemcpyAsync(h.get(), ctr.get() + kCtr - 1, sizeof(unsigned long long), hipMemcpyDeviceToHost,
                                 s));
        if (!out_on_device)
            PGABB_HIP(hipMemcpyAsync(out, sup, sizeof(uint32_t) * static_cast<size_t>(m), hipMemcpyDeviceToHost,
                                     s));
        PGABB_HIP(hipStreamSynchronize(s));
        if (in_off_out) *in_off_out = std::move(in_off);
        if (in_pos_out) *in_pos_out = std::move(in_pos_arr);
        triangles = h[0];
        g->t_kernel_ms = tm.ms();
        g->kernel_launches = 1;
    }
    g->t_count_ms = std::chrono::duration<double, std::milli>(std::chrono::steady_clock::now() - t0).count();
    return triangles;
}

}  // namespace pgabb
