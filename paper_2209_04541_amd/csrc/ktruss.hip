// k-truss (the peeling algorithm named in PGAbB Section 3.2): the largest
// subgraph in which every edge lies in at least k - 2 triangles of the
// subgraph.  It is unique, so whole rounds reach it as one-edge-at-a-time
// peeling does.
//
// One support pass counts the triangles of every edge; then each round
// takes the live edges with fewer than k - 2 (the round's frontier: found by
// a scan for the first round, and afterwards listed by whoever takes the
// triangle that brings an edge below), and for
// every triangle a frontier edge closes with two edges that are still there,
// the triangle vanishes: each of its edges outside the frontier loses one
// from its count.  A triangle with two or three frontier edges is handled
// by the frontier edge with the smallest CSR position only, so no count
// loses one twice.  Frontier edges are then dead.  The counts of the live
// edges stay the triangle counts of the live graph, so the rounds are those
// of recounting every round, at the cost of the removed edges' triangles.
//
// The triangles of a frontier edge (u, v), ranks u < v, are the common
// neighbours w of u and v in the undirected graph.  A vertex's neighbours
// are its in-edges (lower ranks, ascending) followed by its out-edges
// (higher ranks, ascending), so each list is sorted: the walk takes every
// neighbour of u (the endpoint of lower degree under degree order),
// flattened over the lanes for 64 frontier edges at a time, and finds it in
// v's list by binary search.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <chrono>

#include "common.hpp"
#include "graph.hpp"
#include "wave.hpp"

namespace pgabb {

namespace {

constexpr int kKB = 256;
constexpr int kPeelWaves = 4;
// Groups of a round per wave (peeling of R-MAT scale 18, k = 8, at 4 / 16 / 64:
// 1.97 / 1.61 / 1.82 ms; of a random geometric graph 0.63 / 0.74 / 1.05).
constexpr int kPeelGroups = 8;
constexpr int kTrussRound = 4;  // rounds queued per host round trip
constexpr int kPeelQueues = 16, kPeelStride = 16;  // work counters of a round, 128 bytes apart

enum : uint8_t { kLive = 0, kDying = 1, kDead = 2 };

// Lower end (row) of every oriented edge.
__global__ __launch_bounds__(kKB) void k_kt_rows(const int64_t *__restrict__ row_off, int32_t n,
                                                  int32_t *__restrict__ lo_end) {
    for_row_entries(row_off, n, [&](int32_t a, int64_t e, int64_t) { lo_end[e] = a; });
}

// Lower end of the edge in every in-edge slot.
__global__ __launch_bounds__(kKB) void k_kt_in_nb(const uint32_t *__restrict__ in_pos,
                                                   const int32_t *__restrict__ lo_end, int64_t m,
                                                   int32_t *__restrict__ in_nb) {
    for (int64_t k = blockIdx.x * static_cast<int64_t>(kKB) + threadIdx.x; k < m;
         k += static_cast<int64_t>(gridDim.x) * kKB)
        in_nb[k] = lo_end[in_pos[k]];
}

__global__ __launch_bounds__(kKB) void k_kt_clear(uint8_t *__restrict__ state, int64_t m) {
    for (int64_t e = blockIdx.x * static_cast<int64_t>(kKB) + threadIdx.x; e < m;
         e += static_cast<int64_t>(gridDim.x) * kKB)
        state[e] = kLive;
}

// The first frontier: live edges with fewer than `need` triangles become dying
// and are appended to `front`, with one counter atomic per workgroup and
// kFrontPer * kKB edges (one per wave of 64 edges took 446 us on R-MAT scale
// 18: 59 K atomics on one word), in the order of their positions: a group of the
// peeling launch takes neighbouring entries, which then share their rows.
constexpr int kFrontPer = 16;
__global__ __launch_bounds__(kKB) void k_kt_front(const uint32_t *__restrict__ sup, int64_t m, uint32_t need,
                                                   uint8_t *__restrict__ state, uint32_t *__restrict__ front,
                                                   unsigned long long *__restrict__ nfront) {
    static_assert(kFrontPer * (kKB / kWave) == kWave, "one wave scans the counts");
    __shared__ uint32_t s_pre[kWave];  // by 256 edges and wave: edges taken, then those taken before
    __shared__ unsigned long long s_at;
    const int lane = lane_id(), w = threadIdx.x / kWave;
    const uint64_t below = lane ? (~0ull >> (64 - lane)) : 0ull;
    for (int64_t base = blockIdx.x * static_cast<int64_t>(kKB) * kFrontPer; base < m;
         base += static_cast<int64_t>(gridDim.x) * kKB * kFrontPer) {
        uint64_t taken[kFrontPer];  // by the wave's lanes
#pragma unroll
        for (int q = 0; q < kFrontPer; ++q) {
            const int64_t e = base + q * kKB + threadIdx.x;
            taken[q] = __ballot(e < m && sup[e] < need);
            if (lane == 0) s_pre[q * (kKB / kWave) + w] = static_cast<uint32_t>(__popcll(taken[q]));
        }
        __syncthreads();
        if (w == 0) {
            const uint32_t c = s_pre[lane], incl = wave_inclusive_scan(c);
            s_pre[lane] = incl - c;
            if (lane == kWave - 1 && incl) s_at = atomicAdd(nfront, static_cast<unsigned long long>(incl));
        }
        __syncthreads();
#pragma unroll
        for (int q = 0; q < kFrontPer; ++q) {
            if (!((taken[q] >> lane) & 1ull)) continue;
            const int64_t e = base + q * kKB + threadIdx.x;
            state[e] = kDying;
            front[s_at + s_pre[q * (kKB / kWave) + w] + __popcll(taken[q] & below)] = static_cast<uint32_t>(e);
        }
        __syncthreads();  // before the next turn's counts
    }
}

// After a round: its frontier is dead, the next one's edges are dying.
__global__ __launch_bounds__(kKB) void k_kt_turn(const uint32_t *__restrict__ front,
                                                  const unsigned long long *__restrict__ nfront,
                                                  const uint32_t *__restrict__ after,
                                                  const unsigned long long *__restrict__ nafter,
                                                  uint8_t *__restrict__ state) {
    const int64_t a = static_cast<int64_t>(*nfront), b = static_cast<int64_t>(*nafter);
    for (int64_t i = blockIdx.x * static_cast<int64_t>(kKB) + threadIdx.x; i < a + b;
         i += static_cast<int64_t>(gridDim.x) * kKB) {
        if (i < a) state[front[i]] = kDead;
        else state[after[i - a]] = kDying;
    }
}

// Edges that a wave keeps for the next frontier before it adds them to the
// device's list, of which one batch can bring two a lane.  The list's counter is
// one word: an addition per batch made the longest launches longer (figures at
// k_kt_peel).
constexpr int kDropBuf = 2 * kWave;

struct PeelLds {
    int32_t pre[kWave];   // position of each lane's list in the flattened walk
    uint32_t e[kWave];    // the frontier edge (u, v)
    int32_t v[kWave];
    int32_t nin_u[kWave];   // u's in-edges
    uint32_t iu0[kWave];     // u's first in-edge slot (m' < 2^32)
    uint32_t ou0[kWave];     // u's first out-edge position
    uint32_t iv0[kWave], iv1[kWave];  // v's in-edge slots
    uint32_t ov0[kWave], ov1[kWave];  // v's out-edge positions
    int32_t own[kWave];     // list starts of the current batch
    int32_t left[kWave];    // triangles of the frontier edge still to be met
    int32_t from[kWave];    // first of u's neighbours in the walk
    uint32_t drop[kDropBuf];  // edges for the next frontier
};

// First index in [lo, hi) of the sorted x whose value is at least w.
template <class I>
__device__ __forceinline__ I lower_at(gptr<int32_t> x, I lo, I hi, int32_t w) {
    while (lo < hi) {
        const I mid = lo + ((hi - lo) >> 1);
        if (x[mid] < w) lo = mid + 1;
        else hi = mid;
    }
    return lo;
}

// One round's triangle updates: groups of up to 64 frontier edges, one per
// lane.  A group is a chain of dependent loads (each batch of 64 neighbours
// ends in binary searches), so small frontiers are cut into groups of few
// edges, down to a part of one edge's neighbours.  Groups of fewer than
// kTakenEdges edges are dealt to the waves in turn: taken from a counter, every
// wave's last (empty) take alone made a round of any size last 100 us, one word
// serving some 80 M atomics a second.  Larger rounds last milliseconds, and the
// longest of a wave's turns held them up; there the waves take their groups
// (UnitTaker).  An edge's count says how many of its triangles are left to be
// met, so an edge in none walks nothing and the others' neighbours after the
// last triangle cost no load.  An edge that a vanished triangle brings below
// `need` joins `after`, the next round's frontier, by the one decrement that
// does; a wave gathers those in LDS.  The launch keeps eight workgroups on a CU
// (the grid's size): positions are 32 bits wide for that.
//
// Longest launch on R-MAT scale 20, k = 8 / 20 / 64, ms: 4.9 / 11.6 / 24.6 with
// groups from one counter and a scan for the next frontier (all rounds 8.5 /
// 20.3 / 41.8); dealt in turn, an addition per batch 5.8 / 13.9 / 28.2 (6.8 /
// 16.7 / 36.0); with the buffer 5.2 / 13.6 / 27.9 (6.0 / 15.6 / 34.0), and seven
// workgroups on a CU 6.3 / 18.5 / 41.6; with large rounds taken 4.5 / 12.0 /
// 26.0 (5.5 / 14.9 / 33.8).  Large rounds taken without the buffer: 5.2 / 11.0 /
// 24.3 (6.2 / 13.7 / 32.0), but slower on clustered graphs (a random geometric
// graph of 200,003 vertices, k = 8, all kernels 1.35 ms, 1.24 with it).
constexpr int64_t kTakenEdges = 8;

__global__ __launch_bounds__(kPeelWaves *kWave) void k_kt_peel(const uint32_t *__restrict__ front_,
                                                                const unsigned long long *__restrict__ nfront_,
                                                                const int64_t *__restrict__ row_off_,
                                                                const int32_t *__restrict__ col_,
                                                                const int32_t *__restrict__ lo_end_,
                                                                const int64_t *__restrict__ in_off_,
                                                                const uint32_t *__restrict__ in_pos_,
                                                                const int32_t *__restrict__ in_nb_,
                                                                const uint8_t *__restrict__ state_,
                                                                uint32_t *__restrict__ sup, uint32_t need,
                                                                uint32_t *__restrict__ after,
                                                                unsigned long long *__restrict__ nafter,
                                                                unsigned long long *__restrict__ next) {
    __shared__ PeelLds s_lds[kPeelWaves];
    PeelLds &L = s_lds[threadIdx.x / kWave];
    const int lane = lane_id();
    const gptr<uint32_t> front = as_global(front_);
    const gptr<int64_t> ro = as_global(row_off_);
    const gptr<int32_t> col = as_global(col_), lo_end = as_global(lo_end_), in_nb = as_global(in_nb_);
    const gptr<int64_t> io = as_global(in_off_);
    const gptr<uint32_t> ip = as_global(in_pos_);
    const gptr<uint8_t> state = as_global(state_);
    const int64_t cnt = static_cast<int64_t>(*as_global(nfront_));
    if (cnt == 0) return;
    L.own[lane] = 0;
    wave_lds_sync();
    // edges per group, and groups per edge: about kPeelGroups groups per wave
    // of the launch
    const int64_t want = static_cast<int64_t>(gridDim.x) * kPeelWaves * kPeelGroups;
    const int64_t per = max(min(cnt / want, static_cast<int64_t>(kWave)), static_cast<int64_t>(1));
    const int32_t parts = static_cast<int32_t>(max(min(want / cnt, static_cast<int64_t>(kWave)), static_cast<int64_t>(1)));
    const uint64_t below = lane ? (~0ull >> (64 - lane)) : 0ull;
    const int64_t waves = static_cast<int64_t>(gridDim.x) * kPeelWaves;
    int ndrop = 0;  // edges in L.drop
    auto append = [&](int num) {
        unsigned long long at = 0;
        if (lane == 0) at = atomicAdd(nafter, static_cast<unsigned long long>(num));
        at = shfl_t(at, 0);
        for (int i = lane; i < num; i += kWave) after[at + i] = L.drop[i];
        wave_lds_sync();  // before the buffer is filled again
    };
    const int64_t wave = blockIdx.x * static_cast<int64_t>(kPeelWaves) + threadIdx.x / kWave;
    const int64_t groups = (cnt + per - 1) / per * parts;
    auto peel_group = [&](int64_t g0) {
        const int64_t first = g0 / parts * per;
        const int32_t part = static_cast<int32_t>(g0 % parts);
        const int64_t idx = first + lane;
        int32_t len = 0;
        if (lane < per && idx < cnt) {
            const uint32_t e = front[idx];
            const int32_t u = lo_end[e], v = col[e];
            const int64_t iu0 = io[u], iu1 = io[u + 1], ou0 = ro[u], ou1 = ro[u + 1];
            // the edge's count: its triangles with edges still present
            const int32_t left = static_cast<int32_t>(sup[e]);
            L.left[lane] = left;
            const int32_t all = left ? static_cast<int32_t>((iu1 - iu0) + (ou1 - ou0)) : 0;
            // this part's neighbours [from, from + len)
            const int32_t share = (all + parts - 1) / parts, from = min(share * part, all);
            len = min(share, all - from);
            L.from[lane] = from;
            L.e[lane] = e;
            L.v[lane] = v;
            L.nin_u[lane] = static_cast<int32_t>(iu1 - iu0);
            L.iu0[lane] = static_cast<uint32_t>(iu0);
            L.ou0[lane] = static_cast<uint32_t>(ou0);
            L.iv0[lane] = static_cast<uint32_t>(io[v]);
            L.iv1[lane] = static_cast<uint32_t>(io[v + 1]);
            L.ov0[lane] = static_cast<uint32_t>(ro[v]);
            L.ov1[lane] = static_cast<uint32_t>(ro[v + 1]);
        }
        const int32_t incl = wave_inclusive_scan(len);
        const int32_t pre = incl - len;
        const int32_t total = __builtin_amdgcn_readlane(incl, kWave - 1);
        L.pre[lane] = pre;
        wave_lds_sync();
        uint32_t carry = 0;
        for (int32_t base = 0; base < total; base += kWave) {
            // the lane whose list holds element base + lane: list starts
            // scattered into LDS, then a running maximum over the lanes
            const int32_t p = pre - base;
            if (len > 0 && p >= 0 && p < kWave) L.own[p] = lane + 1;
            wave_lds_sync();
            const uint32_t o = static_cast<uint32_t>(L.own[lane]);
            L.own[lane] = 0;
            wave_lds_sync();
            const uint32_t sl1 = max(wave_max_scan_dpp(o), carry);
            carry = __builtin_amdgcn_readlane(sl1, kWave - 1);
            const int32_t el = base + lane;
            // the lane's neighbour w of u: one off the counts of (u, w) and (v,
            // w) if all three edges are there; f, gq: those that fell below need
            uint32_t drop_f = UINT32_MAX, drop_g = UINT32_MAX;
            auto visit = [&]() {
                const int sl = static_cast<int>(sl1) - 1;
                if (L.left[sl] <= 0) return;  // all met
                const int32_t t = L.from[sl] + (el - L.pre[sl]);  // neighbour t of u
                const uint32_t e = L.e[sl];
                const int32_t v = L.v[sl];
                int32_t w;
                uint32_t f;  // edge (u, w)
                if (t < L.nin_u[sl]) {
                    const int64_t k = static_cast<int64_t>(L.iu0[sl]) + t;
                    w = in_nb[k];
                    f = ip[k];
                } else {
                    const int64_t q = static_cast<int64_t>(L.ou0[sl]) + (t - L.nin_u[sl]);
                    w = col[q];
                    f = static_cast<uint32_t>(q);
                }
                if (w == v) return;
                const uint8_t sf = state[f];
                if (sf == kDead) return;
                uint32_t gq;  // edge (v, w), if any
                if (w < v) {
                    const int64_t k0 = L.iv0[sl], k1 = L.iv1[sl];
                    const int64_t k = lower_at<int64_t>(in_nb, k0, k1, w);
                    if (k >= k1 || in_nb[k] != w) return;
                    gq = ip[k];
                } else {
                    const int64_t q0 = L.ov0[sl], q1 = L.ov1[sl];
                    const int64_t q = lower_at<int64_t>(col, q0, q1, w);
                    if (q >= q1 || col[q] != w) return;
                    gq = static_cast<uint32_t>(q);
                }
                const uint8_t sg = state[gq];
                if (sg == kDead) return;
                atomicSub(&L.left[sl], 1);
                // the triangle vanishes; only its frontier edge of smallest
                // position updates the others
                if ((sf == kDying && f < e) || (sg == kDying && gq < e)) return;
                if (sf == kLive && atomicSub(&sup[f], 1u) == need) drop_f = f;
                if (sg == kLive && atomicSub(&sup[gq], 1u) == need) drop_g = gq;
            };
            if (el < total) visit();
            const uint64_t mf = __ballot(drop_f != UINT32_MAX), mg = __ballot(drop_g != UINT32_MAX);
            if ((mf | mg) == 0) continue;
            const int nf = __popcll(mf), ng = __popcll(mg);
            if (ndrop + nf + ng > kDropBuf) {
                append(ndrop);
                ndrop = 0;
            }
            if (drop_f != UINT32_MAX) L.drop[ndrop + __popcll(mf & below)] = drop_f;
            if (drop_g != UINT32_MAX) L.drop[ndrop + nf + __popcll(mg & below)] = drop_g;
            ndrop += nf + ng;
            wave_lds_sync();
        }
        wave_lds_sync();  // before the next group overwrites the lane records
    };
    if (per >= kTakenEdges) {
        UnitTaker<kPeelQueues, kPeelStride> taker(next, groups, waves, wave);
        for (int64_t g0; (g0 = taker.take(lane)) >= 0;) peel_group(g0);
    } else {
        for (int64_t g0 = wave; g0 < groups; g0 += waves) peel_group(g0);
    }
    if (ndrop) append(ndrop);
}

// Clears p[0, n), p[0] to *first if given (by one wave: all its lanes have read
// *first, which lies in there, before one of them writes).
__global__ void k_kt_zero(unsigned long long *p, const unsigned long long *first, int32_t n) {
    const unsigned long long f = first ? *first : 0ull;
    for (int32_t i = threadIdx.x; i < n; i += kWave) p[i] = i == 0 ? f : 0ull;
}

__global__ __launch_bounds__(kKB) void k_kt_keep(const uint8_t *__restrict__ state, int64_t m,
                                                  uint8_t *__restrict__ keep) {
    for (int64_t e = blockIdx.x * static_cast<int64_t>(kKB) + threadIdx.x; e < m;
         e += static_cast<int64_t>(gridDim.x) * kKB)
        keep[e] = state[e] == kLive ? 1 : 0;
}

}  // namespace

int64_t ktruss(pgabb_graph *g, int32_t k, uint8_t *keep, bool on_device, int32_t *rounds_out) {
    hipStream_t s = g->stream;
    const auto t0 = std::chrono::steady_clock::now();
    const int32_t n = g->n;
    const int64_t m = g->m;
    int32_t rounds = 0;
    int64_t live = m;
    double kernel_ms = 0;
    if (m > 0) {
        PGABB_REQUIRE(m < (int64_t{1} << 32), PGABB_EINVAL, "k-truss needs m' < 2^32 (m' = %lld)",
                      static_cast<long long>(m));
        const uint32_t need = k > 2 ? static_cast<uint32_t>(k - 2) : 0u;
        DArray<uint8_t> state(static_cast<size_t>(m), s);
        k_kt_clear<<<grid_for(m, kKB), kKB, 0, s>>>(state.get(), m);
        PGABB_HIP(hipGetLastError());
        if (need > 0) {  // k <= 2: every edge stays
            DArray<uint32_t> sup(static_cast<size_t>(m), s);
            DArray<int64_t> in_off;
            DArray<uint32_t> in_pos;
            edge_support(g, sup.get(), true, &in_off, &in_pos);
            kernel_ms += g->t_kernel_ms;
            DArray<int32_t> lo_end(static_cast<size_t>(m), s), in_nb(static_cast<size_t>(m), s);
            k_kt_rows<<<std::min(grid_for(n, kKB / 16), 16384u), kKB, 0, s>>>(g->row_off.get(), n, lo_end.get());
            k_kt_in_nb<<<grid_for(m, kKB), kKB, 0, s>>>(in_pos.get(), lo_end.get(), m, in_nb.get());
            PGABB_HIP(hipGetLastError());
            DArray<uint32_t> front_a(static_cast<size_t>(m), s), front_b(static_cast<size_t>(m), s);
            // kTrussRound rounds are queued per host round trip (a round after
            // an empty frontier does nothing): frontier sizes of the rounds
            // and of the one after, then the rounds' work counters
            constexpr int kCtr = kTrussRound + 1 + kTrussRound * kPeelQueues * kPeelStride;
            DArray<unsigned long long> ctr(kCtr, s);
            Staged<unsigned long long> h_front(kTrussRound + 1, s);
            uint32_t *front = front_a.get(), *after = front_b.get();
            k_kt_zero<<<1, kWave, 0, s>>>(ctr.get(), nullptr, kCtr);
            k_kt_front<<<std::min(grid_for(m, kKB * kFrontPer), 256u * 8u), kKB, 0, s>>>(sup.get(), m, need, state.get(),
                                                                                       front, ctr.get());
            PGABB_HIP(hipGetLastError());
            const unsigned grid = std::min(grid_for(m, kPeelWaves), 256u * 8u);
            StreamTimer tm;
            for (bool more = true; more;) {
                tm.start(s);
                for (int q = 0; q < kTrussRound; ++q) {
                    k_kt_peel<<<grid, kPeelWaves * kWave, 0, s>>>(front, ctr.get() + q, g->row_off.get(), g->col.get(),
                                                                   lo_end.get(), in_off.get(), in_pos.get(),
                                                                   in_nb.get(), state.get(), sup.get(), need, after,
                                                                   ctr.get() + q + 1,
                                                                   ctr.get() + kTrussRound + 1 + q * kPeelQueues * kPeelStride);
                    k_kt_turn<<<std::min(grid_for(m, kKB), 1024u), kKB, 0, s>>>(front, ctr.get() + q, after,
                                                                             ctr.get() + q + 1, state.get());
                    std::swap(front, after);
                }
                tm.stop(s);
                PGABB_HIP(hipGetLastError());
                PGABB_HIP(hipMemcpyAsync(h_front.get(), ctr.get(), h_front.bytes(), hipMemcpyDeviceToHost, s));
                // the next rounds start from the last frontier
                k_kt_zero<<<1, kWave, 0, s>>>(ctr.get(), ctr.get() + kTrussRound, kCtr);
                PGABB_HIP(hipStreamSynchronize(s));
                kernel_ms += tm.ms();
                more = h_front[kTrussRound] != 0;
                for (int q = 0; q < kTrussRound; ++q) {
                    rounds += h_front[q] ? 1 : 0;
                    live -= static_cast<int64_t>(h_front[q]);
                }
            }
        }
        if (keep) {
            DArray<uint8_t> own;
            uint8_t *dst = keep;
            if (!on_device) {
                own.reset(static_cast<size_t>(m), s);
                dst = own.get();
            }
            k_kt_keep<<<grid_for(m, kKB), kKB, 0, s>>>(state.get(), m, dst);
            PGABB_HIP(hipGetLastError());
            if (!on_device) PGABB_HIP(hipMemcpyAsync(keep, dst, static_cast<size_t>(m), hipMemcpyDeviceToHost, s));
            PGABB_HIP(hipStreamSynchronize(s));
        }
    }
    g->t_kernel_ms = kernel_ms;
    g->kernel_launches = rounds;
    g->t_count_ms = std::chrono::duration<double, std::milli>(std::chrono::steady_clock::now() - t0).count();
    if (rounds_out) *rounds_out = rounds;
    return live;
}

}  // namespace pgabb
