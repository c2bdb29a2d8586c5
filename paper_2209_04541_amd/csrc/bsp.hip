// Single-block bulk-synchronous computations (PGAbB Section 3.2: every
// iteration visits every edge, and block-lists of one block suffice).  Two of
// the paper's examples, the first over the rows of the oriented graph, the
// second over the blocks the triangle count uses:
//
//   * connected components by Shiloach-Vishkin (Section 3.4): hooking
//     iterations put the trees of an edge's ends under one root, linking
//     iterations point every vertex at its tree's root by pointer jumping.
//     The smaller root goes under the larger: ranks ascend with the degree,
//     so trees gather at the hubs.  The first hooking pass puts every vertex
//     under its highest neighbour (the last entry of its row), the second
//     takes each row's last entry but one, which leaves few trees, and the
//     third visits every edge.  A hook that another edge got ahead of is
//     tried again with the roots found then, so the third pass leaves no
//     edge between two trees and no pass is needed to see that (R-MAT scale
//     20 over 8 x 8 blocks: 3.6 -> 0.66 ms a call; five passes over the
//     blocks' items with a host round trip each took 2.8 ms of kernels, these
//     0.35 ms, most of it the gathers of the third pass);
//   * PageRank (Section 5.2, an SpMV-like iteration with damping d,
//     tolerance and iteration limit), pulled through the blocks with atomic
//     additions, as the paper does on its two-dimensional layout.  On R-MAT
//     scale 20 over 8 x 8 blocks an iteration's pull takes 225 us (271 with
//     one entry per lane), for 31 M gathers of shares and one addition per
//     item in device memory; four iterations are queued per host round trip
//     (eight of them 3.07 -> 2.55 ms a call).
//
// PageRank's work items are the blocks' own (x, b, e) records: a run of at
// most kSplitV entries of one row or, through the stored transpose, of one
// column.  All items of all blocks form one list per launch; a wave takes 64
// of them, a lane finding its item's block by a binary search of the item
// prefix, and reads their entries in segments of kSeg, one per lane and load
// (walk_items; see tc_device.hpp).  The components' passes read the rows of
// the oriented graph.
// Vertices are ranks (the ids of the oriented graph); results come back by
// input id through the graph's rank array.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <chrono>
#include <cmath>
#include <cstring>
#include <vector>

#include "common.hpp"
#include "graph.hpp"
#include "tc_device.hpp"
#include "wave.hpp"

namespace pgabb {

namespace {

constexpr int kBB = 256;
constexpr int kBspQueues = 8;
constexpr int kBspStride = 32;  // queue counters 256 bytes apart
constexpr int kBspQueueWords = kBspQueues * kBspStride;
// Rows a wave hooks at a time (R-MAT scale 20, all kernels of a call: 8 / 16
// / 32 / 64 rows 506 / 387 / 346 / 372 us).
constexpr int kHookRows = 32;

// One run of items: the row items of a block (entries in `idx` = col, item
// ids in stripe i, entries in stripe j) or its column items (idx = crow,
// item ids in stripe j, entries in stripe i).
struct BspSeg {
    const int32_t *items;
    const int32_t *idx;
    int32_t base_x;  // rank of local id 0 on the item side
    int32_t base_y;  // rank of local id 0 on the entry side
};

// Last segment s with pre[s] <= q (pre[0] = 0 <= q < pre[nseg]).
__device__ __forceinline__ int32_t find_seg(const int64_t *__restrict__ pre, int32_t nseg, int64_t q) {
    int32_t lo = 0, hi = nseg - 1;
    while (lo < hi) {
        const int32_t mid = (lo + hi + 1) >> 1;
        if (pre[mid] <= q) lo = mid;
        else hi = mid - 1;
    }
    return lo;
}

// Reads the entries of one list per lane -- len of them at src_ptr, vertices
// by + entry -- as one flattened run of segments: own[] is 64 words of the
// wave's LDS, zero on entry and left zero.  Calls seg(n, src, y) for every
// segment on the lane that holds it: n entries (some lanes may hold none) of
// the list of lane src, the vertices y[0 .. n).  The segment of a list's last
// entries reads up to kSeg - 1 words past them: the arrays that lists lie in
// are allocated kSeg words longer.
template <class SegFn>
__device__ __forceinline__ void walk_lists(const int32_t *src_ptr, int32_t len, int32_t by, int32_t *own, int lane,
                                           SegFn seg) {
    const int32_t ns = (len + kSeg - 1) / kSeg;
    const int32_t incl = wave_inclusive_scan(ns);
    const int32_t pre_l = incl - ns;
    const int32_t total = __builtin_amdgcn_readlane(incl, kWave - 1);
    // segment t of the run starts at rel + kSeg t words of its item's lane
    const uint64_t rel = reinterpret_cast<uint64_t>(src_ptr) -
                         static_cast<uint64_t>(pre_l) * (kSeg * sizeof(int32_t));
    const int32_t rel_lo = static_cast<int32_t>(static_cast<uint32_t>(rel));
    const int32_t rel_hi = static_cast<int32_t>(static_cast<uint32_t>(rel >> 32));
    const int32_t last = len + kSeg * pre_l;  // entries of the item before position kSeg t: kSeg t - kSeg pre_l
    uint32_t carry = 0;
    for (int32_t base = 0; base < total; base += kWave) {
        const int32_t p = pre_l - base;
        if (ns > 0 && p >= 0 && p < kWave) own[p] = lane + 1;
        wave_lds_sync();
        const uint32_t o = static_cast<uint32_t>(own[lane]);
        own[lane] = 0;
        wave_lds_sync();
        const uint32_t sl1 = max(wave_max_scan_dpp(o), carry);
        carry = __builtin_amdgcn_readlane(sl1, kWave - 1);
        const int sl = static_cast<int>(sl1) - 1;
        const int32_t t = base + lane;
        const uint64_t r = (static_cast<uint64_t>(static_cast<uint32_t>(__shfl(rel_hi, sl))) << 32) |
                           static_cast<uint32_t>(__shfl(rel_lo, sl));
        const int32_t left = __shfl(last, sl) - kSeg * t;  // (every lane shuffles)
        const int32_t n = t < total ? min(left, kSeg) : 0;
        const int32_t yb = __shfl(by, sl);
        int32_t y[kSeg] = {0, 0, 0, 0};
        if (n > 0) {
            const seg_t v = *reinterpret_cast<const __attribute__((address_space(1))) seg_t *>(
                as_global(reinterpret_cast<const int32_t *>(r)) + static_cast<int64_t>(kSeg) * t);
#pragma unroll
            for (int k = 0; k < kSeg; ++k) y[k] = yb + v[k];
        }
        seg(n, sl, y);
    }
}

// walk_lists over the items [q0, q1), at most 64, after item(x) on every lane
// (x: its item's vertex, or -1).
template <class Item, class SegFn>
__device__ __forceinline__ void walk_items(const BspSeg *__restrict__ segs, const int64_t *__restrict__ pre,
                                           int32_t nseg, int64_t q0, int64_t q1, int32_t *own, int lane, Item item,
                                           SegFn seg) {
    const int64_t q = q0 + lane;
    int32_t x = -1, len = 0, by = 0;
    const int32_t *src_ptr = nullptr;
    if (q < q1) {
        const int32_t s = find_seg(pre, nseg, q);
        const BspSeg sg = segs[s];
        const gptr<int32_t> it = as_global(sg.items) + kItemWords * (q - pre[s]);
        x = sg.base_x + it[0];
        const int32_t b = it[1], e = it[2];
        len = e - b;
        src_ptr = sg.idx + b;
        by = sg.base_y;
    }
    item(x);
    walk_lists(src_ptr, len, by, own, lane, seg);
}

// The first hooking pass: every vertex under its highest neighbour, the last
// entry of its row (itself without one).
__global__ __launch_bounds__(kBB) void k_sv_first(const int64_t *__restrict__ row_off, const int32_t *__restrict__ col,
                                                  int32_t n, int32_t *__restrict__ C) {
    for (int64_t r = blockIdx.x * int64_t(kBB) + threadIdx.x; r < n; r += int64_t(gridDim.x) * kBB) {
        const int64_t e0 = row_off[r], e1 = row_off[r + 1];
        C[r] = e1 > e0 ? col[e1 - 1] : static_cast<int32_t>(r);
    }
}

// Puts the trees of cu and cv (ancestors of an edge's ends) under one root:
// the smaller of two different ancestors is hooked under the larger if it is
// a root; if another hook got there first, both ancestors are read again.
// Parents only ever increase, so the pointers form a forest whatever order
// the hooks land in, and every retry starts from higher ancestors.
__device__ __forceinline__ void sv_hook(int32_t *__restrict__ C, int32_t cu, int32_t cv) {
    while (cu != cv) {
        const int32_t r1 = min(cu, cv), r2 = max(cu, cv);
        const int32_t up = __atomic_load_n(&C[r1], __ATOMIC_RELAXED);
        if (up == r2) return;
        if (up == r1) {
            const int32_t was = atomicCAS(&C[r1], r1, r2);
            if (was == r1 || was == r2) return;
        }
        cu = __atomic_load_n(&C[__atomic_load_n(&C[r1], __ATOMIC_RELAXED)], __ATOMIC_RELAXED);
        cv = __atomic_load_n(&C[r2], __ATOMIC_RELAXED);
    }
}

// The second hooking pass: every row's last entry but one.
__global__ __launch_bounds__(kBB) void k_sv_second(const int64_t *__restrict__ row_off,
                                                   const int32_t *__restrict__ col, int32_t n,
                                                   int32_t *__restrict__ C) {
    for (int64_t r = blockIdx.x * int64_t(kBB) + threadIdx.x; r < n; r += int64_t(gridDim.x) * kBB) {
        const int64_t e0 = row_off[r], e1 = row_off[r + 1];
        if (e1 - e0 >= 2)
            sv_hook(C, __atomic_load_n(&C[r], __ATOMIC_RELAXED), __atomic_load_n(&C[col[e1 - 2]], __ATOMIC_RELAXED));
    }
}

// Hooking over every edge: a wave takes kHookRows consecutive rows of the
// oriented graph, highest ranks (the longest rows) first, from eight work
// counters.
// Rows, not the blocks' items: at 8 x 8 blocks an item holds about four
// entries, and finding 64 items' blocks and records cost more than their
// entries (R-MAT scale 20: 330 us a pass over the items).
__global__ __launch_bounds__(kBB) void k_sv_hook_edges(const int64_t *__restrict__ row_off,
                                                       const int32_t *__restrict__ col, int32_t n,
                                                       int32_t *__restrict__ C,
                                                       unsigned long long *__restrict__ next) {
    __shared__ int32_t s_own[kBB];
    const int lane = lane_id();
    int32_t *own = s_own + (threadIdx.x - lane);
    own[lane] = 0;
    wave_lds_sync();
    const gptr<int64_t> ro = as_global(row_off);
    const int64_t groups = (static_cast<int64_t>(n) + kHookRows - 1) / kHookRows;
    UnitTaker<kBspQueues, kBspStride> taker(next, groups, static_cast<int64_t>(gridDim.x) * (kBB / kWave),
                                            static_cast<int64_t>(blockIdx.x) * (kBB / kWave) + threadIdx.x / kWave);
    for (int64_t g; (g = taker.take(lane)) >= 0;) {
        const int64_t x = lane < kHookRows ? n - 1 - g * kHookRows - lane : -1;
        const int64_t e0 = x >= 0 ? ro[x] : 0, e1 = x >= 0 ? ro[x + 1] : 0;
        const int32_t cu = x >= 0 ? __atomic_load_n(&C[x], __ATOMIC_RELAXED) : 0;
        walk_lists(col + e0, static_cast<int32_t>(e1 - e0), 0, own, lane,
                   [&](int32_t m, int src, const int32_t (&y)[kSeg]) {
                       const int32_t c0 = __shfl(cu, src);
                       int32_t cv[kSeg];
#pragma unroll
                       for (int k = 0; k < kSeg; ++k)
                           cv[k] = k < m ? __atomic_load_n(&C[y[k]], __ATOMIC_RELAXED) : c0;
#pragma unroll
                       for (int k = 0; k < kSeg; ++k) sv_hook(C, c0, cv[k]);
                   });
    }
}

// Linking: every vertex points to the root of its tree (pointer jumping to
// the end; no hook runs meanwhile, so the roots stay fixed).  The ancestors
// reached on the way are stored, which shortens the chains that pass through
// x.
__global__ __launch_bounds__(kBB) void k_sv_link(int32_t *__restrict__ C, int32_t n) {
    for (int64_t x = blockIdx.x * int64_t(kBB) + threadIdx.x; x < n; x += int64_t(gridDim.x) * kBB) {
        int32_t y = __atomic_load_n(&C[x], __ATOMIC_RELAXED);
        for (;;) {
            const int32_t z = __atomic_load_n(&C[y], __ATOMIC_RELAXED);
            if (z == y) break;
            y = z;
            __atomic_store_n(&C[x], y, __ATOMIC_RELAXED);
        }
    }
}

// Smallest input id of each tree: minid[root] over the input ids v whose
// rank lies in the tree.  Also counts the roots (ranks x with C(x) = x; the
// loop index runs over input ids and ranks alike, both 0 .. n - 1).
__global__ __launch_bounds__(kBB) void k_sv_minid(const int32_t *__restrict__ C, const int32_t *__restrict__ rank,
                                                  int32_t n, int32_t *__restrict__ minid,
                                                  unsigned long long *__restrict__ roots) {
    uint32_t c = 0;
    const int lane = lane_id();
    const int64_t stride = int64_t(gridDim.x) * kBB;
    for (int64_t base = blockIdx.x * int64_t(kBB) + (threadIdx.x & ~(kWave - 1)); base < n; base += stride) {
        const int64_t v = base + lane;
        const bool ok = v < n;
        const int32_t root = ok ? C[rank[v]] : -1;
        // one large component holds most vertices: of the lanes whose root is
        // the first lane's, the first holds the smallest id and alone sends
        // it (most ids are above a minimum already there, which one load
        // shows)
        const int32_t r0 = __builtin_amdgcn_readfirstlane(root);
        if (ok && (lane == 0 || root != r0) && v < __atomic_load_n(&minid[root], __ATOMIC_RELAXED))
            atomicMin(&minid[root], static_cast<int32_t>(v));
        c += ok && C[v] == v ? 1u : 0u;
    }
    const unsigned long long sum = group_sum(static_cast<unsigned long long>(c));
    if (threadIdx.x == 0 && sum) atomicAdd(roots, sum);  // one atomic per workgroup, at most 512
}

__global__ void k_zero_words(unsigned long long *__restrict__ p, int32_t n) {
    for (int32_t q = threadIdx.x; q < n; q += blockDim.x) p[q] = 0ull;
}

// Clears n 8-byte words with a fill kernel (no memset node: a caller may
// capture the stream).
void zero_words(unsigned long long *p, int32_t n, hipStream_t s) {
    k_zero_words<<<1, 64, 0, s>>>(p, n);
}

__global__ __launch_bounds__(kBB) void k_fill_i32(int32_t *__restrict__ p, int32_t v, int64_t n) {
    for (int64_t q = blockIdx.x * int64_t(kBB) + threadIdx.x; q < n; q += int64_t(gridDim.x) * kBB) p[q] = v;
}

__global__ __launch_bounds__(kBB) void k_sv_label(const int32_t *__restrict__ C, const int32_t *__restrict__ rank,
                                                  const int32_t *__restrict__ minid, int32_t n,
                                                  int32_t *__restrict__ label) {
    for (int64_t v = blockIdx.x * int64_t(kBB) + threadIdx.x; v < n; v += int64_t(gridDim.x) * kBB)
        label[v] = minid[C[rank[v]]];
}

// PageRank, one iteration in two launches: the pull of the shares
// contrib(x) = r(x) / deg(x) (zero for isolated vertices) over every block's
// rows and columns into acc, and the update r'(x) = (1 - d) / n + d * acc(x)
// with the sum of |r' - r|, the next shares and the clearing of acc.  `prev`
// is the change of the iteration before: below tol, the iterations have
// stopped and the launch does nothing (iterations are queued several at a
// time).
//
// (PageRank walks the items in block order, grid-stride: dealt to per-XCD
// queues by the stripe they gather from, one item per lane, an iteration on
// R-MAT scale 20 took 0.81 ms against 0.72 ms.)
// The pull: each lane adds up its segment's shares and adds them to its
// item's sum in LDS, and every item adds its sum to acc[x] once.
__global__ __launch_bounds__(kBB) void k_pr_pull(const BspSeg *__restrict__ segs, const int64_t *__restrict__ pre,
                                                 int32_t nseg, const double *__restrict__ contrib_,
                                                 double *__restrict__ acc, const double *__restrict__ prev,
                                                 double tol) {
    if (prev && *prev < tol) return;
    __shared__ double s_sum[kBB];
    __shared__ int32_t s_own[kBB];
    const int lane = lane_id();
    double *sum = s_sum + (threadIdx.x - lane);
    int32_t *own = s_own + (threadIdx.x - lane);
    const gptr<double> contrib = as_global(contrib_);
    own[lane] = 0;
    wave_lds_sync();
    const int64_t total = pre[nseg];
    const int64_t stride = static_cast<int64_t>(gridDim.x) * kBB;
    for (int64_t q0 = blockIdx.x * int64_t(kBB) + (threadIdx.x - lane); q0 < total; q0 += stride) {
        int32_t x = -1;
        walk_items(
            segs, pre, nseg, q0, min(q0 + kWave, total), own, lane,
            [&](int32_t v) {
                x = v;
                sum[lane] = 0.0;
            },
            [&](int32_t n, int src, const int32_t (&y)[kSeg]) {
                double c[kSeg];
#pragma unroll
                for (int k = 0; k < kSeg; ++k) c[k] = k < n ? contrib[y[k]] : 0.0;
                if (n > 0) unsafeAtomicAdd(&sum[src], (c[0] + c[1]) + (c[2] + c[3]));
            });
        wave_lds_sync();
        if (x >= 0) unsafeAtomicAdd(&acc[x], sum[lane]);
        wave_lds_sync();  // before the next items reset the sums
    }
}

__global__ __launch_bounds__(kBB) void k_pr_update(double *__restrict__ r, double *__restrict__ acc,
                                                   const int32_t *__restrict__ outdeg,
                                                   const int32_t *__restrict__ indeg, int32_t n, double teleport,
                                                   double d, double *__restrict__ contrib, double *__restrict__ err,
                                                   const double *__restrict__ prev, double tol) {
    if (prev && *prev < tol) return;
    double e = 0.0;
    for (int64_t x = blockIdx.x * int64_t(kBB) + threadIdx.x; x < n; x += int64_t(gridDim.x) * kBB) {
        const double nx = teleport + d * acc[x];
        e += fabs(nx - r[x]);
        r[x] = nx;
        const int32_t deg = outdeg[x] + indeg[x];
        contrib[x] = deg ? nx / static_cast<double>(deg) : 0.0;
        acc[x] = 0.0;
    }
#pragma unroll
    for (int m = 1; m < kWave; m <<= 1) e += __shfl_xor(e, m);
    // one atomic per workgroup: the launch keeps its grid small, so the
    // additions to the one address stay few
    __shared__ double s_part[kBB / kWave];
    if (lane_id() == 0) s_part[threadIdx.x / kWave] = e;
    __syncthreads();
    if (threadIdx.x == 0) {
        double t = 0.0;
        for (int w = 0; w < kBB / kWave; ++w) t += s_part[w];
        if (t != 0.0) unsafeAtomicAdd(err, t);
    }
}

__global__ __launch_bounds__(kBB) void k_pr_init(double *__restrict__ r, double *__restrict__ acc,
                                                 const int32_t *__restrict__ outdeg,
                                                 const int32_t *__restrict__ indeg, int32_t n, double v,
                                                 double *__restrict__ contrib) {
    for (int64_t x = blockIdx.x * int64_t(kBB) + threadIdx.x; x < n; x += int64_t(gridDim.x) * kBB) {
        r[x] = v;
        const int32_t deg = outdeg[x] + indeg[x];
        contrib[x] = deg ? v / static_cast<double>(deg) : 0.0;
        acc[x] = 0.0;
    }
}

__global__ __launch_bounds__(kBB) void k_pr_by_id(const double *__restrict__ r, const int32_t *__restrict__ rank,
                                                  int32_t n, double *__restrict__ out) {
    for (int64_t v = blockIdx.x * int64_t(kBB) + threadIdx.x; v < n; v += int64_t(gridDim.x) * kBB)
        out[v] = r[rank[v]];
}

// Iterations of PageRank queued between two reads of their changes (a round
// trip costs about five launches).
constexpr int kPrRound = 4;

// Grid of a grid-stride launch over `work` elements: enough workgroups to
// fill every CU a few times over, no more than the work needs.
unsigned bsp_grid(int64_t work) {
    const unsigned need = grid_for(work, kBB);
    return std::min(need, 256u * 16u);
}

// The item segments of the graph's blocks (rows and columns), staged on the
// device.
struct Segs {
    DArray<BspSeg> segs;
    DArray<int64_t> pre;
    int32_t n = 0;
    int64_t total = 0;
};

void make_segs(pgabb_graph *g, Segs &out) {
    hipStream_t s = g->stream;
    const int32_t *arena = g->arena.get();
    std::vector<BspSeg> sv;
    std::vector<int64_t> pv(1, 0);
    for (const BlockInfo &bi : g->blocks) {
        if (bi.nnz == 0) continue;
        if (bi.nitems > 0) {
            sv.push_back({arena + bi.off_items(), arena + bi.off_col(), g->base[bi.i], g->base[bi.j]});
            pv.push_back(pv.back() + bi.nitems);
        }
        if (bi.ncitems > 0) {
            sv.push_back({arena + bi.off_citems(), arena + bi.off_crow(), g->base[bi.j], g->base[bi.i]});
            pv.push_back(pv.back() + bi.ncitems);
        }
    }
    out.n = static_cast<int32_t>(sv.size());
    out.total = pv.back();
    if (out.n == 0) return;
    Staged<BspSeg> hs(sv.size(), s);
    Staged<int64_t> hp(pv.size(), s);
    std::copy(sv.begin(), sv.end(), hs.get());
    std::copy(pv.begin(), pv.end(), hp.get());
    out.segs.reset(sv.size(), s);
    out.pre.reset(pv.size(), s);
    PGABB_HIP(hipMemcpyAsync(out.segs.get(), hs.get(), hs.bytes(), hipMemcpyHostToDevice, s));
    PGABB_HIP(hipMemcpyAsync(out.pre.get(), hp.get(), hp.bytes(), hipMemcpyHostToDevice, s));
}

// The computation runs on the graph's device blocks; a graph that was never
// partitioned is partitioned with p = 1 first.
void require_blocks(pgabb_graph *g) {
    if (g->p == 0) partition_graph(g, 1, PGABB_CUT_NNZ, nullptr);
    PGABB_REQUIRE(!g->blocks_on_host, PGABB_ESTATE,
                  "the graph's blocks are held in host memory (streamed); the bulk-synchronous "
                  "computations need them in device memory: partition the graph again");
}

}  // namespace

int64_t components(pgabb_graph *g, int32_t *label, bool on_device, int32_t *iterations) {
    const auto t0 = std::chrono::steady_clock::now();
    hipStream_t s = g->stream;
    const int32_t n = g->n;
    int32_t iters = 0;
    int64_t comps = 0;
    double kernel_ms = 0;
    if (n > 0) {
        require_blocks(g);
        DArray<int32_t> C(static_cast<size_t>(n), s);
        DArray<unsigned long long> ctr(1 + kBspQueueWords, s);  // roots, work queues
        Staged<unsigned long long> hctr(1, s);
        StreamTimer tm;
        tm.start(s);
        zero_words(ctr.get(), 1 + kBspQueueWords, s);
        k_sv_first<<<bsp_grid(n), kBB, 0, s>>>(g->row_off.get(), g->col.get(), n, C.get());
        k_sv_link<<<bsp_grid(n), kBB, 0, s>>>(C.get(), n);
        iters = 2;
        if (g->m > 0) {
            k_sv_second<<<bsp_grid(n), kBB, 0, s>>>(g->row_off.get(), g->col.get(), n, C.get());
            k_sv_link<<<bsp_grid(n), kBB, 0, s>>>(C.get(), n);
            k_sv_hook_edges<<<std::min(bsp_grid(n), 2048u), kBB, 0, s>>>(g->row_off.get(), g->col.get(), n, C.get(),
                                                                        ctr.get() + 1);
            k_sv_link<<<bsp_grid(n), kBB, 0, s>>>(C.get(), n);
            iters = 6;
        }
        PGABB_HIP(hipGetLastError());
        DArray<int32_t> minid(static_cast<size_t>(n), s);
        DArray<int32_t> own;
        int32_t *dst = label;
        if (!on_device) {
            own.reset(static_cast<size_t>(n), s);
            dst = own.get();
        }
        k_fill_i32<<<bsp_grid(n), kBB, 0, s>>>(minid.get(), INT32_MAX, n);
        k_sv_minid<<<std::min(bsp_grid(n), 512u), kBB, 0, s>>>(C.get(), g->rank.get(), n, minid.get(), ctr.get());
        k_sv_label<<<bsp_grid(n), kBB, 0, s>>>(C.get(), g->rank.get(), minid.get(), n, dst);
        PGABB_HIP(hipGetLastError());
        tm.stop(s);
        PGABB_HIP(hipMemcpyAsync(hctr.get(), ctr.get(), sizeof(unsigned long long), hipMemcpyDeviceToHost, s));
        if (!on_device)
            PGABB_HIP(hipMemcpyAsync(label, dst, sizeof(int32_t) * static_cast<size_t>(n), hipMemcpyDeviceToHost, s));
        PGABB_HIP(hipStreamSynchronize(s));
        kernel_ms += tm.ms();
        comps = static_cast<int64_t>(hctr[0]);
    }
    if (iterations) *iterations = iters;
    g->t_kernel_ms = kernel_ms;
    g->kernel_launches = iters;
    g->t_count_ms = std::chrono::duration<double, std::milli>(std::chrono::steady_clock::now() - t0).count();
    return comps;
}

int32_t pagerank(pgabb_graph *g, double damping, double tol, int32_t max_iter, double *ranks, bool on_device,
                 double *last_err) {
    const auto t0 = std::chrono::steady_clock::now();
    hipStream_t s = g->stream;
    const int32_t n = g->n;
    int32_t iters = 0;
    double err = 0, kernel_ms = 0;
    if (n > 0) {
        require_blocks(g);
        Segs sg;
        make_segs(g, sg);
        DArray<double> r(static_cast<size_t>(n), s), contrib(static_cast<size_t>(n), s), acc(static_cast<size_t>(n), s);
        DArray<double> derr(kPrRound, s);
        Staged<double> herr(kPrRound, s);
        const double teleport = (1.0 - damping) / n;
        StreamTimer tm;
        tm.start(s);
        k_pr_init<<<bsp_grid(n), kBB, 0, s>>>(r.get(), acc.get(), g->outdeg.get(), g->indeg.get(), n, 1.0 / n,
                                              contrib.get());
        PGABB_HIP(hipGetLastError());
        tm.stop(s);
        kernel_ms += tm.ms();
        for (bool stop = max_iter <= 0; !stop;) {
            const int round = std::min(kPrRound, max_iter - iters);
            tm.start(s);
            zero_words(reinterpret_cast<unsigned long long *>(derr.get()), kPrRound, s);  // +0.0 is all zero bits
            for (int q = 0; q < round; ++q) {
                const double *prev = q ? derr.get() + q - 1 : nullptr;
                if (sg.total > 0)
                    k_pr_pull<<<bsp_grid(sg.total), kBB, 0, s>>>(sg.segs.get(), sg.pre.get(), sg.n, contrib.get(),
                                                                 acc.get(), prev, tol);
                k_pr_update<<<std::min(bsp_grid(n), 512u), kBB, 0, s>>>(r.get(), acc.get(), g->outdeg.get(),
                                                                       g->indeg.get(), n, teleport, damping,
                                                                       contrib.get(), derr.get() + q, prev, tol);
            }
            PGABB_HIP(hipGetLastError());
            tm.stop(s);
            PGABB_HIP(hipMemcpyAsync(herr.get(), derr.get(), sizeof(double) * kPrRound, hipMemcpyDeviceToHost, s));
            PGABB_HIP(hipStreamSynchronize(s));
            kernel_ms += tm.ms();
            for (int q = 0; q < round && !stop; ++q) {
                ++iters;
                err = herr[q];
                stop = err < tol;
            }
            stop = stop || iters >= max_iter;
        }
        DArray<double> own;
        double *dst = ranks;
        if (!on_device) {
            own.reset(static_cast<size_t>(n), s);
            dst = own.get();
        }
        k_pr_by_id<<<bsp_grid(n), kBB, 0, s>>>(r.get(), g->rank.get(), n, dst);
        PGABB_HIP(hipGetLastError());
        if (!on_device)
            PGABB_HIP(hipMemcpyAsync(ranks, dst, sizeof(double) * static_cast<size_t>(n), hipMemcpyDeviceToHost, s));
        PGABB_HIP(hipStreamSynchronize(s));
    }
    if (last_err) *last_err = err;
    g->t_kernel_ms = kernel_ms;
    g->kernel_launches = iters;
    g->t_count_ms = std::chrono::duration<double, std::milli>(std::chrono::steady_clock::now() - t0).count();
    return iters;
}

}  // namespace pgabb
