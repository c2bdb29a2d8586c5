// Triangles at each vertex (the numerator of the local clustering
// coefficient, PGAbB Section 1), from the per-edge counts: a triangle lies
// on two edges at each of its vertices, so t(v) is half the sum of the
// counts of v's edges.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <chrono>
#include <cstring>

#include "common.hpp"
#include "graph.hpp"
#include "wave.hpp"

namespace pgabb {

namespace {

constexpr int kVB = 256;

// Edges of a vertex that 16 lanes add up; a vertex with more is cut into parts
// of as many, a wave each.
constexpr int64_t kVertexPart = 1024;

// tv[r] (by rank): the counts of r's out-edges (its row) and of its in-edges
// (their CSR positions), 16 lanes a vertex.  No atomics: adding each edge's
// count to both of its ends took 116 us on 200,003 vertices of a random
// geometric graph, the additions going past the L2s.  Vertices of more than
// kVertexPart edges only list their parts (r, part) for the next launch: left
// to 16 lanes, the launch lasted as long as the longest list (R-MAT scale 20 /
// 22 2.37 / 7.2 ms, 0.30 / 1.24 with parts).
__global__ __launch_bounds__(kVB) void k_vertex_sums(const int64_t *__restrict__ row_off,
                                                      const int64_t *__restrict__ in_off,
                                                      const uint32_t *__restrict__ in_pos,
                                                      const uint32_t *__restrict__ sup, int32_t n,
                                                      unsigned long long *__restrict__ tv,
                                                      int2 *__restrict__ parts, unsigned int *__restrict__ nparts) {
    const int64_t per = kVB / 16;
    const int sub = threadIdx.x & 15, lane = lane_id();
    // (the loop bound is uniform across a wave: every lane shuffles)
    for (int64_t r0 = blockIdx.x * per + (threadIdx.x / kWave) * (kWave / 16); r0 < n; r0 += gridDim.x * per) {
        const int64_t r = r0 + lane / 16;
        unsigned long long sum = 0;
        int32_t mine = 0;  // parts of the vertex
        if (r < n) {
            const int64_t e0 = row_off[r], e1 = row_off[r + 1], k0 = in_off[r], k1 = in_off[r + 1];
            const int64_t len = (e1 - e0) + (k1 - k0);
            if (len <= kVertexPart) {
                for (int64_t e = e0 + sub; e < e1; e += 16) sum += sup[e];
                for (int64_t k = k0 + sub; k < k1; k += 16) sum += sup[in_pos[k]];
            } else {
                mine = static_cast<int32_t>((len + kVertexPart - 1) / kVertexPart);
            }
        }
#pragma unroll
        for (int m = 1; m < 16; m <<= 1) sum += shfl_xor_t(sum, m);
        if (r < n && sub == 0) tv[r] = sum;
        if (__ballot(mine != 0) == 0) continue;
        // one addition for the wave's vertices
        const int32_t incl = wave_inclusive_scan(sub == 0 ? mine : 0);
        unsigned int at = 0;
        if (lane == kWave - 1) at = atomicAdd(nparts, static_cast<unsigned int>(incl));
        at = __shfl(at, kWave - 1) + static_cast<unsigned int>(__shfl(incl, lane & ~15) - mine);
        for (int32_t q = sub; q < mine; q += 16) parts[at + q] = make_int2(static_cast<int32_t>(r), q);
    }
}

// The parts of the long vertices: part q of r takes the entries from q *
// kVertexPart on of r's row followed by its in-edges.
__global__ __launch_bounds__(kVB) void k_vertex_parts(const int64_t *__restrict__ row_off,
                                                       const int64_t *__restrict__ in_off,
                                                       const uint32_t *__restrict__ in_pos,
                                                       const uint32_t *__restrict__ sup,
                                                       const int2 *__restrict__ parts,
                                                       const unsigned int *__restrict__ nparts,
                                                       unsigned long long *__restrict__ tv) {
    const int64_t total = *nparts;
    const int64_t waves = static_cast<int64_t>(gridDim.x) * (kVB / kWave);
    for (int64_t w = static_cast<int64_t>(blockIdx.x) * (kVB / kWave) + threadIdx.x / kWave; w < total; w += waves) {
        const int2 part = parts[w];
        const int64_t r = part.x, e0 = row_off[r], out = row_off[r + 1] - e0, k0 = in_off[r];
        const int64_t lo = part.y * kVertexPart, hi = min(lo + kVertexPart, out + (in_off[r + 1] - k0));
        unsigned long long sum = 0;
#pragma unroll 4
        for (int64_t i = lo + lane_id(); i < hi; i += kWave) sum += sup[i < out ? e0 + i : in_pos[k0 + (i - out)]];
        sum = wave_sum(sum);
        if (lane_id() == 0 && sum) atomicAdd(&tv[r], sum);
    }
}

__global__ void k_vertex_zero(unsigned int *p) { *p = 0; }

// out[v] for input id v: half the sum at its rank.
__global__ __launch_bounds__(kVB) void k_vertex_by_id(const int32_t *__restrict__ rank,
                                                       const unsigned long long *__restrict__ tv, int32_t n,
                                                       uint64_t *__restrict__ out) {
    for (int64_t v = blockIdx.x * static_cast<int64_t>(kVB) + threadIdx.x; v < n;
         v += static_cast<int64_t>(gridDim.x) * kVB)
        out[v] = tv[rank[v]] / 2;
}

}  // namespace

uint64_t vertex_counts(pgabb_graph *g, uint64_t *out, bool out_on_device) {
    hipStream_t s = g->stream;
    const auto t0 = std::chrono::steady_clock::now();
    const int32_t n = g->n;
    const int64_t m = g->m;
    uint64_t triangles = 0;
    if (n == 0) {
        g->t_kernel_ms = 0;
        g->kernel_launches = 0;
    } else if (m == 0) {
        g->t_kernel_ms = 0;
        g->kernel_launches = 0;
        if (out_on_device) {
            PGABB_HIP(hipMemsetAsync(out, 0, sizeof(uint64_t) * static_cast<size_t>(n), s));
            PGABB_HIP(hipStreamSynchronize(s));
        } else {
            std::memset(out, 0, sizeof(uint64_t) * static_cast<size_t>(n));
        }
    } else {
        DArray<uint32_t> sup(static_cast<size_t>(m), s);
        DArray<int64_t> in_off;
        DArray<uint32_t> in_pos;
        triangles = edge_support(g, sup.get(), true, &in_off, &in_pos);  // kernel time and launches of the support pass
        DArray<unsigned long long> tv(static_cast<size_t>(n), s);
        // a long vertex has its edges over kVertexPart in parts, rounded up; there
        // are fewer such vertices than whole parts
        const bool some_long = static_cast<int64_t>(g->max_out) + g->max_in > kVertexPart;
        const int64_t max_parts = some_long ? 4 * m / kVertexPart + 1 : 0;
        DArray<int2> parts(static_cast<size_t>(max_parts), s);
        DArray<unsigned int> nparts(1, s);
        if (some_long) k_vertex_zero<<<1, 1, 0, s>>>(nparts.get());
        k_vertex_sums<<<std::min(grid_for(n, kVB / 16), 16384u), kVB, 0, s>>>(
            g->row_off.get(), in_off.get(), in_pos.get(), sup.get(), n, tv.get(), parts.get(), nparts.get());
        if (some_long)
            k_vertex_parts<<<std::min(grid_for(max_parts, kVB / kWave), 4096u), kVB, 0, s>>>(
                g->row_off.get(), in_off.get(), in_pos.get(), sup.get(), parts.get(), nparts.get(), tv.get());
        DArray<uint64_t> own;
        uint64_t *dst = out;
        if (!out_on_device) {
            own.reset(static_cast<size_t>(n), s);
            dst = own.get();
        }
        k_vertex_by_id<<<grid_for(n, kVB), kVB, 0, s>>>(g->rank.get(), tv.get(), n, dst);
        PGABB_HIP(hipGetLastError());
        if (!out_on_device)
            PGABB_HIP(hipMemcpyAsync(out, dst, sizeof(uint64_t) * static_cast<size_t>(n), hipMemcpyDeviceToHost, s));
        PGABB_HIP(hipStreamSynchronize(s));
    }
    g->t_count_ms = std::chrono::duration<double, std::milli>(std::chrono::steady_clock::now() - t0).count();
    return triangles;
}

}  // namespace pgabb
