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

// tv[r] (by rank): the counts of r's out-edges (its row) and of its in-edges
// (their CSR positions), 16 lanes a vertex.  No atomics: adding each edge's
// count to both of its ends took 116 us on 200,003 vertices of a random
// geometric graph, the additions going past the L2s.
__global__ __launch_bounds__(kVB) void k_vertex_sums(const int64_t *__restrict__ row_off,
                                                      const int64_t *__restrict__ in_off,
                                                      const uint32_t *__restrict__ in_pos,
                                                      const uint32_t *__restrict__ sup, int32_t n,
                                                      unsigned long long *__restrict__ tv) {
    const int64_t per = kVB / 16;
    const int sub = threadIdx.x & 15;
    // (the loop bound is uniform across a wave: every lane shuffles)
    for (int64_t r0 = blockIdx.x * per + (threadIdx.x / kWave) * (kWave / 16); r0 < n; r0 += gridDim.x * per) {
        const int64_t r = r0 + (threadIdx.x & (kWave - 1)) / 16;
        unsigned long long sum = 0;
        if (r < n) {
            const int64_t e1 = row_off[r + 1], k1 = in_off[r + 1];
            for (int64_t e = row_off[r] + sub; e < e1; e += 16) sum += sup[e];
            for (int64_t k = in_off[r] + sub; k < k1; k += 16) sum += sup[in_pos[k]];
        }
#pragma unroll
        for (int m = 1; m < 16; m <<= 1) sum += shfl_xor_t(sum, m);
        if (r < n && sub == 0) tv[r] = sum;
    }
}

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
        k_vertex_sums<<<std::min(grid_for(n, kVB / 16), 16384u), kVB, 0, s>>>(
            g->row_off.get(), in_off.get(), in_pos.get(), sup.get(), n, tv.get());
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
