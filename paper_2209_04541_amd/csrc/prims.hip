// Device-wide primitives used by the build phase: exclusive prefix sums and
// the radix sort of stored keys (radix.hpp).
#include "common.hpp"
#include "radix.hpp"
#include "wave.hpp"

namespace pgabb {

// ---------------------------------------------------------------- scans

namespace {

constexpr int SC_BLOCK = 256;
constexpr int SC_ITEMS = 8;
constexpr int SC_TILE = SC_BLOCK * SC_ITEMS;

// Up to this many tiles a workgroup of the second launch adds up the sums of
// the tiles before its own itself (from L2: at most 64 KB, 128 of 64-bit sums),
// so a scan is two launches; above, the sums are scanned first.
constexpr int64_t SC_DIRECT = 16384;
// Up to this many tiles, out not aliasing in, one launch does it all: a
// workgroup adds up the input before its own tile (at most 32 K values).  A
// small scan is bound by its launches.
constexpr int64_t SC_SMALL = 16;

template <class I, class T>
__global__ __launch_bounds__(SC_BLOCK) void k_tile_sums(const I *__restrict__ in, int64_t n,
                                                        T *__restrict__ sums) {
    __shared__ T wt[SC_BLOCK / 64];
    const int64_t base = static_cast<int64_t>(blockIdx.x) * SC_TILE;
    T acc = 0;
#pragma unroll
    for (int i = 0; i < SC_ITEMS; ++i) {
        int64_t idx = base + i * SC_BLOCK + threadIdx.x;
        if (idx < n) acc += static_cast<T>(in[idx]);
    }
    acc = wave_sum(acc);
    if ((threadIdx.x & 63) == 0) wt[threadIdx.x >> 6] = acc;
    __syncthreads();
    if (threadIdx.x == 0) {
        T t = 0;
        for (int w = 0; w < SC_BLOCK / 64; ++w) t += wt[w];
        sums[blockIdx.x] = t;
    }
}

// What `before` holds: nothing (one tile), the tiles' sums, the scanned sums,
// or the input itself.
enum : int { kBeforeNone = 0, kBeforeSums = 1, kBeforeScanned = 2, kBeforeInput = 3 };

template <class I, class T, int BEFORE>
__global__ __launch_bounds__(SC_BLOCK) void k_tile_scan(const I *in, T *out, int64_t n, const T *__restrict__ sums,
                                                        T *total_dev) {
    __shared__ T s[SC_TILE];
    __shared__ T wt[SC_BLOCK / 64];
    const int64_t base = static_cast<int64_t>(blockIdx.x) * SC_TILE;
    const int tid = threadIdx.x;
    const int lane = tid & 63, w = tid >> 6;
    T tile_off = 0;  // sum of the input before this tile
    if (BEFORE == kBeforeScanned) tile_off = sums[blockIdx.x];
    if (BEFORE == kBeforeSums || BEFORE == kBeforeInput) {
        const int64_t count = BEFORE == kBeforeSums ? static_cast<int64_t>(blockIdx.x) : base;
        T acc = 0;
        for (int64_t q = tid; q < count; q += SC_BLOCK)
            acc += BEFORE == kBeforeSums ? sums[q] : static_cast<T>(in[q]);
        acc = wave_sum(acc);
        if (lane == 0) wt[w] = acc;
        __syncthreads();
        for (int q = 0; q < SC_BLOCK / 64; ++q) tile_off += wt[q];
        __syncthreads();
    }
#pragma unroll
    for (int i = 0; i < SC_ITEMS; ++i) {
        int64_t idx = base + i * SC_BLOCK + tid;
        s[i * SC_BLOCK + tid] = idx < n ? static_cast<T>(in[idx]) : T(0);
    }
    __syncthreads();
    T v[SC_ITEMS];
    T run = 0;
#pragma unroll
    for (int i = 0; i < SC_ITEMS; ++i) {
        v[i] = run;
        run += s[tid * SC_ITEMS + i];
    }
    // exclusive scan of the per-thread totals across the workgroup
    T incl = wave_inclusive_scan(run);
    if (lane == 63) wt[w] = incl;
    __syncthreads();
    T wave_off = 0, block_total = 0;
    for (int q = 0; q < SC_BLOCK / 64; ++q) {
        if (q < w) wave_off += wt[q];
        block_total += wt[q];
    }
    const T off = tile_off + wave_off + incl - run;
#pragma unroll
    for (int i = 0; i < SC_ITEMS; ++i) s[tid * SC_ITEMS + i] = v[i] + off;
    __syncthreads();
#pragma unroll
    for (int i = 0; i < SC_ITEMS; ++i) {
        int64_t idx = base + i * SC_BLOCK + tid;
        if (idx < n) out[idx] = s[i * SC_BLOCK + tid];
    }
    if (total_dev && blockIdx.x == gridDim.x - 1 && tid == 0) *total_dev = tile_off + block_total;
}

template <class I, class T>
void scan_exclusive(const I *in, T *out, int64_t n, T *total_dev, hipStream_t s) {
    if (n <= 0) {
        if (total_dev) PGABB_HIP(hipMemsetAsync(total_dev, 0, sizeof(T), s));
        return;
    }
    const int64_t ntiles = (n + SC_TILE - 1) / SC_TILE;
    const unsigned grid = static_cast<unsigned>(ntiles);
    if (ntiles == 1) {
        k_tile_scan<I, T, kBeforeNone><<<1, SC_BLOCK, 0, s>>>(in, out, n, nullptr, total_dev);
    } else if (ntiles <= SC_SMALL && static_cast<const void *>(in) != static_cast<const void *>(out)) {
        k_tile_scan<I, T, kBeforeInput><<<grid, SC_BLOCK, 0, s>>>(in, out, n, nullptr, total_dev);
    } else {
        DArray<T> sums(static_cast<size_t>(ntiles), s);
        k_tile_sums<I, T><<<grid, SC_BLOCK, 0, s>>>(in, n, sums.get());
        PGABB_HIP(hipGetLastError());
        if (ntiles <= SC_DIRECT) {
            k_tile_scan<I, T, kBeforeSums><<<grid, SC_BLOCK, 0, s>>>(in, out, n, sums.get(), total_dev);
        } else {
            scan_exclusive<T, T>(sums.get(), sums.get(), ntiles, nullptr, s);
            k_tile_scan<I, T, kBeforeScanned><<<grid, SC_BLOCK, 0, s>>>(in, out, n, sums.get(), total_dev);
        }
    }
    PGABB_HIP(hipGetLastError());
}

}  // namespace

void scan_exclusive_u32(const uint32_t *in, uint32_t *out, int64_t n, uint32_t *total_dev,
                        hipStream_t s) {
    scan_exclusive<uint32_t, uint32_t>(in, out, n, total_dev, s);
}

void scan_exclusive_i64(const int64_t *in, int64_t *out, int64_t n, int64_t *total_dev,
                        hipStream_t s) {
    scan_exclusive<int64_t, int64_t>(in, out, n, total_dev, s);
}

void scan_exclusive_i32(const int32_t *in, int64_t *out, int64_t n, int64_t *total_dev, hipStream_t s) {
    scan_exclusive<int32_t, int64_t>(in, out, n, total_dev, s);
}

bool radix_sort_u64(uint64_t *keys, uint64_t *keys_alt, uint32_t *vals, uint32_t *vals_alt,
                    int64_t n, int nbits, hipStream_t s) {
    return radix_sort_impl<uint64_t>(keys, keys_alt, vals, vals_alt, n, 0, nbits, s);
}

bool radix_sort_u64_bits(uint64_t *keys, uint64_t *keys_alt, uint32_t *vals, uint32_t *vals_alt,
                         int64_t n, int lo_bit, int hi_bit, hipStream_t s) {
    return radix_sort_impl<uint64_t>(keys, keys_alt, vals, vals_alt, n, lo_bit, hi_bit, s);
}

bool radix_sort_u32(uint32_t *keys, uint32_t *keys_alt, uint32_t *vals, uint32_t *vals_alt,
                    int64_t n, int nbits, hipStream_t s) {
    return radix_sort_impl<uint32_t>(keys, keys_alt, vals, vals_alt, n, 0, nbits, s);
}

}  // namespace pgabb
