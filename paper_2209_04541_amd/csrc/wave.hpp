// Wave64 helpers (CDNA: 64 lanes per wavefront).
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>
#include <type_traits>

namespace pgabb {

constexpr int kWave = 64;

__device__ __forceinline__ int lane_id() { return static_cast<int>(threadIdx.x) & (kWave - 1); }

// Shuffles of 32- and 64-bit integers built from 32-bit lane moves.
template <class T>
__device__ __forceinline__ T shfl_up_t(T v, int d) {
    if constexpr (sizeof(T) == 8) {
        const uint64_t u = static_cast<uint64_t>(v);
        const uint32_t lo = __shfl_up(static_cast<uint32_t>(u), d);
        const uint32_t hi = __shfl_up(static_cast<uint32_t>(u >> 32), d);
        return static_cast<T>((static_cast<uint64_t>(hi) << 32) | lo);
    } else {
        return static_cast<T>(__shfl_up(static_cast<uint32_t>(v), d));
    }
}

template <class T>
__device__ __forceinline__ T shfl_xor_t(T v, int m) {
    if constexpr (sizeof(T) == 8) {
        const uint64_t u = static_cast<uint64_t>(v);
        const uint32_t lo = __shfl_xor(static_cast<uint32_t>(u), m);
        const uint32_t hi = __shfl_xor(static_cast<uint32_t>(u >> 32), m);
        return static_cast<T>((static_cast<uint64_t>(hi) << 32) | lo);
    } else {
        return static_cast<T>(__shfl_xor(static_cast<uint32_t>(v), m));
    }
}

template <class T>
__device__ __forceinline__ T shfl_t(T v, int src) {
    if constexpr (sizeof(T) == 8) {
        const uint64_t u = static_cast<uint64_t>(v);
        const uint32_t lo = __shfl(static_cast<uint32_t>(u), src);
        const uint32_t hi = __shfl(static_cast<uint32_t>(u >> 32), src);
        return static_cast<T>((static_cast<uint64_t>(hi) << 32) | lo);
    } else {
        return static_cast<T>(__shfl(static_cast<uint32_t>(v), src));
    }
}

// Inclusive prefix sum of 32-bit values across the 64 lanes of a wave (all
// lanes active), with DPP lane moves only (no LDS traffic): shifts by 1, 2, 4
// and 8 within each row of 16 lanes, then lane 15 of rows 0 and 2 into rows
// 1 and 3, then lane 31 into rows 2 and 3.  A lane whose shifted source lies
// outside its row adds 0.
__device__ __forceinline__ uint32_t wave_scan_dpp(uint32_t x) {
    x += __builtin_amdgcn_update_dpp(0u, x, 0x111, 0xf, 0xf, false);  // row_shr:1
    x += __builtin_amdgcn_update_dpp(0u, x, 0x112, 0xf, 0xf, false);  // row_shr:2
    x += __builtin_amdgcn_update_dpp(0u, x, 0x114, 0xf, 0xf, false);  // row_shr:4
    x += __builtin_amdgcn_update_dpp(0u, x, 0x118, 0xf, 0xf, false);  // row_shr:8
    x += __builtin_amdgcn_update_dpp(0u, x, 0x142, 0xa, 0xf, false);  // row_bcast:15
    x += __builtin_amdgcn_update_dpp(0u, x, 0x143, 0xc, 0xf, false);  // row_bcast:31
    return x;
}

// Inclusive running maximum of 32-bit values across the 64 lanes of a wave
// (all lanes active), with the lane moves of wave_scan_dpp; a lane whose
// shifted source lies outside its row takes 0.
__device__ __forceinline__ uint32_t wave_max_scan_dpp(uint32_t x) {
    x = max(x, static_cast<uint32_t>(__builtin_amdgcn_update_dpp(0u, x, 0x111, 0xf, 0xf, false)));  // row_shr:1
    x = max(x, static_cast<uint32_t>(__builtin_amdgcn_update_dpp(0u, x, 0x112, 0xf, 0xf, false)));  // row_shr:2
    x = max(x, static_cast<uint32_t>(__builtin_amdgcn_update_dpp(0u, x, 0x114, 0xf, 0xf, false)));  // row_shr:4
    x = max(x, static_cast<uint32_t>(__builtin_amdgcn_update_dpp(0u, x, 0x118, 0xf, 0xf, false)));  // row_shr:8
    x = max(x, static_cast<uint32_t>(__builtin_amdgcn_update_dpp(0u, x, 0x142, 0xa, 0xf, false)));  // row_bcast:15
    x = max(x, static_cast<uint32_t>(__builtin_amdgcn_update_dpp(0u, x, 0x143, 0xc, 0xf, false)));  // row_bcast:31
    return x;
}

// Inclusive prefix sum across the 64 lanes of a wave (all lanes active).
template <class T>
__device__ __forceinline__ T wave_inclusive_scan(T x) {
    if constexpr (sizeof(T) == 4) {
        return static_cast<T>(wave_scan_dpp(static_cast<uint32_t>(x)));
    } else {
        const int lane = lane_id();
#pragma unroll
        for (int d = 1; d < kWave; d <<= 1) {
            const T y = shfl_up_t(x, d);
            if (lane >= d) x += y;
        }
        return x;
    }
}

// Pointers that reach a kernel through structs in memory are generic to the
// compiler, and loads through generic pointers are flat loads, which count
// against the LDS counter too: every LDS access or lane shuffle after them
// would wait for them.  Loads through these views are global loads.
template <class T>
using gptr = const __attribute__((address_space(1))) T *;

template <class T>
__device__ __forceinline__ gptr<T> as_global(const T *p) {
    return (gptr<T>)(p);
}

// Calls f(row, e, e1) for every entry e of every row of a CSR, e1 the row's
// end: 16 lanes take a row (rows are mostly short; a thread per row reads them
// uncoalesced and waits for the longest of 64).
template <class F>
__device__ __forceinline__ void for_row_entries(const int64_t *__restrict__ row_off, int32_t n, F f) {
    const int64_t per = blockDim.x / 16;
    for (int64_t r = blockIdx.x * per + threadIdx.x / 16; r < n; r += gridDim.x * per) {
        const int64_t e1 = row_off[r + 1];
        for (int64_t e = row_off[r] + (threadIdx.x & 15); e < e1; e += 16) f(static_cast<int32_t>(r), e, e1);
    }
}

// Sum across the wave, returned to every lane.
template <class T>
__device__ __forceinline__ T wave_sum(T x) {
#pragma unroll
    for (int m = 1; m < kWave; m <<= 1) x += shfl_xor_t(x, m);
    return x;
}

// Sum of v over the workgroup, returned to thread 0; every thread calls it.
// Additions of all workgroups to one word serialise at 5 to 25 ns each, so a
// workgroup adds once (edge support of R-MAT scale 14, one addition per wave 104
// us, per workgroup 63).
__device__ __forceinline__ unsigned long long group_sum(unsigned long long v) {
    __shared__ unsigned long long s_part[1024 / kWave];
    v = wave_sum(v);
    __syncthreads();  // before a further sum's parts
    if (lane_id() == 0) s_part[threadIdx.x / kWave] = v;
    __syncthreads();
    if (threadIdx.x == 0)
        for (unsigned q = 1; q < blockDim.x / kWave; ++q) v += s_part[q];
    return v;
}

// For the 64 consecutive elements handled by one wave, where equal keys form
// runs (the input is sorted), add each run's length to counter[key] with one
// atomic from the run's first lane.  `valid` lanes must form a prefix.
__device__ __forceinline__ void add_run_lengths(bool valid, int64_t key, int32_t *counter) {
    const int lane = lane_id();
    const uint64_t vmask = __ballot(valid);
    const int nvalid = __popcll(vmask);
    const uint32_t klo = __shfl_up(static_cast<uint32_t>(key), 1);
    const uint32_t khi = __shfl_up(static_cast<uint32_t>(static_cast<uint64_t>(key) >> 32), 1);
    const int64_t prev = static_cast<int64_t>((static_cast<uint64_t>(khi) << 32) | klo);
    const bool start = valid && (lane == 0 || prev != key);
    const uint64_t starts = __ballot(start);
    if (start) {
        const uint64_t after = lane == 63 ? 0ull : (starts & (~0ull << (lane + 1)));
        const int next = after ? __ffsll(static_cast<long long>(after)) - 1 : nvalid;
        atomicAdd(&counter[key], next - lane);
    }
}

// Hands the units [0, units) of a persistent launch to its waves.  A wave's
// first unit is its own number; the others are dealt round-robin to Q
// counters (STRIDE words apart, zero before the launch), of which a wave
// starts with that of its workgroup, b mod Q, and moves on when it runs dry.
//
// Operations on one word take some 25 ns each whoever makes them, so a wave's
// first take and its takes that come back empty count: with all takes from
// counters and every wave trying each of 16 queues at the end, a launch of
// 7,168 waves spent over 200 us on them (R-MAT scale 14 counted in one block,
// 137 us with 5,188 waves).  Queues run dry nearly together, so a wave gives
// up after kTakeTries of them, unless the launch is too small for every queue
// to have a workgroup of its own.  (Reading the counters before a take made it
// worse: those reads wait for the same words.)
constexpr int kTakeTries = 2;

template <int Q, int STRIDE>
class UnitTaker {
  public:
    // waves: waves of the launch, wave: this one's number (workgroup by
    // workgroup)
    __device__ __forceinline__ UnitTaker(unsigned long long *next, int64_t units, int64_t waves, int64_t wave)
        : next_(next), units_(units), waves_(waves), first_(wave), q_(static_cast<int>(blockIdx.x % Q)),
          tries_(units <= waves ? 0 : gridDim.x >= Q ? kTakeTries : Q) {}
    // The next unit, or -1 when this wave is done; every lane calls it.
    __device__ __forceinline__ int64_t take(int lane) {
        if (first_ >= 0) {
            const int64_t u = first_;
            first_ = -1;
            if (u >= units_) return -1;
            return u;
        }
        while (tries_ > 0) {
            unsigned long long c = 0;
            if (lane == 0) c = atomicAdd(&next_[q_ * STRIDE], 1ull);
            c = shfl_t(c, 0);
            const int64_t u = waves_ + static_cast<int64_t>(c) * Q + q_;
            if (u < units_) return u;
            --tries_;
            q_ = (q_ + 1) % Q;
        }
        return -1;
    }

  private:
    unsigned long long *next_;
    int64_t units_, waves_, first_;
    int q_, tries_;
};

// Order LDS accesses of the lanes of one wave: what a lane wrote before the
// call is visible to every lane of the wave after it.
__device__ __forceinline__ void wave_lds_sync() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

}  // namespace pgabb
