// A stable least-significant-digit radix sort.  Written for wave64: digit
// ranks inside a wave come from eight ballots (one per digit bit), so a
// 256-thread workgroup ranks 256 keys per round without per-thread
// histograms.
//
// The kernels sit in a header because a sort's input may come from a maker
// that is compiled into its first histogram, which makes the keys, stores them
// for the scatter and counts them at once: a launch less, and the keys are read
// once less (R-MAT scale 20: packing 16.8 M pairs 48 + 31 -> 56 us, orienting 15.7
// M keys 103 + 43 -> 137; a scatter that made the packed keys again took 98 us
// instead of 70).
#pragma once

#include "common.hpp"
#include "wave.hpp"

namespace pgabb {

namespace {

constexpr int RS_BLOCK = 256;
constexpr int RS_WAVES = RS_BLOCK / 64;
constexpr int RS_BINS = 256;
// Keys per thread of a tile: 16, or 4 for inputs of at most RS_DIRECT tiles of
// that size, which then spread over more CUs (a pass over few tiles is bound
// by one tile's chain of steps).
constexpr int RS_LARGE = 16, RS_SMALL = 4;
// Up to this many tiles a pass is two launches: the scatter adds up the tiles'
// histograms itself.  (One launch, each workgroup counting all keys itself,
// took 40 us for 32 K keys against 18 for three.)
constexpr uint32_t RS_DIRECT = 64;

// Tile layout (RS_ITEMS = 16): wave w of the workgroup owns the 1024
// consecutive keys [base + w * 1024, base + (w + 1) * 1024) of the tile, item i
// of lane l being key base + w * 1024 + i * 64 + l.  Every load is 64 consecutive
// keys, and the wave-major order is the keys' own order, which keeps the
// scatter stable.
template <int RS_ITEMS>
__device__ __forceinline__ int64_t rs_index(int64_t base, int w, int i, int lane) {
    return base + static_cast<int64_t>(w) * (RS_ITEMS * 64) + i * 64 + lane;
}

// The lanes of the wave holding the same digit d (< 256, valid lanes only):
// eight ballots, one per digit bit.
__device__ __forceinline__ uint64_t rs_peers(bool valid, uint32_t d) {
    uint64_t same = __ballot(valid);
#pragma unroll
    for (int b = 0; b < 8; ++b) {
        const bool bit = (d >> b) & 1u;
        const uint64_t bb = __ballot(bit);
        same &= bit ? bb : ~bb;
    }
    return same;
}

// Input keys as they lie in memory.
template <class K>
struct StoredKeys {
    const K *keys;
    __device__ __forceinline__ K operator()(int64_t i) const { return keys[i]; }
};

// Per-tile digit histogram, written digit-major: hist[d * ntiles + tile].
template <class K, int RS_ITEMS, class Make>
__global__ __launch_bounds__(RS_BLOCK) void k_rs_hist(Make make, int64_t n,
                                                      int shift, uint32_t mask,
                                                      uint32_t *__restrict__ hist,
                                                      uint32_t ntiles) {
    constexpr int RS_TILE = RS_BLOCK * RS_ITEMS;
    __shared__ uint32_t h[RS_WAVES][RS_BINS];
    const int tid = threadIdx.x, w = tid >> 6;
    for (int i = tid; i < RS_WAVES * RS_BINS; i += RS_BLOCK) (&h[0][0])[i] = 0;
    __syncthreads();
    const int64_t base = static_cast<int64_t>(blockIdx.x) * RS_TILE;
#pragma unroll 4
    for (int i = 0; i < RS_ITEMS; ++i) {
        int64_t idx = base + i * RS_BLOCK + tid;
        if (idx < n) atomicAdd(&h[w][static_cast<uint32_t>(make(idx) >> shift) & mask], 1u);
    }
    __syncthreads();
    uint32_t c = 0;
#pragma unroll
    for (int q = 0; q < RS_WAVES; ++q) c += h[q][tid];
    hist[static_cast<size_t>(tid) * ntiles + blockIdx.x] = c;
}

// One workgroup per digit d: the exclusive scan of hist[d][0 .. ntiles) in
// place (keys of digit d in earlier tiles) and the digit's total in tot[d].
__global__ __launch_bounds__(RS_BLOCK) void k_rs_rowscan(uint32_t *__restrict__ hist, uint32_t ntiles,
                                                         uint32_t *__restrict__ tot) {
    constexpr int ITEMS = 8, CHUNK = RS_BLOCK * ITEMS;
    __shared__ uint32_t s[CHUNK];
    __shared__ uint32_t wt[RS_WAVES];
    uint32_t *row = hist + static_cast<size_t>(blockIdx.x) * ntiles;
    const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
    uint32_t carry = 0;
    for (uint32_t base = 0; base < ntiles; base += CHUNK) {
#pragma unroll
        for (int i = 0; i < ITEMS; ++i) {
            const uint32_t idx = base + i * RS_BLOCK + tid;
            s[i * RS_BLOCK + tid] = idx < ntiles ? row[idx] : 0u;
        }
        __syncthreads();
        uint32_t v[ITEMS], run = 0;
#pragma unroll
        for (int i = 0; i < ITEMS; ++i) {
            v[i] = run;
            run += s[tid * ITEMS + i];
        }
        const uint32_t incl = wave_inclusive_scan(run);
        if (lane == 63) wt[w] = incl;
        __syncthreads();
        uint32_t off = carry, chunk_total = 0;
        for (int q = 0; q < RS_WAVES; ++q) {
            if (q < w) off += wt[q];
            chunk_total += wt[q];
        }
        off += incl - run;
#pragma unroll
        for (int i = 0; i < ITEMS; ++i) s[tid * ITEMS + i] = v[i] + off;
        __syncthreads();
#pragma unroll
        for (int i = 0; i < ITEMS; ++i) {
            const uint32_t idx = base + i * RS_BLOCK + tid;
            if (idx < ntiles) row[idx] = s[i * RS_BLOCK + tid];
        }
        carry += chunk_total;
        __syncthreads();
    }
    if (tid == 0) tot[blockIdx.x] = carry;
}

// Stable scatter of one tile: each wave ranks its keys by digit with
// running per-digit counts of its own (no workgroup barrier per item), the
// tile's digit offsets follow from one scan, the tile is staged in digit
// order in LDS, and each digit run is written to its global offset
// (consecutive threads write consecutive addresses within a run).
// DIRECT: the tiles are few, and the workgroup adds up their histograms itself
// (hist holds counts, not their scan; tot unused), which saves a launch.
// inverse (HAS_V): instead of keys and values, the place of each value goes to
// inverse[value].
template <class K, bool HAS_V, int RS_ITEMS, bool DIRECT>
__global__ __launch_bounds__(RS_BLOCK) void k_rs_scatter(const K *__restrict__ kin,
                                                         K *__restrict__ kout,
                                                         const uint32_t *__restrict__ vin,
                                                         uint32_t *__restrict__ vout,
                                                         int32_t *__restrict__ inverse, int64_t n,
                                                         int shift, uint32_t mask,
                                                         const uint32_t *__restrict__ hist,
                                                         const uint32_t *__restrict__ tot,
                                                         uint32_t ntiles) {
    constexpr int RS_TILE = RS_BLOCK * RS_ITEMS;
    __shared__ K sk[RS_TILE];
    __shared__ uint32_t sv[HAS_V ? RS_TILE : 1];
    __shared__ uint32_t tile_pre[RS_BINS];
    __shared__ uint32_t gofs[RS_BINS];
    __shared__ uint32_t wcnt[RS_WAVES][RS_BINS];
    __shared__ uint32_t wtot[RS_WAVES];

    const int tid = threadIdx.x, w = tid >> 6, lane = tid & 63;
    const int64_t base = static_cast<int64_t>(blockIdx.x) * RS_TILE;
    for (int i = lane; i < RS_BINS; i += 64) wcnt[w][i] = 0;
    {
        // global offset of this tile's digit-tid keys: all keys of lower
        // digits (a scan of the digit totals) plus this digit's keys in
        // earlier tiles (the row scan)
        uint32_t before = 0, t = 0;
        if (tid <= static_cast<int>(mask)) {
            const uint32_t *row = hist + static_cast<size_t>(tid) * ntiles;
            if constexpr (DIRECT) {
                for (uint32_t q = 0; q < ntiles; ++q) {
                    const uint32_t c = row[q];
                    t += c;
                    before += q < blockIdx.x ? c : 0u;
                }
            } else {
                t = tot[tid];
                before = row[blockIdx.x];
            }
        }
        const uint32_t incl = wave_inclusive_scan(t);
        if (lane == 63) wtot[w] = incl;
        __syncthreads();
        uint32_t below = incl - t;
        for (int q = 0; q < w; ++q) below += wtot[q];
        gofs[tid] = below + before;
        __syncthreads();
    }

    K key[RS_ITEMS];
    uint32_t val[HAS_V ? RS_ITEMS : 1];
    uint32_t pos[RS_ITEMS];
#pragma unroll
    for (int i = 0; i < RS_ITEMS; ++i) {
        const int64_t idx = rs_index<RS_ITEMS>(base, w, i, lane);
        key[i] = idx < n ? kin[idx] : K(0);
        if constexpr (HAS_V) val[i] = idx < n ? vin[idx] : 0u;
    }
    wave_lds_sync();

    // ---- rank inside the wave: earlier items, then lower lanes
    const uint64_t lt_mask = (lane == 0) ? 0ull : (~0ull >> (64 - lane));
#pragma unroll
    for (int i = 0; i < RS_ITEMS; ++i) {
        const bool valid = rs_index<RS_ITEMS>(base, w, i, lane) < n;
        const uint32_t d = valid ? (static_cast<uint32_t>(key[i] >> shift) & mask) : 0u;
        const uint64_t same = rs_peers(valid, d);
        const uint32_t below = static_cast<uint32_t>(__popcll(same & lt_mask));
        const uint32_t seen = valid ? wcnt[w][d] : 0u;  // every lane reads before the update
        wave_lds_sync();
        if (valid && below == 0) wcnt[w][d] = seen + static_cast<uint32_t>(__popcll(same));
        wave_lds_sync();
        pos[i] = seen + below;
    }
    __syncthreads();

    // ---- per digit (one per thread): the waves' counts and the tile scan
    uint32_t c = 0;
#pragma unroll
    for (int q = 0; q < RS_WAVES; ++q) {
        const uint32_t x = wcnt[q][tid];
        wcnt[q][tid] = c;  // now: keys of this digit in earlier waves
        c += x;
    }
    const uint32_t incl = wave_inclusive_scan(c);
    if (lane == 63) wtot[w] = incl;
    __syncthreads();
    uint32_t off = 0;
    for (int q = 0; q < w; ++q) off += wtot[q];
    tile_pre[tid] = off + incl - c;
    __syncthreads();

#pragma unroll
    for (int i = 0; i < RS_ITEMS; ++i) {
        if (rs_index<RS_ITEMS>(base, w, i, lane) < n) {
            const uint32_t d = static_cast<uint32_t>(key[i] >> shift) & mask;
            const uint32_t at = tile_pre[d] + wcnt[w][d] + pos[i];
            sk[at] = key[i];
            if constexpr (HAS_V) sv[at] = val[i];
        }
    }
    __syncthreads();

    const int count = static_cast<int>(min<int64_t>(RS_TILE, n - base));
    for (int e = tid; e < count; e += RS_BLOCK) {
        const K k = sk[e];
        const uint32_t d = static_cast<uint32_t>(k >> shift) & mask;
        const uint32_t dst = gofs[d] + (static_cast<uint32_t>(e) - tile_pre[d]);
        if constexpr (HAS_V) {
            if (inverse) {
                inverse[sv[e]] = static_cast<int32_t>(dst);
                continue;
            }
            vout[dst] = sv[e];
        }
        kout[dst] = k;
    }
}

template <class K, int RS_ITEMS, class Make>
void radix_pass(Make make, const K *kc, K *ko, const uint32_t *vc, uint32_t *vo, int32_t *inverse, int64_t n,
                int shift, uint32_t mask, uint32_t *hist, uint32_t ntiles, hipStream_t s) {
    uint32_t *tot = hist + static_cast<size_t>(RS_BINS) * ntiles;
    const bool direct = ntiles <= RS_DIRECT;
    k_rs_hist<K, RS_ITEMS><<<ntiles, RS_BLOCK, 0, s>>>(make, n, shift, mask, hist, ntiles);
    if (!direct) k_rs_rowscan<<<mask + 1, RS_BLOCK, 0, s>>>(hist, ntiles, tot);
    PGABB_HIP(hipGetLastError());
    if (vc && direct)
        k_rs_scatter<K, true, RS_ITEMS, true><<<ntiles, RS_BLOCK, 0, s>>>(kc, ko, vc, vo, inverse, n, shift, mask,
                                                                          hist, tot, ntiles);
    else if (vc)
        k_rs_scatter<K, true, RS_ITEMS, false><<<ntiles, RS_BLOCK, 0, s>>>(kc, ko, vc, vo, inverse, n, shift, mask,
                                                                           hist, tot, ntiles);
    else if (direct)
        k_rs_scatter<K, false, RS_ITEMS, true><<<ntiles, RS_BLOCK, 0, s>>>(kc, ko, nullptr, nullptr, nullptr, n,
                                                                           shift, mask, hist, tot, ntiles);
    else
        k_rs_scatter<K, false, RS_ITEMS, false><<<ntiles, RS_BLOCK, 0, s>>>(kc, ko, nullptr, nullptr, nullptr, n,
                                                                            shift, mask, hist, tot, ntiles);
    PGABB_HIP(hipGetLastError());
}

// Sorts the n keys that make(i) gives, by their bits [lo_bit, hi_bit), n > 1
// and hi_bit > lo_bit.  make(i) leaves key i in keys[i] (and its value, if any,
// in vals[i]) and is called once for each i.  Returns true when
// the sorted data ended in the *_alt buffers.  With inverse, only the place of
// each value is written, to inverse[value].
template <class K, int RS_ITEMS, class Make>
bool radix_sort_tiles(Make make, K *keys, K *keys_alt, uint32_t *vals, uint32_t *vals_alt, int32_t *inverse, int64_t n,
                      int lo_bit, int hi_bit, hipStream_t s) {
    const int64_t tile = RS_BLOCK * RS_ITEMS;
    const uint32_t ntiles = static_cast<uint32_t>((n + tile - 1) / tile);
    DArray<uint32_t> hist(static_cast<size_t>(RS_BINS) * ntiles + RS_BINS, s);
    K *kc = keys, *ko = keys_alt;
    uint32_t *vc = vals, *vo = vals_alt;
    for (int shift = lo_bit; shift < hi_bit; shift += 8) {
        const int width = hi_bit - shift < 8 ? hi_bit - shift : 8;
        const uint32_t mask = (1u << width) - 1u;
        int32_t *inv = shift + 8 >= hi_bit ? inverse : nullptr;
        if (shift == lo_bit)
            radix_pass<K, RS_ITEMS>(make, kc, ko, vc, vo, inv, n, shift, mask, hist.get(), ntiles, s);
        else
            radix_pass<K, RS_ITEMS>(StoredKeys<K>{kc}, kc, ko, vc, vo, inv, n, shift, mask, hist.get(), ntiles, s);
        std::swap(kc, ko);
        std::swap(vc, vo);
    }
    return kc == keys_alt;
}

template <class K, class Make>
bool radix_sort_made(Make make, K *keys, K *keys_alt, uint32_t *vals, uint32_t *vals_alt, int32_t *inverse, int64_t n,
                     int lo_bit, int hi_bit, hipStream_t s) {
    PGABB_REQUIRE(n < (int64_t(1) << 32), PGABB_EINVAL, "radix sort of %lld keys exceeds 2^32",
                  static_cast<long long>(n));
    if (n <= static_cast<int64_t>(RS_DIRECT) * RS_BLOCK * RS_SMALL)
        return radix_sort_tiles<K, RS_SMALL>(make, keys, keys_alt, vals, vals_alt, inverse, n, lo_bit, hi_bit, s);
    return radix_sort_tiles<K, RS_LARGE>(make, keys, keys_alt, vals, vals_alt, inverse, n, lo_bit, hi_bit, s);
}

template <class K>
bool radix_sort_impl(K *keys, K *keys_alt, uint32_t *vals, uint32_t *vals_alt, int64_t n,
                     int lo_bit, int hi_bit, hipStream_t s) {
    if (n <= 1 || hi_bit <= lo_bit) return false;
    return radix_sort_made<K>(StoredKeys<K>{keys}, keys, keys_alt, vals, vals_alt, nullptr, n, lo_bit, hi_bit, s);
}

}  // namespace

}  // namespace pgabb
