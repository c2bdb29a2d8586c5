// Where the resident blocks of a streamed count sit in its device pool, and
// which of them make room for the next one.
//
// A block is placed where that costs least: in the tightest free gap that
// holds it, else over the run of resident blocks with the smallest sum of the
// caller's costs, never over a pinned one.  The tasks' order is known before
// the first copy, so those costs follow each block's next use.  (Evicting the
// least recently used block until some gap was large enough copied each block
// 2.9 times on R-MAT scale 21 cut 16 x 16 under 45 % of the blocks' bytes:
// blocks about to be read again went out, and the holes that they left were
// scattered, so the whole pool was cleared every other window.)
//
// Host-only code (no HIP types), so the bookkeeping can be checked on the
// CPU.
#pragma once

#include <algorithm>
#include <cstdint>
#include <vector>

namespace pgabb {

class BlockPool {
  public:
    explicit BlockPool(uint64_t cap) : cap_(cap) {}

    // Finds room for `bytes` of block b (not resident) and makes it resident:
    // its offset, or UINT64_MAX if every place that could hold it is taken by
    // pinned blocks.  pinned(v): v must stay.  cost(v) >= 0: what making room
    // by v costs.  evict(v) is called for every block that makes room.
    template <class Pinned, class Cost, class Evict>
    uint64_t place(int32_t b, uint64_t bytes, Pinned &&pinned, Cost &&cost, Evict &&evict) {
        // a place as far left as what stays allows starts at 0 or at the end
        // of a resident block
        const size_t n = at_.size();
        size_t best = SIZE_MAX, best_end = 0;
        double best_cost = 0;
        uint64_t best_gap = 0;
        for (size_t s = 0; s <= n; ++s) {
            const uint64_t lo = s ? at_[s - 1].off + at_[s - 1].bytes : 0;
            if (bytes > cap_ || lo > cap_ - bytes) break;
            size_t e = s;
            double sum = 0;
            bool ok = true;
            for (; ok && e < n && at_[e].off < lo + bytes; ++e) {
                if (pinned(at_[e].block)) ok = false;
                else sum += cost(at_[e].block);
            }
            if (!ok) continue;
            const uint64_t gap = (e < n ? at_[e].off : cap_) - lo - bytes;
            // among equals: nothing evicted, then the tightest fit
            if (best == SIZE_MAX || sum < best_cost ||
                (sum == best_cost && ((e > s) < (best_end > best) ||
                                       ((e > s) == (best_end > best) && gap < best_gap)))) {
                best = s;
                best_end = e;
                best_cost = sum;
                best_gap = gap;
            }
        }
        if (best == SIZE_MAX) return UINT64_MAX;
        const uint64_t off = best ? at_[best - 1].off + at_[best - 1].bytes : 0;
        for (size_t e = best; e < best_end; ++e) evict(at_[e].block);
        at_.erase(at_.begin() + best, at_.begin() + best_end);
        at_.insert(at_.begin() + best, Resident{off, bytes, b});
        return off;
    }

    void clear() { at_.clear(); }

  private:
    struct Resident {
        uint64_t off, bytes;
        int32_t block;
    };
    uint64_t cap_;
    std::vector<Resident> at_;  // by offset
};

}  // namespace pgabb
