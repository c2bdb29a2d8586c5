// Streamed counts over the host model of the runtime (see hip/hip_runtime.h):
// random blocks and tasks, caps and stream counts.  The counting launch checks,
// when it runs, that every word its walk reads is the block's and that the words
// a last segment reads past it lie in the pool, that its tasks, prefix and queue
// counters are there, and adds a known count per task.  usage: trials [seed]
#include <hip/hip_runtime.h>

#include <algorithm>
#include <chrono>

#include "common.hpp"
#include "count.hpp"
#include "graph.hpp"

Sim sim;

namespace pgabb {

int g_orient = kOrientCol, g_parts = 1;
pgabb_graph *g_cur;

void fail(pgabb_status st, const char *fmt, ...) {
    char buf[512];
    va_list a;
    va_start(a, fmt);
    vsnprintf(buf, sizeof buf, fmt, a);
    va_end(a);
    throw Error{st, buf};
}

StreamTimer::~StreamTimer() = default;

// ---- what the streamer calls of the counting code
int orient_of_option(const pgabb_tc_options &, const pgabb_graph *) { return g_orient; }
int32_t staged_max(const pgabb_graph *, const Task &, int) { return 10; }
LaunchKind launch_kind(int32_t, int32_t, int32_t, int32_t) {
    LaunchKind k;
    k.mode = 0;
    k.words = 320;
    k.nparts = g_parts;
    return k;
}
int64_t task_items(const pgabb_graph *g, const Task &t, int orient) {
    const BlockInfo &b = g->blocks[t.bij];
    return orient == kOrientCol ? b.ncitems : b.nitems;
}
int default_grab(int64_t, uint64_t) { return 2; }
int64_t task_work_estimate(const pgabb_graph *g, const Task &t, int) { return 1 + g->blocks[t.bij].nnz; }
uint64_t host_count_task(const pgabb_graph *, const int32_t *, const Task &) { return 0; }

// word w from p on (p may lie before the memory it leads to)
static const int32_t *word(const int32_t *p, int64_t w) {
    return reinterpret_cast<const int32_t *>(reinterpret_cast<intptr_t>(p) + 4 * w);
}

TaskDesc make_desc(const pgabb_graph *g, const int32_t *base, const Task &t, int32_t slot, const int64_t *chunk_dev) {
    auto ref = [&](int32_t b) {
        const BlockInfo &bi = g->blocks[b];
        auto at = [&](int64_t off) { return word(base, chunk_dev[b] + off - bi.chunk_off); };
        return BlockRef{at(bi.off_rptr()), at(bi.off_items()), at(bi.off_col()), at(bi.off_citems()),
                        at(bi.off_crow()), bi.nitems, bi.ncitems};
    };
    return TaskDesc{ref(t.bij), ref(t.bik), ref(t.bjk), 1, slot};
}

static int32_t pattern(int32_t b, int64_t w) { return static_cast<int32_t>((b + 1) * 100003 + w * 7 + 11); }

static void check_block(int32_t b, const BlockRef &r) {
    const BlockInfo &bi = g_cur->blocks[b];
    const int64_t lo = bi.walk_lo(g_orient), hi = bi.walk_hi(g_orient);
    sim.in(sim.dev, word(r.rptr, lo - bi.off_rptr()), 4 * (hi - lo + kSeg - 1), "a block's segments leave the pool");
    for (int64_t w = lo; w < hi; ++w)
        if (*word(r.rptr, w - bi.off_rptr()) != pattern(b, w - bi.chunk_off)) sim.die("a block's words are not there");
}

void launch_tc_tasks(const CountArgs &a, const LaunchKind &lk, int, hipStream_t s, int, int) {
    if (a.total <= 0) return;
    const int words = lk.nparts * kQueueWords;
    sim.check(s)->q.push_back({[a, words] {
        if (a.item_pre[0] != 0 || a.item_pre[a.ntasks] != a.total) sim.die("item prefix");
        sim.in(sim.dev, a.next, 8 * static_cast<size_t>(words), "queue counters");
        for (int q = 0; q < words; ++q) {
            if (a.next[q]) sim.die("queue counters are not clear");
            a.next[q] = 5;
        }
        for (int t = 0; t < a.ntasks; ++t) {
            const TaskDesc &d = a.tasks[t];
            if (d.slot < 0 || d.slot >= static_cast<int>(g_cur->tasks.size())) sim.die("task slot");
            const Task &k = g_cur->tasks[d.slot];
            check_block(k.bij, d.ij);
            check_block(k.bik, d.ik);
            check_block(k.bjk, d.jk);
            a.counts[d.slot] += 1000 + d.slot;
        }
    }, nullptr, nullptr});
    sim.drift();
}

}  // namespace pgabb

using namespace pgabb;

static void make_graph(pgabb_graph *g, std::mt19937 &rng) {
    const int p = 1 + rng() % 9, scale = 1 << (rng() % 9);
    g->p = p;
    g->block_of.assign(p * p, -1);
    g->cuts.resize(p + 1, 100);
    g->base.assign(p, 0);
    for (int i = 0; i < p; ++i)
        for (int j = i; j < p; ++j) {
            if (rng() % 8 == 0) continue;
            BlockInfo b;
            b.i = i;
            b.j = j;
            b.width = 1 + rng() % 40;
            b.nitems = 1 + rng() % 20;
            b.ncitems = 1 + rng() % 20;
            b.nnz = 1 + rng() % (16 * scale);
            b.chunk_off = g->arena_words;
            b.chunk_len = b.end() - b.chunk_off;
            g->arena_words += b.chunk_len;
            g->block_of[i * p + j] = static_cast<int32_t>(g->blocks.size());
            g->blocks.push_back(b);
        }
    for (int i = 0; i < p; ++i)
        for (int j = i; j < p; ++j)
            for (int k = j; k < p; ++k) {
                const int a = g->block_of[i * p + j], b = g->block_of[i * p + k], c = g->block_of[j * p + k];
                if (a >= 0 && b >= 0 && c >= 0) g->tasks.push_back({i, j, k, a, b, c, static_cast<int64_t>(rng() % 1000)});
            }
    std::stable_sort(g->tasks.begin(), g->tasks.end(), [](const Task &a, const Task &b) { return a.weight > b.weight; });
    if (g->blocks.empty()) return;
    g->arena.reset(g->arena_words + kSeg, g->stream);
    PinnedArray<int32_t> h;
    h.reset(g->arena_words);
    for (size_t b = 0; b < g->blocks.size(); ++b)
        for (int64_t w = 0; w < g->blocks[b].chunk_len; ++w)
            h[g->blocks[b].chunk_off + w] = pattern(static_cast<int32_t>(b), w);
    (void)hipMemcpyAsync(g->arena.get(), h.get(), 4 * g->arena_words, hipMemcpyHostToDevice, g->stream);
    (void)hipStreamSynchronize(g->stream);
}

int main(int argc, char **argv) {
    const int trials = atoi(argv[1]), seed0 = argc > 2 ? atoi(argv[2]) : 0;
    long ran = 0, refused = 0;
    hipStream_t gs;
    (void)hipStreamCreateWithFlags(&gs, hipStreamNonBlocking);
    for (int trial = seed0; trial < seed0 + trials; ++trial) {
        std::mt19937 rng(trial);
        sim.rng.seed(trial);
        sim.lazy = rng() % 4 == 0 ? 0 : 1 + rng() % 12;  // 0: nothing runs before the host waits
        g_orient = rng() % 2 ? kOrientCol : kOrientRow;
        g_parts = 1 + rng() % kMaxParts;
        pgabb_graph graph;
        g_cur = &graph;
        graph.stream = gs;
        make_graph(&graph, rng);
        const double share[] = {0.2, 0.35, 0.45, 0.6, 0.85, 1.0, 0.0};
        for (int c = 0; c < 5 && !graph.tasks.empty(); ++c) {
            pgabb_tc_options o{};
            o.num_streams = rng() % 6;
            o.device_cap_bytes = static_cast<uint64_t>(4 * graph.arena_words * share[rng() % 7]);
            try {
                count_streamed(&graph, o);
                ++ran;
            } catch (const Error &e) {
                if (e.status != PGABB_ENOMEM) sim.die(e.message.c_str());  // a task's blocks exceed the cap
                ++refused;
                continue;
            }
            for (size_t t = 0; t < graph.tasks.size(); ++t)
                if (graph.task_counts[t] != 1000 + t) sim.die("task count");
            for (size_t b = 0; b < graph.blocks.size(); ++b)
                for (int64_t w = 0; w < graph.blocks[b].chunk_len; ++w)
                    if (graph.host_arena[graph.blocks[b].chunk_off + w] != pattern(static_cast<int32_t>(b), w))
                        sim.die("host store");
        }
        if (rng() % 5 == 0) release_cached_memory();
    }
    (void)hipStreamSynchronize(gs);
    release_cached_memory();
    printf("%ld %ld\n", ran, refused);
}
