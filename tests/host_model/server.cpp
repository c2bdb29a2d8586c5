// The request server over the host model of the runtime (see hip/hip_runtime.h):
// servers come and go, their requests built and counted by stand-ins that take
// and leave blocks of the memory caches on the server's streams, as the builds
// and the counting launch do.  Blocks are taken from the caches by another
// stream after each server has ended.  usage: servers [seed]
#include <hip/hip_runtime.h>

#include "common.hpp"
#include "count.hpp"
#include "graph.hpp"

Sim sim;

namespace pgabb {

void fail(pgabb_status st, const char *fmt, ...) { throw Error{st, fmt}; }
pgabb_status capture_status(const Error &e) { return e.status; }

StreamTimer::StreamTimer() = default;
StreamTimer::~StreamTimer() = default;
void StreamTimer::start(hipStream_t) {}
void StreamTimer::stop(hipStream_t) {}
double StreamTimer::ms() { return 0; }

int orient_of_option(const pgabb_tc_options &, const pgabb_graph *) { return kOrientCol; }
int32_t staged_max(const pgabb_graph *, const Task &, int) { return 10; }
LaunchKind launch_kind(int32_t, int32_t, int32_t, int32_t) { return LaunchKind{0, 320}; }
int64_t task_items(const pgabb_graph *, const Task &, int) { return 1; }
int default_grab(int64_t, uint64_t) { return 2; }
uint64_t walked_entries(const pgabb_graph *, int) { return 1; }
TaskDesc make_desc(const pgabb_graph *, const int32_t *, const Task &, int32_t slot, const int64_t *) {
    TaskDesc d{};
    d.slot = slot;
    return d;
}

void build_graph(pgabb_graph *g, const int32_t *src, const int32_t *, int64_t m) {
    if (m) sim.in(sim.dev, src, 4 * static_cast<size_t>(m), "pairs");
    g->m = m;
    DArray<int32_t> scratch(static_cast<size_t>(m) + 1, g->stream);
    Staged<int32_t> read_back(64, g->stream);
    g->col.reset(static_cast<size_t>(m) + 1, g->stream);
}

void partition_graph(pgabb_graph *g, int32_t, int32_t, const int32_t *) {
    Staged<int64_t> tables(32, g->stream);
    g->arena.reset(static_cast<size_t>(g->m) + 1, g->stream);
    g->tasks.resize(1);
}

void launch_tc_tasks(const CountArgs &a, const LaunchKind &, int, hipStream_t s, int, int) {
    auto lk = sim.lock();
    sim.check(s)->q.push_back({[a] {
        for (int t = 0; t < a.ntasks; ++t) a.counts[a.tasks[t].slot] += 7;
    }, nullptr, nullptr});
    sim.drift();
}

}  // namespace pgabb

using namespace pgabb;

int main(int argc, char **argv) {
    const int servers = atoi(argv[1]);
    std::mt19937 rng(argc > 2 ? atoi(argv[2]) : 0);
    hipStream_t own;
    (void)hipStreamCreateWithFlags(&own, hipStreamNonBlocking);
    std::vector<int32_t> ids(4000, 0);
    for (int q = 0; q < servers; ++q) {
        pgabb_server *s = nullptr;
        pgabb_tc_options o{};
        o.num_streams = rng() % 4;
        if (pgabb_server_create(1ull << 40, &o, &s)) return 1;
        std::vector<uint64_t> tickets(1 + rng() % 6);
        for (auto &t : tickets)
            if (pgabb_server_submit(s, 100, static_cast<int64_t>(rng() % 4000), ids.data(), ids.data(), &t)) return 1;
        if (pgabb_server_drain(s)) return 1;
        for (auto t : tickets) {
            int32_t done = 0;
            uint64_t count = 0;
            if (pgabb_server_poll(s, t, &done, &count) || !done || count != 7) return 2;
        }
        pgabb_server_destroy(s);
        // what the next graph does: blocks of every size that the server left
        for (size_t n = 16; n < 40000; n = n * 5 / 4) {
            Staged<int32_t> h(n, own);
            DArray<int32_t> d(n, own);
        }
        if (q % 3 == 2) release_cached_memory();
    }
    (void)hipStreamSynchronize(own);
    release_cached_memory();
    printf("%d\n", servers);
}
