// Host model of the HIP runtime calls that the streamer, the server and the
// memory caches make (for tests/test_streamer_model.py and
// tests/test_server_model.py): a stream is a queue whose operations run later,
// in any order that the streams' order and the events allow; copies and fills
// are checked against the allocations they name, events and streams for use
// after they were destroyed, and events for being asked or waited for after the
// stream they were recorded on was.
#pragma once
#include <cstdint>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <deque>
#include <functional>
#include <map>
#include <memory>
#include <mutex>
#include <random>
#include <set>
#include <vector>
#define __host__
#define __device__
#define __forceinline__ inline
typedef int hipError_t;
enum { hipSuccess = 0, hipErrorOutOfMemory = 2, hipErrorNotReady = 600, hipErrorInvalidHandle = 400 };
enum hipMemcpyKind { hipMemcpyHostToDevice, hipMemcpyDeviceToHost, hipMemcpyDeviceToDevice };
enum { hipStreamNonBlocking = 1, hipEventDisableTiming = 2, hipHostMallocDefault = 0 };
struct Rec { bool done = false; };
struct StreamT;
struct EventT { std::shared_ptr<Rec> last; StreamT *on = nullptr; bool alive = true; };
struct Op { std::function<void()> run; std::shared_ptr<Rec> wait, mark; };
struct StreamT { std::deque<Op> q; };
typedef StreamT *hipStream_t;
typedef EventT *hipEvent_t;
struct Sim {
    std::recursive_mutex mu;
    std::unique_lock<std::recursive_mutex> lock() { return std::unique_lock<std::recursive_mutex>(mu); }
    std::mt19937 rng{1};
    std::set<StreamT *> streams;
    std::vector<std::unique_ptr<StreamT>> all_s;
    std::vector<std::unique_ptr<EventT>> all_e;
    std::map<char *, size_t> dev, host;  // live allocations
    StreamT null_stream;
    long ops = 0;
    int lazy = 2;  // mean number of ops run per API call
    bool ready(StreamT *s) { return !s->q.empty() && (!s->q.front().wait || s->q.front().wait->done); }
    bool step(StreamT *s) {
        if (!ready(s)) return false;
        Op op = std::move(s->q.front());
        s->q.pop_front();
        if (op.run) op.run();
        if (op.mark) op.mark->done = true;
        ++ops;
        return true;
    }
    bool any() {
        std::vector<StreamT *> r;
        for (auto *s : streams) if (ready(s)) r.push_back(s);
        if (ready(&null_stream)) r.push_back(&null_stream);
        if (r.empty()) return false;
        return step(r[rng() % r.size()]);
    }
    void drift() { int k = lazy ? rng() % (2 * lazy) : 0; while (k-- > 0 && any()) {} }
    void finish(StreamT *s) { while (!s->q.empty()) if (!any()) die("deadlock"); }
    void finish_rec(std::shared_ptr<Rec> r) { while (r && !r->done) if (!any()) die("deadlock on event"); }
    [[noreturn]] void die(const char *m) { fprintf(stderr, "SIM: %s\n", m); abort(); }
    StreamT *check(StreamT *s) { if (!s) return &null_stream; if (!streams.count(s)) die("destroyed or unknown stream"); return s; }
    void in(std::map<char *, size_t> &m, const void *p, size_t n, const char *what) {
        char *c = (char *)p; auto it = m.upper_bound(c);
        if (it == m.begin()) die(what);
        --it;
        if (c + n > it->first + it->second) die(what);
    }
};
extern Sim sim;
inline hipError_t hipGetLastError() { return 0; }
inline const char *hipGetErrorString(int) { return "err"; }
inline hipError_t hipGetDevice(int *d) { *d = 0; return 0; }
inline hipError_t hipSetDevice(int) { return 0; }
inline hipError_t hipMemGetInfo(size_t *f, size_t *t) { *f = *t = size_t(1) << 24; return 0; }
inline hipError_t hipStreamCreateWithFlags(hipStream_t *s, int) {
    auto lk = sim.lock();
    sim.all_s.emplace_back(new StreamT);
    *s = sim.all_s.back().get();
    sim.streams.insert(*s);
    return 0;
}
inline hipError_t hipStreamDestroy(hipStream_t s) {
    auto lk = sim.lock();
    sim.check(s);
    sim.finish(s);
    sim.streams.erase(s);
    return 0;
}
inline hipError_t hipStreamSynchronize(hipStream_t s) { auto lk = sim.lock(); s = sim.check(s); sim.finish(s); return 0; }
inline hipError_t hipDeviceSynchronize() { auto lk = sim.lock(); for (auto *s : sim.streams) sim.finish(s); return 0; }
inline hipError_t hipEventCreateWithFlags(hipEvent_t *e, int) {
    auto lk = sim.lock();
    sim.all_e.emplace_back(new EventT);
    *e = sim.all_e.back().get();
    return 0;
}
inline hipError_t hipEventCreate(hipEvent_t *e) { return hipEventCreateWithFlags(e, 0); }
inline void hip_live(hipEvent_t e) { if (!e || !e->alive) sim.die("dead event"); }
inline void hip_known(hipEvent_t e) {
    hip_live(e);
    if (e->on && !sim.streams.count(e->on)) sim.die("event of a destroyed stream");
}
inline hipError_t hipEventDestroy(hipEvent_t e) { auto lk = sim.lock(); hip_live(e); e->alive = false; return 0; }
inline hipError_t hipEventRecord(hipEvent_t e, hipStream_t s) {
    auto lk = sim.lock();
    hip_live(e);
    s = sim.check(s);
    auto r = std::make_shared<Rec>();
    e->last = r;
    e->on = s == &sim.null_stream ? nullptr : s;
    s->q.push_back({nullptr, nullptr, r});
    sim.drift();
    return 0;
}
inline hipError_t hipStreamWaitEvent(hipStream_t s, hipEvent_t e, int) {
    auto lk = sim.lock();
    hip_known(e);
    s = sim.check(s);
    if (e->last) s->q.push_back({nullptr, e->last, nullptr});
    sim.drift();
    return 0;
}
inline hipError_t hipEventSynchronize(hipEvent_t e) {
    auto lk = sim.lock();
    hip_known(e);
    sim.finish_rec(e->last);
    return 0;
}
inline hipError_t hipEventQuery(hipEvent_t e) {
    auto lk = sim.lock();
    hip_known(e);
    sim.drift();
    return !e->last || e->last->done ? 0 : hipErrorNotReady;
}
inline hipError_t hipEventElapsedTime(float *t, hipEvent_t a, hipEvent_t b) {
    auto lk = sim.lock();
    hip_live(a);
    hip_live(b);
    if (!a->last || !a->last->done || !b->last || !b->last->done) sim.die("elapsed of unfinished events");
    *t = 1;
    return 0;
}
inline hipError_t hip_alloc(std::map<char *, size_t> &m, void **p, size_t n) {
    auto lk = sim.lock();
    char *c = (char *)malloc(n);
    memset(c, 0xEE, n);
    m[c] = n;
    *p = c;
    return 0;
}
inline hipError_t hipMalloc(void **p, size_t n) { return hip_alloc(sim.dev, p, n); }
inline hipError_t hipHostMalloc(void **p, size_t n, int) { return hip_alloc(sim.host, p, n); }
inline hipError_t hipFree(void *p) {
    auto lk = sim.lock();
    hipDeviceSynchronize();
    if (!sim.dev.erase((char *)p)) sim.die("bad free");
    free(p);
    return 0;
}
inline hipError_t hipHostFree(void *p) {
    auto lk = sim.lock();
    hipDeviceSynchronize();
    if (!sim.host.erase((char *)p)) sim.die("bad host free");
    free(p);
    return 0;
}
inline hipError_t hipMemcpyAsync(void *d, const void *s, size_t n, hipMemcpyKind k, hipStream_t st) {
    auto lk = sim.lock();
    st = sim.check(st);
   
    if (!n) return 0;
    if (k == hipMemcpyHostToDevice) sim.in(sim.dev, d, n, "H2D outside a device allocation");
    if (k == hipMemcpyDeviceToHost) sim.in(sim.dev, s, n, "D2H outside a device allocation");
    bool pinned = false;
    {
        char *c = (char *)(k == hipMemcpyHostToDevice ? s : d);
        auto it = sim.host.upper_bound(c);
        if (it != sim.host.begin()) {
            --it;
            pinned = c < it->first + it->second;
            if (pinned && c + n > it->first + it->second) sim.die("copy past a pinned allocation");
        }
    }
    st->q.push_back({[=] { memcpy(d, s, n); }, nullptr, nullptr});
    if (!pinned) sim.finish(st);  // pageable: complete on return
    sim.drift();
    return 0;
}
inline hipError_t hipMemsetAsync(void *d, int v, size_t n, hipStream_t st) {
    auto lk = sim.lock();
    st = sim.check(st);
    sim.in(sim.dev, d, n, "memset outside");
    st->q.push_back({[=] { memset(d, v, n); }, nullptr, nullptr});
    sim.drift();
    return 0;
}
