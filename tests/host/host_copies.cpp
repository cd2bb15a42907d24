// Staged host copies (HostStage) on the CPU, over a stand-in for the few
// runtime calls they make: a stream is a queue of copies that nothing carries
// out before somebody waits, so a slot that is filled again before its copy was
// waited for shows in the bytes; pinned memory can be refused; and the last
// error stays set until it is read, as launch checks find it.
// Prints one line per failure and "ok" at the end; the exit status is the
// number of failures (capped at 100).
#include "dbg_runtime.h"

#include <cstdio>
#include <deque>
#include <map>
#include <random>
#include <vector>

namespace {

struct Op {
    void *to;
    const void *from;
    size_t bytes;
};
struct State {
    std::deque<Op> ops;
    uint64_t pushed = 0, done = 0;
};
struct Queue {
    std::shared_ptr<State> state = std::make_shared<State>();
};
struct Event {
    std::shared_ptr<State> q;  // (an event outlives its stream)
    uint64_t upto = 0;
};

std::mutex mu;
hipError_t last = hipSuccess;
bool refuse_pinned = false, refuse_events = false;
uint64_t pinned_calls = 0, pinned_bytes = 0, pinned_most = 0;
std::map<void *, size_t> pinned;

hipError_t said(hipError_t e) {
    if (e != hipSuccess) last = e;
    return e;
}

void drain(State *q, uint64_t upto) {
    while (q->done < upto) {
        const Op op = q->ops.front();
        q->ops.pop_front();
        std::memcpy(op.to, op.from, op.bytes);
        ++q->done;
    }
}

std::shared_ptr<State> &queue(hipStream_t s) { return reinterpret_cast<Queue *>(s)->state; }
Event *event(hipEvent_t e) { return reinterpret_cast<Event *>(e); }

}  // namespace

extern "C" {
hipError_t hipHostMalloc(void **p, size_t bytes, unsigned int) {
    std::lock_guard<std::mutex> lock(mu);
    ++pinned_calls;
    if (refuse_pinned) return said(hipErrorOutOfMemory);
    *p = std::malloc(bytes);
    pinned[*p] = bytes;
    pinned_bytes += bytes;
    pinned_most = std::max(pinned_most, pinned_bytes);
    return hipSuccess;
}
hipError_t hipHostFree(void *p) {
    std::lock_guard<std::mutex> lock(mu);
    pinned_bytes -= pinned[p];
    pinned.erase(p);
    std::free(p);
    return hipSuccess;
}
hipError_t hipMalloc(void **, size_t) {
    std::lock_guard<std::mutex> lock(mu);
    return said(hipErrorOutOfMemory);
}
hipError_t hipFree(void *) { return hipSuccess; }
hipError_t hipEventCreateWithFlags(hipEvent_t *e, unsigned) {
    std::lock_guard<std::mutex> lock(mu);
    if (refuse_events) return said(hipErrorOutOfMemory);
    *e = reinterpret_cast<hipEvent_t>(new Event);
    return hipSuccess;
}
hipError_t hipEventDestroy(hipEvent_t e) {
    delete event(e);
    return hipSuccess;
}
hipError_t hipEventRecord(hipEvent_t e, hipStream_t s) {
    std::lock_guard<std::mutex> lock(mu);
    event(e)->q = queue(s);
    event(e)->upto = queue(s)->pushed;
    return hipSuccess;
}
hipError_t hipEventSynchronize(hipEvent_t e) {
    std::lock_guard<std::mutex> lock(mu);
    if (event(e)->q) drain(event(e)->q.get(), event(e)->upto);
    return hipSuccess;
}
hipError_t hipMemcpyAsync(void *to, const void *from, size_t bytes, hipMemcpyKind, hipStream_t s) {
    std::lock_guard<std::mutex> lock(mu);
    queue(s)->ops.push_back({to, from, bytes});
    ++queue(s)->pushed;
    return hipSuccess;
}
hipError_t hipStreamSynchronize(hipStream_t s) {
    std::lock_guard<std::mutex> lock(mu);
    drain(queue(s).get(), queue(s)->pushed);
    return hipSuccess;
}
hipError_t hipSetDevice(int) { return hipSuccess; }
hipError_t hipGetLastError() {
    std::lock_guard<std::mutex> lock(mu);
    const hipError_t e = last;
    last = hipSuccess;
    return e;
}
}  // extern "C"

static int failures = 0;
#define CHECK(cond, ...)                                                            \
    do {                                                                            \
        if (!(cond)) {                                                              \
            std::lock_guard<std::mutex> lock(mu);                                   \
            if (failures < 20) std::printf("FAIL %s: ", #cond), std::printf(__VA_ARGS__), std::printf("\n"); \
            ++failures;                                                             \
        }                                                                           \
    } while (0)

using dbgrt::HostStage;

// Spans of these sizes there and back again through one stage and stream.
static void round_trip(HostStage &stage, Queue &q, const std::vector<uint64_t> &sizes, uint64_t seed) {
    std::vector<std::vector<unsigned char>> host, dev, back;
    std::vector<HostStage::Span> in, out;
    std::mt19937_64 rng(seed);
    std::vector<uint64_t> block(5003);  // (a prime: no two chunks look alike)
    for (auto &x : block) x = rng();
    for (const uint64_t n : sizes) {
        host.emplace_back(n);
        for (size_t i = 0; i < n; i += 8 * block.size())
            std::memcpy(host.back().data() + i, block.data(), std::min<size_t>(8 * block.size(), n - i));
        dev.emplace_back(n);
        back.emplace_back(n);
    }
    for (size_t i = 0; i < sizes.size(); ++i) {
        in.push_back({sizes[i] ? host[i].data() : nullptr, dev[i].data(), sizes[i]});
        out.push_back({sizes[i] ? back[i].data() : nullptr, dev[i].data(), sizes[i]});
    }
    const uint32_t n = (uint32_t)sizes.size();
    const auto s = reinterpret_cast<hipStream_t>(&q);
    uint64_t total = 0;
    for (const uint64_t x : sizes) total += x;
    CHECK(stage.move(in.data(), n, false, 0, s) == hipSuccess, "in, %llu bytes", (unsigned long long)total);
    CHECK(stage.move(out.data(), n, true, 0, s) == hipSuccess, "out, %llu bytes", (unsigned long long)total);
    for (size_t i = 0; i < sizes.size(); ++i)
        CHECK(host[i] == back[i], "span %zu of %llu bytes", i, (unsigned long long)sizes[i]);
}

static void check_sizes() {
    HostStage stage;
    Queue q;
    const uint64_t small = HostStage::kSmall, chunk = HostStage::kChunk;
    uint64_t seed = 0;
    for (const uint64_t n : {uint64_t(0), uint64_t(1), small - 1, small, small + 1, 2 * small + chunk - 1, 2 * small + 13 * chunk + 7})
        round_trip(stage, q, {n}, ++seed);
    round_trip(stage, q, {0, small + 3, 0, 5, chunk, small + 1}, ++seed);
    round_trip(stage, q, {small, 0}, ++seed);
    stage.release();
}

// What may be refused is done without, and no later launch check finds the error.
static void check_refusals() {
    Queue q;
    for (int what = 0; what < 2; ++what) {
        HostStage stage;
        (what ? refuse_events : refuse_pinned) = true;
        for (int rep = 0; rep < 2; ++rep) {
            round_trip(stage, q, {3 * HostStage::kSmall + 5}, 77);
            CHECK(hipGetLastError() == hipSuccess, "an error is left behind by copies without %s", what ? "events" : "slots");
        }
        refuse_pinned = refuse_events = false;
        round_trip(stage, q, {3 * HostStage::kSmall + 5}, 78);
        stage.release();
    }
    dbgrt::DevBuf d;
    CHECK(d.reserve(64) == hipErrorOutOfMemory && hipGetLastError() == hipSuccess, "device buffer");
    refuse_pinned = true;
    dbgrt::HostBuf h;
    CHECK(h.reserve(64) == hipErrorOutOfMemory && hipGetLastError() == hipSuccess, "pinned buffer");
    dbgrt::PinnedWord w;
    CHECK(!w.get() && hipGetLastError() == hipSuccess, "pinned word");
    refuse_pinned = false;
    CHECK(w.get() != nullptr, "pinned word after a refusal");
    w.release();
}

// Many handles keep no more pinned memory than one, and none when all are gone.
static void check_kept() {
    const uint64_t before = pinned_bytes;  // a page of pinned words
    std::vector<HostStage> stages(10);
    Queue q;
    pinned_most = 0;
    for (size_t i = 0; i < stages.size(); ++i) round_trip(stages[i], q, {HostStage::kSmall + i}, i);
    CHECK(pinned_most == before + HostStage::kSlotBytes, "%llu bytes pinned", (unsigned long long)(pinned_most - before));
    std::vector<std::thread> threads;
    for (size_t t = 0; t < 6; ++t)
        threads.emplace_back([&, t] {
            Queue own;
            round_trip(stages[t], own, {HostStage::kSmall + 64 * t}, t);
        });
    for (auto &t : threads) t.join();
    CHECK(pinned_bytes <= before + HostStage::kIdle * HostStage::kSlotBytes, "%llu bytes kept", (unsigned long long)(pinned_bytes - before));
    for (auto &x : stages) x.release();
    CHECK(pinned_bytes == before, "%llu bytes left", (unsigned long long)(pinned_bytes - before));
    round_trip(stages[0], q, {HostStage::kSmall}, 5);  // and from the start again
    stages[0].release();
    CHECK(pinned_bytes == before, "%llu bytes left", (unsigned long long)(pinned_bytes - before));
}

static void check_threads() {
    std::vector<std::thread> threads;
    for (int t = 0; t < 3; ++t)
        threads.emplace_back([t] {
            HostStage stage;
            Queue q;
            for (int rep = 0; rep < 2; ++rep)
                round_trip(stage, q, {2 * HostStage::kSmall + 4097u * t, 100 + HostStage::kSmall}, 1000 + 10 * t + rep);
            stage.release();
        });
    for (auto &t : threads) t.join();
}

int main() {
    check_sizes();
    check_refusals();
    check_kept();
    check_threads();
    if (failures) std::printf("%d failures\n", failures);
    else std::printf("ok\n");
    return failures > 100 ? 100 : failures;
}
