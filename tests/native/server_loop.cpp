// The request loop (csrc/server.cpp) on the host: the HIP calls and launches it makes are replaced by
// the ones below, a launch being an event that is done when the scenario says so.  Built and run by
// test_server_loop.py under the host address sanitizer; argv[1] names the scenario.
#include <hip/hip_runtime.h>

#include <atomic>
#include <chrono>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <map>
#include <mutex>
#include <thread>
#include <vector>

#include "nam_internal.h"

namespace {

std::mutex g_mu;
std::map<void*, int> g_on_stream;           // material shape width of the last launch on a stream
std::map<void*, int> g_on_event;            // of the launch an event follows
std::atomic<bool> g_hold[128];              // launches of materials of this width stay on the device
std::atomic<int> g_fail_groups{0};          // grouped launches to fail
std::atomic<int64_t> g_queries{0};          // launched

void launched(const nam_material* m, int64_t n, hipStream_t s) {
    std::lock_guard<std::mutex> g(g_mu);
    g_on_stream[s] = m->shape.H;
    g_queries += n;
}

}  // namespace

// ---- what server.cpp calls
namespace nam {
static std::string g_error;
nam_status set_error(nam_status s, const std::string& msg) { g_error = msg; return s; }
nam_status hip_error(hipError_t, const char* what) { return set_error(NAM_E_HIP, what); }
bool mfma_same_kernel(const nam_material* a, const nam_material* b) { return a->wprec == b->wprec && a->shape.H == b->shape.H; }
hipError_t decode_launch(const nam_material* m, int64_t n, const float*, const float*, const float*, const float*,
                         const float*, float*, hipStream_t s) {
    launched(m, n, s);
    return hipSuccess;
}
hipError_t launch_decode_mfma_group(int count, const nam_material* const* m, const int64_t* n, const float* const*,
                                    const float* const*, const float* const*, const float* const*, float* const*,
                                    hipStream_t s) {
    if (g_fail_groups > 0) {
        --g_fail_groups;
        return hipErrorUnknown;
    }
    for (int i = 0; i < count; ++i) launched(m[i], n[i], s);
    return hipSuccess;
}
}  // namespace nam

extern "C" {
hipError_t hipSetDevice(int) { return hipSuccess; }
hipError_t hipMalloc(void** p, size_t n) { return (*p = std::malloc(n)) ? hipSuccess : hipErrorOutOfMemory; }
hipError_t hipFree(void* p) { std::free(p); return hipSuccess; }
hipError_t hipMemcpyAsync(void* d, const void* s, size_t n, hipMemcpyKind, hipStream_t) { std::memcpy(d, s, n); return hipSuccess; }
hipError_t hipStreamCreateWithFlags(hipStream_t* s, unsigned) { *s = reinterpret_cast<hipStream_t>(new int(0)); return hipSuccess; }
hipError_t hipStreamDestroy(hipStream_t s) { delete reinterpret_cast<int*>(s); return hipSuccess; }
hipError_t hipStreamSynchronize(hipStream_t) { return hipSuccess; }
hipError_t hipEventCreateWithFlags(hipEvent_t* e, unsigned) { *e = reinterpret_cast<hipEvent_t>(new int(0)); return hipSuccess; }
hipError_t hipEventDestroy(hipEvent_t e) { delete reinterpret_cast<int*>(e); return hipSuccess; }
hipError_t hipEventRecord(hipEvent_t e, hipStream_t s) {
    std::lock_guard<std::mutex> g(g_mu);
    g_on_event[e] = g_on_stream[s];
    return hipSuccess;
}
hipError_t hipEventQuery(hipEvent_t e) {
    std::lock_guard<std::mutex> g(g_mu);
    return g_hold[g_on_event[e]] ? hipErrorNotReady : hipSuccess;
}
}

// ---- scenarios
namespace {

using Clock = std::chrono::steady_clock;
constexpr int64_t kTile = 1024;

#define CHECK(c)                                                             \
    do {                                                                     \
        if (!(c)) {                                                          \
            std::printf("line %d: %s\n", __LINE__, #c);                      \
            std::fflush(stdout);                                             \
            std::_Exit(1);                                                   \
        }                                                                    \
    } while (0)

struct Fixture {
    nam_ctx ctx;
    std::vector<nam_material*> mats;
    nam_server* s = nullptr;
    std::vector<float> buf = std::vector<float>(64 * kTile);

    Fixture(int streams, std::vector<int> widths) {
        CHECK(nam_server_create(&ctx, 64 * 48 * kTile, streams, kTile, &s) == NAM_OK);
        for (int w : widths) {
            nam_material* m = new nam_material();
            m->ctx = &ctx;
            m->shape.H = w;
            m->wprec = NAM_F16;
            int id;
            CHECK(nam_server_add_material(s, m, &id) == NAM_OK);
            mats.push_back(m);
        }
    }
    ~Fixture() {
        CHECK(nam_server_destroy(s) == NAM_OK);
        for (auto m : mats) delete m;
    }
    uint64_t submit(int material, int64_t n, double arrival = -1.0) {
        uint64_t t = 0;
        float* p = buf.data();
        CHECK(nam_server_submit(s, material, n, p, p, p, p, p, 0, arrival, &t) == NAM_OK);
        return t;
    }
    nam_status poll(uint64_t t, bool* done) {
        int d = 0;
        const nam_status st = nam_server_poll(s, t, &d, nullptr);
        *done = d != 0;
        return st;
    }
    // until done, at most two seconds
    bool finishes(uint64_t t, nam_status* st = nullptr) {
        const auto end = Clock::now() + std::chrono::seconds(2);
        bool done = false;
        while (Clock::now() < end) {
            const nam_status x = poll(t, &done);
            if (st) *st = x;
            if (done) return true;
        }
        return false;
    }
    void launched_reaches(int64_t n) {
        const auto end = Clock::now() + std::chrono::seconds(2);
        while (g_queries < n && Clock::now() < end) std::this_thread::yield();
        CHECK(g_queries >= n);
    }
    // time for the worker to take a few turns
    static void turns() { std::this_thread::sleep_for(std::chrono::milliseconds(10)); }
};

// A request of one kernel (X), a long one of another (Y), again X: the X's go out together while Y is in
// line, finish and are forgotten by a reset.
void reset_behind_other_kernel() {
    for (int round = 0; round < 5; ++round) {
        g_queries = 0;
        Fixture f(1, {16, 32});
        g_hold[16] = true;
        g_hold[32] = true;
        const uint64_t first = f.submit(0, kTile);
        f.launched_reaches(kTile);                 // on the device alone
        const uint64_t a = f.submit(0, kTile), y = f.submit(1, 12 * kTile), b = f.submit(0, kTile);
        f.turns();                                 // all are in line
        g_hold[16] = false;                        // one X, then the next two X's past Y
        CHECK(f.finishes(first) && f.finishes(a) && f.finishes(b));
        bool done = true;
        CHECK(f.poll(y, &done) == NAM_OK && !done);
        CHECK(nam_server_reset_stats(f.s) == NAM_OK);
        CHECK(f.poll(b, &done) == NAM_E_INVALID_ARG);
        // more requests in the memory that b leaves; replayed ones must not start early
        const uint64_t late = f.submit(0, kTile, 0.05);
        f.turns();
        CHECK(f.poll(late, &done) == NAM_OK && !done);
        g_hold[32] = false;
        CHECK(f.finishes(y) && f.finishes(late));
        CHECK(nam_server_wait_all(f.s) == NAM_OK);
        nam_server_stats_t st;
        CHECK(nam_server_stats(f.s, &st) == NAM_OK && st.completed == 2);
        CHECK(g_queries == 16 * kTile);
    }
}

// A grouped launch fails: its requests fail wherever they stand in line, the others run, a reset forgets
// the failed ones.
void reset_after_failed_group() {
    for (int round = 0; round < 5; ++round) {
        g_queries = 0;
        Fixture f(1, {16, 32});
        g_hold[16] = true;
        g_hold[32] = true;
        const uint64_t first = f.submit(0, kTile);
        f.launched_reaches(kTile);
        const uint64_t a = f.submit(0, kTile), y = f.submit(1, 12 * kTile), b = f.submit(0, kTile);
        f.turns();
        g_fail_groups = 1;
        g_hold[16] = false;
        nam_status st = NAM_OK;
        CHECK(f.finishes(first));
        CHECK(f.finishes(a, &st) && st == NAM_E_HIP);
        CHECK(f.finishes(b, &st) && st == NAM_E_HIP);
        bool done = true;
        CHECK(f.poll(y, &done) == NAM_OK && !done);
        CHECK(nam_server_reset_stats(f.s) == NAM_OK);
        f.turns();
        g_hold[32] = false;
        CHECK(f.finishes(y));
        CHECK(nam_server_wait_all(f.s) == NAM_OK);
    }
}

// A request of which one tile is on the device when its next launch fails: a reset leaves it until that
// tile has ended.
void reset_with_tile_of_failed_request() {
    for (int round = 0; round < 5; ++round) {
        g_queries = 0;
        Fixture f(2, {16, 32});
        CHECK(nam_server_set_group(f.s, 2) == NAM_OK);
        g_hold[16] = true;
        g_hold[32] = true;
        const uint64_t y = f.submit(1, 2 * kTile);            // takes one stream
        f.launched_reaches(2 * kTile);
        const uint64_t r = f.submit(0, 4 * kTile);            // two tiles on the other
        f.launched_reaches(4 * kTile);
        g_fail_groups = 1;
        g_hold[32] = false;                                   // the first stream is free: its launch fails
        nam_status st = NAM_OK;
        CHECK(f.finishes(y));
        CHECK(f.finishes(r, &st) && st == NAM_E_HIP);
        CHECK(nam_server_reset_stats(f.s) == NAM_OK);
        f.turns();
        g_hold[16] = false;                                   // the tiles end
        f.turns();
        CHECK(nam_server_reset_stats(f.s) == NAM_OK);
        const uint64_t after = f.submit(0, kTile);
        CHECK(f.finishes(after));
        CHECK(nam_server_wait_all(f.s) == NAM_OK);
    }
}

// A client that submits to an idle server and asks until the request is done: whatever takes the
// submission over from the inbox, the worker hears of it.
void poll_from_idle() {
    Fixture f(2, {16});
    constexpr int kTimes = 200;
    double sum = 0.0;
    for (int i = 0; i < kTimes; ++i) {
        std::this_thread::sleep_for(std::chrono::milliseconds(1));            // the worker sleeps
        const auto t0 = Clock::now();
        const uint64_t t = f.submit(0, kTile);
        nam_server_stats_t st;
        if (i % 2) CHECK(nam_server_stats(f.s, &st) == NAM_OK);
        CHECK(f.finishes(t));
        sum += std::chrono::duration<double>(Clock::now() - t0).count();
    }
    std::printf("mean %.1f us\n", sum / kTimes * 1e6);
    CHECK(sum / kTimes < 500e-6);                                             // it sleeps for 2 ms at a time
}

}  // namespace

int main(int argc, char** argv) {
    const std::string what = argc > 1 ? argv[1] : "";
    if (what == "reset_behind_other_kernel") reset_behind_other_kernel();
    else if (what == "reset_after_failed_group") reset_after_failed_group();
    else if (what == "reset_with_tile_of_failed_request") reset_with_tile_of_failed_request();
    else if (what == "poll_from_idle") poll_from_idle();
    else return 2;
    std::printf("%s: done\n", what.c_str());
    return 0;
}
