// Reuse of a context's batch tables on the CPU -- TEST INFRASTRUCTURE ONLY.
//
// The "device" of this folder reads a batch's table when its stream gets to the
// launch, frame by frame, so a table that is rewritten before the launch has ended
// gives other frames' outputs.  Every case has a slow batch on its stream (frames that
// take milliseconds) while later calls go round all of the context's tables, and then
// compares every frame with the oracle.  Run under AddressSanitizer and ThreadSanitizer by
// tests/test_batch_slots.py; prints "ok <name>" or "FAIL <name>: ...".
#include <hip/hip_runtime.h>

#include <atomic>
#include <cstdio>
#include <cstring>
#include <functional>
#include <memory>
#include <string>
#include <thread>
#include <vector>

#include "knnf.h"

extern "C" int knn_oracle_filter(int H, int W, int C, int K, int R, float lambda, const float* pc1,
                                 const float* prob, float* out_prob, int32_t* out_class,
                                 int32_t* out_nbr, float* out_dist, int nthreads);

namespace fakedev {
extern std::atomic<double> ns_per_pixel;
}  // namespace fakedev

namespace {

std::string g_why;
#define CHECK(cond)                                                                         \
    do {                                                                                    \
        if (!(cond)) {                                                                      \
            g_why = std::string(#cond) + " (line " + std::to_string(__LINE__) + "): " +     \
                    knnf_last_error();                                                      \
            return false;                                                                   \
        }                                                                                   \
    } while (0)

struct Frame {
    int H, W, C = 2, K, R = 3;
    std::vector<float> pc1, prob, op, ref;
    std::vector<int32_t> oc, refc;
    Frame(int h, int w, int k, uint32_t seed) : H(h), W(w), K(k) {
        uint32_t s = seed * 2654435761u + 99u;
        auto rnd = [&s] {
            s = s * 1664525u + 1013904223u;
            return (float)((s >> 8) & 0xffffff) / 16777216.0f;
        };
        const size_t px = (size_t)H * W;
        pc1.resize(px), prob.resize(px * C), op.assign(px * C, -1.f), oc.assign(px, -1);
        for (float& v : pc1) v = rnd();
        for (float& v : prob) v = rnd();
        ref.resize(px * C), refc.resize(px);
        std::vector<float> d(px * K);
        std::vector<int32_t> n(px * K);
        knn_oracle_filter(H, W, C, K, R, 0.01f, pc1.data(), prob.data(), ref.data(), refc.data(),
                          n.data(), d.data(), 1);
    }
    knnf_frame c() {
        return knnf_frame{H, W, C, K, R, 0.01f, pc1.data(), prob.data(), op.data(), oc.data(),
                          nullptr, nullptr};
    }
    bool right() const { return op == ref && oc == refc; }
};

// n frames filtered by one call.
struct Batch {
    std::vector<std::unique_ptr<Frame>> frames;
    std::vector<knnf_frame> c;
    Batch(int n, uint32_t seed, int tall = 1) {
        for (int k = 0; k < n; ++k) {
            frames.emplace_back(new Frame(tall * (5 + k % 4), 9 + (int)(seed % 5) + k % 3, 4 + k % 3, seed * 100 + k));
            c.push_back(frames.back()->c());
        }
    }
    knnf_status run(knnf_ctx* ctx, hipStream_t s, int launch = KNNF_LAUNCH_GRID) {
        knnf_plan p{};
        p.search = KNNF_SEARCH_PRUNED;
        p.launch = launch;
        p.flags = KNNF_PLAN_NO_INPUT_CHECK;
        return knnf_filter_batch(ctx, c.data(), (int)c.size(), &p, s);
    }
    void clear() {
        for (auto& f : frames) {
            std::fill(f->op.begin(), f->op.end(), -1.f);
            std::fill(f->oc.begin(), f->oc.end(), -1);
        }
    }
    bool right() const {
        for (auto& f : frames)
            if (!f->right()) return false;
        return true;
    }
};

hipStream_t make_stream() {
    hipStream_t s = nullptr;
    hipStreamCreateWithFlags(&s, hipStreamNonBlocking);
    return s;
}

constexpr int kSizes[] = {3, 45};  // a table as a kernel argument, and through the staging

std::vector<std::unique_ptr<Batch>> batches(int count, int n, uint32_t seed) {
    std::vector<std::unique_ptr<Batch>> v;
    for (int k = 0; k < count; ++k) v.emplace_back(new Batch(n, seed + k));
    return v;
}

// The first batch's stream is destroyed while the batch runs, and another, idle
// stream has its handle when the table comes round again.
bool test_destroyed_stream() {
    for (int n : kSizes) {
        knnf_ctx* ctx = nullptr;
        CHECK(knnf_create(&ctx, 0) == KNNF_OK);
        Batch first(n, 1, 8);
        auto later = batches(9, n, 10);
        fakehip::reuse_stream_handles(true);
        hipStream_t a = make_stream();
        CHECK(first.run(ctx, a) == KNNF_OK);
        CHECK(hipStreamDestroy(a) == hipSuccess);
        hipStream_t b = make_stream();
        CHECK(b == a);
        fakehip::reuse_stream_handles(false);
        for (auto& x : later) CHECK(x->run(ctx, nullptr) == KNNF_OK);  // (the fake's runs at once)
        CHECK(hipDeviceSynchronize() == hipSuccess);
        CHECK(first.right());
        for (auto& x : later) CHECK(x->right());
        CHECK(knnf_ctx_status(ctx) == KNNF_OK);
        hipStreamDestroy(b);
        CHECK(knnf_destroy(ctx) == KNNF_OK);
    }
    return true;
}

// Two threads, each on its own per-thread stream: one handle, two streams.
bool test_per_thread_streams() {
    for (int n : kSizes) {
        knnf_ctx* ctx = nullptr;
        CHECK(knnf_create(&ctx, 0) == KNNF_OK);
        Batch first(n, 2, 8);
        auto later = batches(9, n, 30);
        std::atomic<int> at{0};
        knnf_status st = KNNF_OK;
        std::thread a([&] {
            st = first.run(ctx, hipStreamPerThread);
            at.store(1);
            while (at.load() != 2) std::this_thread::yield();
            hipStreamSynchronize(hipStreamPerThread);
        });
        while (at.load() != 1) std::this_thread::yield();
        for (size_t k = 0; k < later.size(); ++k)
            CHECK(later[k]->run(ctx, k < 6 ? nullptr : hipStreamPerThread, KNNF_LAUNCH_PERSISTENT) == KNNF_OK);
        at.store(2);
        a.join();
        hipStreamSynchronize(hipStreamPerThread);
        CHECK(st == KNNF_OK && first.right());
        for (auto& x : later) CHECK(x->right());
        CHECK(knnf_destroy(ctx) == KNNF_OK);
    }
    return true;
}

// Batches recorded in a capture: replays read their tables whenever they come,
// with the context's other batches in between and at the same time.
bool test_captured_batches() {
    for (int n : kSizes) {
        knnf_ctx* ctx = nullptr;
        CHECK(knnf_create(&ctx, 0) == KNNF_OK);
        hipStream_t s = make_stream(), t = make_stream();
        auto rec = batches(6, n, 50), plain = batches(9, n, 70);
        CHECK(plain[0]->run(ctx, s) == KNNF_OK);
        CHECK(hipStreamSynchronize(s) == hipSuccess);
        fakehip::begin_capture(s);
        for (auto& x : rec) CHECK(x->run(ctx, s) == KNNF_OK);
        const fakehip::Graph g = fakehip::end_capture(s);
        for (int turn = 0; turn < 3; ++turn) {
            for (auto& x : rec) x->clear();
            for (auto& x : plain) x->clear();
            fakehip::replay(g, s);
            for (size_t k = 0; k < plain.size(); ++k) {
                CHECK(plain[k]->run(ctx, k % 2 ? t : s) == KNNF_OK);
                if (k == 4) fakehip::replay(g, s);
            }
            CHECK(hipDeviceSynchronize() == hipSuccess);
            for (auto& x : rec) CHECK(x->right());
            for (auto& x : plain) CHECK(x->right());
        }
        hipStreamDestroy(s);
        hipStreamDestroy(t);
        CHECK(knnf_destroy(ctx) == KNNF_OK);
    }
    return true;
}

// A server whose frames are done is closed after its context.
bool test_server_closed_after_its_context() {
    knnf_ctx* ctx = nullptr;
    CHECK(knnf_create(&ctx, 0) == KNNF_OK);
    void* pool = nullptr;
    CHECK(hipMalloc(&pool, 1 << 20) == hipSuccess);
    knnf_server* srv = nullptr;
    CHECK(knnf_server_create(&srv, ctx, pool, 1 << 20, nullptr) == KNNF_OK);
    Batch b(6, 90);
    for (auto& f : b.frames) {
        knnf_host_frame h{};
        h.H = f->H, h.W = f->W, h.C = f->C, h.K = f->K, h.R = f->R, h.lambda = 0.01f;
        h.pc1 = f->pc1.data(), h.prob = f->prob.data(), h.t_arrival = -1.0;
        uint64_t t = 0;
        CHECK(knnf_server_submit(srv, &h, &t) == KNNF_OK);
    }
    CHECK(knnf_server_drain(srv, 60.0) == KNNF_OK);
    CHECK(knnf_destroy(ctx) == KNNF_OK);
    CHECK(knnf_server_destroy(srv) == KNNF_OK);
    hipFree(pool);
    return true;
}

// Windows of more rows than the frame has, up to the largest R, are the whole frame.
bool test_whole_frame_windows() {
    knnf_ctx* ctx = nullptr;
    CHECK(knnf_create(&ctx, 0) == KNNF_OK);
    for (int R : {8, 100000, 0x7fffffff}) {
        Batch b(3, 95);
        for (size_t k = 0; k < b.frames.size(); ++k) {
            Frame& f = *b.frames[k];
            std::vector<float> d(f.pc1.size() * f.K);
            std::vector<int32_t> n(d.size());
            knn_oracle_filter(f.H, f.W, f.C, f.K, f.H, 0.01f, f.pc1.data(), f.prob.data(), f.ref.data(),
                              f.refc.data(), n.data(), d.data(), 1);
            b.c[k].R = R;
        }
        CHECK(b.run(ctx, nullptr) == KNNF_OK);
        CHECK(b.right());
        b.clear();
        for (knnf_frame& c : b.c) CHECK(knnf_filter(ctx, &c, nullptr, nullptr) == KNNF_OK);
        CHECK(b.right());
    }
    CHECK(knnf_destroy(ctx) == KNNF_OK);
    return true;
}

}  // namespace

int main() {
    fakedev::ns_per_pixel.store(2e4);
    const std::vector<std::pair<const char*, std::function<bool()>>> tests = {
        {"destroyed_stream", test_destroyed_stream},
        {"per_thread_streams", test_per_thread_streams},
        {"captured_batches", test_captured_batches},
        {"server_closed_after_its_context", test_server_closed_after_its_context},
        {"whole_frame_windows", test_whole_frame_windows},
    };
    int failed = 0;
    for (const auto& t : tests) {
        const bool ok = t.second();
        if (ok) std::printf("ok %s\n", t.first);
        else std::printf("FAIL %s: %s\n", t.first, g_why.c_str());
        std::fflush(stdout);
        failed += !ok;
    }
    return failed ? 1 : 0;
}
