// CPU tests of how finished results reach the threads that collect them
// (paper_0904_4152_amd/csrc/scheduler.h): the pool of solution buffers, results
// of several problems fetched together, and the collecting threads' share.
// Built and run by tests/test_native_results.py; prints "ALL PASS".
#include <atomic>
#include <chrono>
#include <cstdio>
#include <cstdlib>
#include <new>
#include <thread>
#include <vector>

#include "scheduler.h"

using namespace mg;

#define CHECK(cond)                                                                   \
    do {                                                                              \
        if (!(cond)) {                                                                \
            std::fprintf(stderr, "FAIL %s:%d: %s\n", __FILE__, __LINE__, #cond);     \
            std::exit(1);                                                             \
        }                                                                             \
    } while (0)

// An allocation while `refuse` is set on this thread fails (not under
// ThreadSanitizer, whose runtime has the allocation functions itself).
static thread_local bool refuse = false;
#ifndef SANITIZE_THREAD
void* operator new(size_t n) {
    if (refuse) throw std::bad_alloc();
    if (void* p = std::malloc(n)) return p;
    throw std::bad_alloc();
}
void operator delete(void* p) noexcept { std::free(p); }
void operator delete(void* p, size_t) noexcept { std::free(p); }
#endif

static std::atomic<int> held{0};  // buffers allocated and not freed
static double* hold(size_t bytes) {
    ++held;
    return (double*)std::malloc(bytes);
}
static void drop(double* p) {
    --held;
    std::free(p);
}

static void scenario_pool() {
    {
        ResultPool pool(10 * sizeof(double), hold, drop);
        SolutionBuffer a = pool.take(4), b = pool.take(4);
        CHECK(a.size() == 4 && b.size() == 4 && a.data() != b.data() && held == 2);
        CHECK(pool.take(4).empty());  // over the limit
        // giving a buffer back needs no memory
        refuse = true;
        a = SolutionBuffer();
        b = SolutionBuffer();
        refuse = false;
        CHECK(held == 2);
        a = pool.take(4);  // one of the two again
        CHECK(!a.empty() && held == 2);
        b = pool.take(5);  // the idle one of length 4 makes room
        CHECK(b.size() == 5 && held == 2);
        // no memory for the pool's own lists: no buffer, nothing lost
        b = SolutionBuffer();
        SolutionBuffer c;
#ifndef SANITIZE_THREAD
        refuse = true;
        c = pool.take(3);
        refuse = false;
        CHECK(c.empty());
#endif
        c = pool.take(3);
        CHECK(c.size() == 3);
    }
    CHECK(held == 0);
    std::printf("PASS pool\n");
}

static std::atomic<bool> executor_alive{false};
static std::atomic<bool> releasing{false};

// One iteration per problem; results fetched in begin_finish.
class Exec final : public Executor {
public:
    explicit Exec(int slots, bool slow) : slow_(slow), used_(slots, 0), done_(slots, 0), x_(slots) {
        executor_alive = true;
    }
    ~Exec() override { executor_alive = false; }
    double now() override { return 0.0; }
    int capacity() const override { return (int)used_.size(); }
    size_t hierarchy_bytes(int) const override { return 1; }
    void* create_hierarchy(int L) override { return new int(L); }
    void destroy_hierarchy(void* h) override { delete (int*)h; }
    mg_status admit(int slot, void*, const SchedRequest& r) override {
        used_[slot] = r.ticket;
        return MG_OK;
    }
    mg_status upload() override { return MG_OK; }
    mg_status launch_iteration() override {
        ++launched_;
        return MG_OK;
    }
    int64_t launched() const override { return launched_; }
    mg_status wait_iteration(int64_t, const int** done) override {
        for (size_t s = 0; s < used_.size(); ++s) done_[s] = used_[s] != 0;
        *done = done_.data();
        return MG_OK;
    }
    mg_status begin_finish(const int* slots, void* const* hs, const int* keep_x, int n) override {
        for (int i = 0; i < n; ++i) {
            if (!keep_x[i]) continue;
            SolutionBuffer& b = x_[slots[i]];
            b = slow_ ? SolutionBuffer(new double[2], 2, &Exec::slow_release, this) : pool_.take(2);
            if (b.empty()) b = SolutionBuffer::plain(2);
            b.data()[0] = (double)used_[slots[i]];
            b.data()[1] = *(int*)hs[i];
        }
        return MG_OK;
    }
    mg_status finish(int slot, void*, int, SchedResult* out) override {
        out->stats.status = MG_OK;
        out->x = std::move(x_[slot]);
        used_[slot] = 0;
        return MG_OK;
    }

private:
    static void slow_release(void* self, double* p, size_t) {
        releasing = true;
        std::this_thread::sleep_for(std::chrono::milliseconds(200));
        CHECK(executor_alive);
        ++((Exec*)self)->released_;
        delete[] p;
    }
    const bool slow_;
    ResultPool pool_{8 * sizeof(double), hold, drop};  // four results
    std::vector<uint64_t> used_;
    std::vector<int> done_;
    std::vector<SolutionBuffer> x_;
    int64_t launched_ = 0;
    int released_ = 0;
};

// Three threads collect the results of two submitters, by ticket and in order
// of completion: each is its ticket's, from the pool or beyond it.
static void scenario_collectors() {
    auto* ex = new Exec(8, false);
    auto* sched = new Scheduler(ex, 1 << 20);
    sched->start();
    const int per = 300;
    std::atomic<int> got{0};
    std::vector<std::thread> ts;
    for (int id = 0; id < 2; ++id)
        ts.emplace_back([&, id] {
            for (int i = 0; i < per; ++i) {
                uint64_t t = 0;
                std::string err;
                CHECK(sched->submit(3 + id, 1e-8, 0.0, 1, 1, 1, &t, &err) == MG_OK);
            }
        });
    for (int id = 0; id < 3; ++id)
        ts.emplace_back([&] {
            while (got.load() < 2 * per) {
                uint64_t t = 0;
                double x[2] = {0, 0};
                mg_stats st{};
                std::string err;
                const mg_status r = sched->next(0.05, &t, x, &st, &err);
                if (r == MG_ERR_BUSY) continue;
                CHECK(r == MG_OK && x[0] == (double)t && (x[1] == 3 || x[1] == 4));
                ++got;
            }
        });
    for (std::thread& t : ts) t.join();
    CHECK(got == 2 * per);
    delete sched;
    delete ex;
    CHECK(held == 0);
    std::printf("PASS collectors\n");
}

// A server is destroyed while a thread is still taking a result out of it: the
// executor lives until the result's buffer is back.
static void scenario_destroyed_while_collecting() {
    auto* ex = new Exec(1, true);
    auto* sched = new Scheduler(ex, 1 << 20);
    sched->start();
    uint64_t t = 0;
    std::string err;
    CHECK(sched->submit(3, 1e-8, 0.0, 1, 1, 1, &t, &err) == MG_OK);
    mg_server_info_t info{};
    for (int i = 0; i < 20000 && info.completed == 0; ++i) {
        std::this_thread::sleep_for(std::chrono::microseconds(100));
        sched->info(&info);
    }
    CHECK(info.completed == 1);
    std::thread collector([&] {
        double x[2] = {0, 0};
        mg_stats st{};
        std::string e;
        CHECK(sched->poll(t, x, &st, &e) == MG_OK && x[0] == (double)t);
    });
    for (int i = 0; i < 20000 && !releasing; ++i)
        std::this_thread::sleep_for(std::chrono::microseconds(100));
    CHECK(releasing);
    delete sched;
    delete ex;
    collector.join();
    std::printf("PASS destroyed_while_collecting\n");
}

int main() {
    scenario_pool();
    scenario_collectors();
    scenario_destroyed_while_collecting();
    std::printf("ALL PASS\n");
    return 0;
}
