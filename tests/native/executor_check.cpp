// Host-only checks of what the serving scheduler (tc_sched.cpp) promises its
// round executor: the order of the calls that memory reuse relies on.  Built and
// run by tests/test_native_executor.py, also under ASan/UBSan and TSan.  Exit
// status 0 when every check passes.
#include <atomic>
#include <chrono>
#include <cstdio>
#include <map>
#include <thread>
#include <vector>

#include "tc_sched.h"

using namespace tc::sched;

static int g_failures = 0;
#define CHECK(cond)                                                                      \
    do {                                                                                 \
        if (!(cond)) {                                                                   \
            std::fprintf(stderr, "%s:%d: check failed: %s\n", __FILE__, __LINE__, #cond); \
            ++g_failures;                                                                \
        }                                                                                \
    } while (0)

// Rounds never finish: the watchdog ends them all.
struct stuck_exec : round_executor {
    std::atomic<bool> dead[2] = {{false}, {false}};
    std::map<job*, int> slot_of;       // worker thread only
    std::atomic<int> done_before_mark{0}, done{0};

    int slot_count() const override { return 2; }
    int launch(int slot, std::vector<job*>& jobs) override {
        for (job* j : jobs) slot_of[j] = slot;
        return kOk;
    }
    void collect(int, std::vector<job*>&) override {}
    void job_done(job* j) override {
        // from here on a caller may release the job's graph
        if (!dead[slot_of.at(j)].load()) ++done_before_mark;
        ++done;
    }
    void release(bool) override {}
    uint64_t held_bytes() const override { return 0; }
    void abandon(int slot) override { dead[slot].store(true); }
    void drain() override {}
};

static void abandoned_slot_marked_before_its_jobs_end() {
    stuck_exec ex;
    sched_limits lim;
    lim.budget = 1 << 20;
    lim.watchdog_ms = 5;
    scheduler S(&ex, lim);
    std::vector<uint64_t> tickets;
    for (int k = 0; k < 2; ++k) {
        uint64_t t = 0;
        CHECK(S.submit(new job(), &t) == kOk);
        tickets.push_back(t);
    }
    for (uint64_t t : tickets) {
        uint64_t counts[16];
        int over = 0, rc = kOk;
        for (int i = 0; i < 20000 && !over; ++i) {
            rc = S.poll(t, counts, &over);
            if (!over) std::this_thread::sleep_for(std::chrono::milliseconds(1));
        }
        CHECK(over && rc == kErrDevice);
    }
    S.stop();
    CHECK(ex.done.load() == 2);
    CHECK(ex.done_before_mark.load() == 0);
}

// thread_start comes first on the thread that makes the other calls.
struct thread_exec : round_executor {
    scheduler* S = nullptr;
    std::atomic<int> starts{0}, out_of_order{0};
    std::thread::id id;
    void here() {
        if (starts.load() != 1 || std::this_thread::get_id() != id) ++out_of_order;
    }
    void thread_start() override {
        id = std::this_thread::get_id();
        ++starts;
    }
    int slot_count() const override { return 1; }
    int launch(int slot, std::vector<job*>&) override {
        here();
        S->round_done(slot);
        return kOk;
    }
    void collect(int, std::vector<job*>&) override { here(); }
    void job_done(job*) override { here(); }
    void release(bool) override { here(); }
    uint64_t held_bytes() const override { return 0; }
    void abandon(int) override {}
    void drain() override { here(); }
};

static void worker_thread_starts_first() {
    thread_exec ex;
    sched_limits lim;
    lim.budget = 1 << 20;
    scheduler S(&ex, lim);
    ex.S = &S;
    uint64_t t = 0, counts[16];
    CHECK(S.submit(new job(), &t) == kOk);
    int over = 0;
    for (int i = 0; i < 20000 && !over; ++i) {
        CHECK(S.poll(t, counts, &over) == kOk);
        if (!over) std::this_thread::sleep_for(std::chrono::milliseconds(1));
    }
    CHECK(over);
    S.stop();
    CHECK(ex.starts.load() == 1);
    CHECK(ex.out_of_order.load() == 0);
}

// Before a round starts, memory kept for reuse shrinks to what the admitted
// jobs and the held bytes leave of the budget.
struct room_exec : round_executor {
    scheduler* S = nullptr;
    std::atomic<uint64_t> held{0};
    uint64_t room = ~0ull;                 // worker thread only
    std::atomic<int> launches{0}, wrong{0};
    int slot_count() const override { return 1; }
    void make_room(uint64_t bytes) override { room = bytes; }
    int launch(int slot, std::vector<job*>& jobs) override {
        uint64_t fp = 0;
        for (job* j : jobs) fp += j->footprint;
        if (room != 1000 - fp - held.load()) ++wrong;
        room = ~0ull;
        ++launches;
        S->round_done(slot);
        return kOk;
    }
    void collect(int, std::vector<job*>&) override {}
    void job_done(job*) override {}
    void release(bool) override {}
    uint64_t held_bytes() const override { return held.load(); }
    void abandon(int) override {}
    void drain() override {}
};

static void kept_memory_makes_room() {
    room_exec ex;
    sched_limits lim;
    lim.budget = 1000;
    scheduler S(&ex, lim);
    ex.S = &S;
    const uint64_t footprints[] = {100, 600, 1}, held[] = {0, 300, 999};
    for (int k = 0; k < 3; ++k) {
        ex.held.store(held[k]);
        job* j = new job();
        j->footprint = footprints[k];
        uint64_t t = 0, counts[16];
        CHECK(S.submit(j, &t) == kOk);
        int over = 0;
        for (int i = 0; i < 20000 && !over; ++i) {
            CHECK(S.poll(t, counts, &over) == kOk);
            if (!over) std::this_thread::sleep_for(std::chrono::milliseconds(1));
        }
        CHECK(over);
    }
    S.stop();
    CHECK(ex.launches.load() == 3);
    CHECK(ex.wrong.load() == 0);
}

int main() {
    kept_memory_makes_room();
    worker_thread_starts_first();
    abandoned_slot_marked_before_its_jobs_end();
    if (g_failures) return 1;
    std::printf("all executor checks passed\n");
    return 0;
}
