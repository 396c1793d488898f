// What a flush of a ring without a drain thread may and may not do, one scenario per rule, on the CPU
// stand-in runtime -- TEST INFRASTRUCTURE ONLY.  A gate (a task that waits to be let go) stands for
// work of the caller's that keeps a stream busy, so every scenario has one outcome.  Built and run, one
// scenario per process, by tests/test_flush_rules.py.
#include <hip/hip_runtime.h>

#include <atomic>
#include <chrono>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <string>
#include <thread>
#include <vector>

#include "dmi.h"

#define CHECK(cond)                                                                          \
    do {                                                                                     \
        if (!(cond)) {                                                                       \
            fprintf(stderr, "%s:%d: CHECK failed: %s (last error: %s)\n", __FILE__, __LINE__, #cond, \
                    dmi_last_error());                                                       \
            exit(3);                                                                         \
        }                                                                                    \
    } while (0)

namespace {

constexpr uint32_t kWidth = 512;

struct Bench {
    dmi_ring_t *ring = nullptr;
    hipStream_t stream = nullptr;
    std::vector<uint16_t> data = std::vector<uint16_t>(64 * kWidth, 0x3F80);
    std::atomic<bool> gate_open{true};

    Bench(uint32_t flags, uint32_t timeout_ms, uint64_t dev = 1u << 20, uint64_t host = 1u << 20)
    {
        dmi_ring_config_t cfg;
        memset(&cfg, 0, sizeof cfg);
        cfg.device_ring_bytes = dev;
        cfg.host_ring_bytes = host;
        cfg.flags = flags;
        cfg.max_reqs_per_observe = 128;
        cfg.block_timeout_ms = timeout_ms;
        CHECK(dmi_ring_create(&cfg, &ring) == DMI_OK);
        CHECK(hipStreamCreate(&stream) == hipSuccess);
    }
    ~Bench()
    {
        open_gate();
        CHECK(hipStreamSynchronize(stream) == hipSuccess);
        CHECK(dmi_ring_destroy(ring) == DMI_OK);
        CHECK(hipStreamDestroy(stream) == hipSuccess);
    }
    // everything enqueued from here on waits until open_gate()
    void close_gate()
    {
        gate_open.store(false);
        fake_enqueue(stream, [this] {
            while (!gate_open.load()) std::this_thread::sleep_for(std::chrono::microseconds(20));
        });
    }
    void open_gate() { gate_open.store(true); }
    // one row of `width` elements per record
    dmi_status_t observe(uint32_t n = 1, const uint8_t *keep = nullptr)
    {
        dmi_tensor_t t = {data.data(), DMI_DTYPE_BF16, {64, kWidth}, {kWidth, 1}};
        const dmi_req_sel_t one = {1, 2, 0, 1, 1};
        const dmi_selection_t sel = {1, &one, keep, nullptr};
        const dmi_transform_t raw = {DMI_DTYPE_BF16, 0};
        for (uint32_t i = 0; i < n; i++) {
            const dmi_status_t rc = dmi_observe(ring, 1, &t, &sel, &raw, 0, stream);
            if (rc != DMI_OK) return rc;
        }
        return DMI_OK;
    }
    uint32_t poll()
    {
        dmi_record_view_t v[128];
        uint32_t n = 0;
        CHECK(dmi_poll_host(ring, v, 128, &n) == DMI_OK);
        return n;
    }
    static uint64_t record() { return dmi_record_bytes(1, 1, kWidth, DMI_DTYPE_BF16, 0); }
};

// A flush that gave up leaves its copy under way: a drain that waits says so, and does not say OK
// before the copy is over.
void waiting_drain_after_a_flush_that_gave_up()
{
    Bench b(0, 5);
    b.close_gate();
    CHECK(b.observe() == DMI_OK);
    CHECK(dmi_drain(b.ring, DMI_DRAIN_FLUSH, nullptr) == DMI_ERR_AGAIN);
    CHECK(dmi_drain(b.ring, 0, nullptr) == DMI_ERR_AGAIN);
    CHECK(b.poll() == 0);
    b.open_gate();
    dmi_status_t rc = DMI_ERR_AGAIN;
    for (int i = 0; rc == DMI_ERR_AGAIN && i < 1000; i++) rc = dmi_drain(b.ring, 0, nullptr);
    CHECK(rc == DMI_OK && b.poll() == 1);
}

// A consumer that only polls sees the records of a flush that gave up, once their copy is over.
void polling_alone_sees_a_flush_that_gave_up()
{
    Bench b(0, 5);
    b.close_gate();
    CHECK(b.observe() == DMI_OK);
    CHECK(dmi_drain(b.ring, DMI_DRAIN_FLUSH, nullptr) == DMI_ERR_AGAIN);
    CHECK(b.poll() == 0);
    b.open_gate();
    uint32_t seen = 0;
    for (int i = 0; !seen && i < 4000; i++) {
        std::this_thread::sleep_for(std::chrono::microseconds(500));
        seen = b.poll();
    }
    CHECK(seen == 1);
}

// A thread other than the producer's leaves the producer's stream alone: its copy goes to the drain stream.
void other_threads_flushes_stay_off_the_producers_stream()
{
    Bench b(0, 2000);
    CHECK(b.observe() == DMI_OK);
    std::thread([&] { CHECK(dmi_drain(b.ring, DMI_DRAIN_FLUSH, nullptr) == DMI_OK); }).join();
    CHECK(fake_drain_launches(b.stream) == 0 && b.poll() == 1);
    CHECK(b.observe() == DMI_OK);           // the producer's own: behind the capture
    CHECK(dmi_drain(b.ring, DMI_DRAIN_FLUSH, nullptr) == DMI_OK);
    CHECK(fake_drain_launches(b.stream) == 1 && b.poll() == 1);
}

// Records whose captures have ended are moved at once, whatever the caller has put on the stream behind them:
// a flush does not queue their copy there.
void captured_records_do_not_wait_for_work_behind_them()
{
    Bench b(0, 2000);
    CHECK(b.observe(16) == DMI_OK);         // (the sixteenth puts a probe behind them)
    CHECK(hipStreamSynchronize(b.stream) == hipSuccess);
    b.close_gate();
    CHECK(dmi_drain(b.ring, DMI_DRAIN_FLUSH, nullptr) == DMI_OK);
    CHECK(b.poll() == 16);
}

// The same where the captures end only while the flush waits for them.
void records_with_a_probe_do_not_wait_for_work_behind_it()
{
    Bench b(0, 2000);
    std::atomic<bool> go{false};
    fake_enqueue(b.stream, [&] { while (!go.load()) std::this_thread::sleep_for(std::chrono::microseconds(20)); });
    CHECK(b.observe(16) == DMI_OK);
    b.close_gate();
    std::thread later([&] {
        std::this_thread::sleep_for(std::chrono::milliseconds(20));
        go.store(true);
    });
    CHECK(dmi_drain(b.ring, DMI_DRAIN_FLUSH, nullptr) == DMI_OK);
    later.join();
    CHECK(b.poll() == 16);
}

// A flush that cannot finish still delivers the records in front of the capture it waits for, whichever engine the ring drains with.
void a_flush_that_gives_up_delivers_what_was_captured()
{
    for (const uint32_t flags : {0u, (uint32_t)DMI_DRAIN_COPY_ENGINE, (uint32_t)DMI_DRAIN_KERNEL}) {
        Bench b(flags, 500);
        CHECK(b.observe(16) == DMI_OK);
        CHECK(hipStreamSynchronize(b.stream) == hipSuccess);
        b.close_gate();
        CHECK(b.observe() == DMI_OK);
        CHECK(dmi_drain(b.ring, DMI_DRAIN_FLUSH, nullptr) == DMI_ERR_AGAIN);
        CHECK(b.poll() == 16);
        b.open_gate();
        CHECK(dmi_drain(b.ring, DMI_DRAIN_FLUSH, nullptr) == DMI_OK);
        CHECK(b.poll() == 1);
    }
}

// The same where those captures end only while it waits.
void a_flush_that_gives_up_delivers_what_gets_captured()
{
    Bench b(0, 1000);
    std::atomic<bool> go{false};
    fake_enqueue(b.stream, [&] { while (!go.load()) std::this_thread::sleep_for(std::chrono::microseconds(20)); });
    CHECK(b.observe(16) == DMI_OK);
    b.close_gate();
    CHECK(b.observe() == DMI_OK);
    std::thread later([&] {
        std::this_thread::sleep_for(std::chrono::milliseconds(20));
        go.store(true);
    });
    CHECK(dmi_drain(b.ring, DMI_DRAIN_FLUSH, nullptr) == DMI_ERR_AGAIN);
    later.join();
    CHECK(b.poll() == 16);
    b.open_gate();
    CHECK(dmi_drain(b.ring, DMI_DRAIN_FLUSH, nullptr) == DMI_OK);
    CHECK(b.poll() == 1);
}

// Nor does it keep the room of captured records from a producer that waits for it.
void a_flush_that_gives_up_leaves_room_to_the_producer()
{
    Bench b(0, 500, 24 * Bench::record());
    CHECK(b.observe(16) == DMI_OK);
    CHECK(hipStreamSynchronize(b.stream) == hipSuccess);
    b.close_gate();
    CHECK(b.observe(2) == DMI_OK);
    CHECK(dmi_drain(b.ring, DMI_DRAIN_FLUSH, nullptr) == DMI_ERR_AGAIN);
    CHECK(b.observe(14) == DMI_OK);
}

// A stream of which the runtime will not say whether it is captured: the flush copies on the drain stream, and
// the error it was answered with is not taken for that of the next launch.
void an_unanswered_capture_query_leaves_no_error()
{
    for (const uint32_t flags : {0u, (uint32_t)DMI_DRAIN_KERNEL}) {
        Bench b(flags, 2000);
        CHECK(b.observe() == DMI_OK);
        fake_fail_capture_queries(1);
        uint64_t moved = 0;
        CHECK(dmi_drain(b.ring, DMI_DRAIN_FLUSH, &moved) == DMI_OK);
        CHECK(moved == Bench::record() && fake_drain_launches(b.stream) == 0);
        CHECK(b.observe() == DMI_OK);
        CHECK(dmi_drain(b.ring, DMI_DRAIN_FLUSH, nullptr) == DMI_OK);
        CHECK(b.poll() == 2);
    }
}

// One record of exactly `bytes` (of 64-byte rows; the stand-in's captures read no source).
dmi_status_t observe_bytes(Bench &b, uint64_t bytes)
{
    const uint32_t rows = (uint32_t)((bytes - 128u) / 64u);
    CHECK(dmi_record_bytes(1, rows, 32, DMI_DTYPE_BF16, 0) == bytes);
    dmi_tensor_t t = {b.data.data(), DMI_DTYPE_BF16, {rows, 32}, {32, 1}};
    const dmi_req_sel_t all = {1, 0, 0, rows, 1};
    const dmi_selection_t sel = {1, &all, nullptr, nullptr};
    const dmi_transform_t raw = {DMI_DTYPE_BF16, 0};
    return dmi_observe(b.ring, 1, &t, &sel, &raw, 0, b.stream);
}

// What goes behind the captures, and what does not: how many drain kernels the producer's stream has seen.
void spans_up_to_the_limit_go_behind_the_captures()
{
    constexpr uint64_t limit = 6u << 20;
    Bench b(0, 2000, 64u << 20, 64u << 20);
    CHECK(observe_bytes(b, limit) == DMI_OK && dmi_drain(b.ring, DMI_DRAIN_FLUSH, nullptr) == DMI_OK);
    CHECK(fake_drain_launches(b.stream) == 1 && b.poll() == 1);
    CHECK(observe_bytes(b, limit + 64) == DMI_OK && dmi_drain(b.ring, DMI_DRAIN_FLUSH, nullptr) == DMI_OK);
    CHECK(fake_drain_launches(b.stream) == 1 && b.poll() == 1);
    CHECK(b.observe(7) == DMI_OK && dmi_drain(b.ring, DMI_DRAIN_FLUSH, nullptr) == DMI_OK);
    CHECK(fake_drain_launches(b.stream) == 2 && b.poll() == 7);
    for (int i = 0; i < 40; i++)            // eight captures and a flush in turn: always
        CHECK(b.observe(8) == DMI_OK && dmi_drain(b.ring, DMI_DRAIN_FLUSH, nullptr) == DMI_OK);
    CHECK(fake_drain_launches(b.stream) == 42 && b.poll() == 128);
    CHECK(dmi_drain(b.ring, DMI_DRAIN_FLUSH, nullptr) == DMI_OK && fake_drain_launches(b.stream) == 42);     // nothing to move
}

void other_rings_and_spans_do_not_go_behind_the_captures()
{
    for (const uint32_t flags : {(uint32_t)DMI_DRAIN_COPY_ENGINE, (uint32_t)DMI_BG_THREAD, (uint32_t)(DMI_BG_THREAD | DMI_DRAIN_KERNEL)}) {
        Bench b(flags, 2000);
        CHECK(b.observe() == DMI_OK && dmi_drain(b.ring, DMI_DRAIN_FLUSH, nullptr) == DMI_OK);
        CHECK(fake_drain_launches(b.stream) == 0 && b.poll() == 1);
    }
    {   // a keep vector of the caller's: the size is the device's secret
        Bench b(0, 2000);
        const uint8_t keep = 1;
        CHECK(b.observe(1, &keep) == DMI_OK && dmi_drain(b.ring, DMI_DRAIN_FLUSH, nullptr) == DMI_OK);
        CHECK(fake_drain_launches(b.stream) == 0 && b.poll() == 1);
    }
    {   // best effort, decided on the device: the host runs more launches ahead than it answers for
        Bench b(0, 2000, 4 * Bench::record());
        const dmi_policy_t drop = {DMI_POLICY_DROP_NEWEST, 1, 0};
        CHECK(dmi_set_policy(b.ring, &drop) == DMI_OK);
        b.close_gate();
        CHECK(b.observe(12) == DMI_OK);
        b.open_gate();
        CHECK(dmi_drain(b.ring, DMI_DRAIN_FLUSH, nullptr) == DMI_OK);
        CHECK(fake_drain_launches(b.stream) == 0 && b.poll() == 4);
    }
    {   // a host ring with room for five of six records
        Bench b(0, 2000, 1u << 20, 5 * Bench::record());
        CHECK(b.observe(6) == DMI_OK && dmi_drain(b.ring, DMI_DRAIN_FLUSH, nullptr) == DMI_ERR_AGAIN);
        CHECK(fake_drain_launches(b.stream) == 0 && b.poll() == 5);
    }
    {   // a stream under capture: nothing of the copy may end up in the graph
        Bench b(0, 200);
        CHECK(b.observe() == DMI_OK);
        fake_begin_capture(b.stream);
        (void)dmi_drain(b.ring, DMI_DRAIN_FLUSH, nullptr);
        CHECK(fake_drain_launches(b.stream) == 0);
        fake_graph_launch(fake_end_capture(b.stream), b.stream);
        CHECK(dmi_drain(b.ring, DMI_DRAIN_FLUSH, nullptr) == DMI_OK && b.poll() == 1);
    }
}

// A launch behind enough bytes notes where it finds the head: what is in front of it is copied while the flush still waits for
// captures behind it.
void noted_records_do_not_wait_for_the_captures_behind_them()
{
    Bench b(0, 500, 64u << 20, 64u << 20);
    constexpr uint64_t bytes = 600u << 10;
    for (int i = 0; i < 4; i++) CHECK(observe_bytes(b, bytes) == DMI_OK);
    b.close_gate();
    CHECK(observe_bytes(b, bytes) == DMI_OK);
    CHECK(dmi_drain(b.ring, DMI_DRAIN_FLUSH, nullptr) == DMI_ERR_AGAIN);
    CHECK(b.poll() == 3);                   // (the fourth launch is the last to have started)
    uint64_t room = 0;
    CHECK(dmi_ring_free_bytes(b.ring, &room) == DMI_OK && room == (64u << 20) - 2 * bytes);
    b.open_gate();
    CHECK(dmi_drain(b.ring, DMI_DRAIN_FLUSH, nullptr) == DMI_OK);
    CHECK(b.poll() == 2 && fake_drain_launches(b.stream) == 0);
    dmi_stats_t s;
    CHECK(dmi_get_stats(b.ring, &s) == DMI_OK && s.captured_records == 5 && s.drained_bytes == 5 * bytes);
}

// Few bytes that have been noted go with the rest, behind the captures.
void a_small_noted_part_goes_with_the_rest()
{
    Bench b(0, 2000, 64u << 20, 64u << 20);
    for (int i = 0; i < 2; i++) CHECK(observe_bytes(b, 600u << 10) == DMI_OK);
    CHECK(dmi_drain(b.ring, DMI_DRAIN_FLUSH, nullptr) == DMI_OK);
    CHECK(fake_drain_launches(b.stream) == 1 && b.poll() == 2);
}

// A batch of which capture and copy both take long goes by two launches: what the first has captured, which the second's note says,
// is copied while the flush waits.  Statistics of eight tensors of 134 MB, 6.3 MB in all: at 5.5 TB/s and 57 GB/s the capture is
// 0.64 of both together, so six of the eight come first.  Two of them alone are not worth a second launch.
void a_batch_in_two_launches()
{
    constexpr uint32_t rows = 65536, width = 1024;
    Bench b(0, 500, 64u << 20, 64u << 20);
    const dmi_tensor_t t = {b.data.data(), DMI_DTYPE_BF16, {rows, width}, {width, 1}};
    const dmi_req_sel_t all = {1, 0, 0, rows, 1};
    const dmi_selection_t sel = {1, &all, nullptr, nullptr};
    const dmi_transform_t sums = {DMI_DTYPE_NONE, 7};
    const uint32_t points[8] = {0, 1, 2, 3, 4, 5, 6, 7};
    const void *data[8];
    for (const void *&d : data) d = b.data.data();
    for (const uint32_t n : {8u, 2u}) {
        CHECK(dmi_observe_batch(b.ring, n, points, data, &t, &sel, &sums, 0, b.stream, nullptr) == DMI_OK);
        if (n == 2u) CHECK(hipStreamSynchronize(b.stream) == hipSuccess);
        b.close_gate();
        CHECK(dmi_drain(b.ring, DMI_DRAIN_FLUSH, nullptr) == DMI_ERR_AGAIN);
        CHECK(b.poll() == (n == 8u ? 6u : 0u));
        b.open_gate();
        CHECK(dmi_drain(b.ring, DMI_DRAIN_FLUSH, nullptr) == DMI_OK);
        CHECK(b.poll() == 2u);
    }
}

// An observe that finds all commit slots taken waits for the oldest launches, also where what tells of those is the copy of a
// flush that gave up, and however long that takes: under best effort no record goes by uncounted.
void commit_slots_wait_for_a_flush_that_gave_up()
{
    Bench b(0, 20, 4 * Bench::record(), 8 * Bench::record());
    const dmi_policy_t drop = {DMI_POLICY_DROP_NEWEST, 1, 0};
    CHECK(dmi_set_policy(b.ring, &drop) == DMI_OK);
    b.close_gate();
    CHECK(b.observe() == DMI_OK);
    CHECK(dmi_drain(b.ring, DMI_DRAIN_FLUSH, nullptr) == DMI_ERR_AGAIN);
    std::thread later([&] {
        std::this_thread::sleep_for(std::chrono::milliseconds(300));
        b.open_gate();
    });
    CHECK(b.observe(1200) == DMI_OK);
    later.join();
    CHECK(fake_drain_launches(b.stream) == 1);
    CHECK(hipStreamSynchronize(b.stream) == hipSuccess);
    CHECK(dmi_drain(b.ring, DMI_DRAIN_FLUSH, nullptr) == DMI_OK);
    dmi_stats_t s;
    CHECK(dmi_get_stats(b.ring, &s) == DMI_OK && s.captured_records + s.dropped_records == 1201);
}

// A GPU that fails while a flush waits for its copy behind the captures: the flush says so, and does so at once; neither it nor
// another thread's drain behind it asks to be called again.
void a_failing_gpu_is_not_a_flush_that_takes_long()
{
    Bench b(0, 10000);
    b.close_gate();
    CHECK(b.observe() == DMI_OK);
    std::thread later([] {
        std::this_thread::sleep_for(std::chrono::milliseconds(30));
        fake_fail_device(true);
    });
    const auto t0 = std::chrono::steady_clock::now();
    CHECK(dmi_drain(b.ring, DMI_DRAIN_FLUSH, nullptr) == DMI_ERR_HIP);
    CHECK(fake_drain_launches(b.stream) == 1);
    std::thread([&] { CHECK(dmi_drain(b.ring, 0, nullptr) == DMI_ERR_HIP); }).join();
    CHECK(std::chrono::steady_clock::now() - t0 < std::chrono::seconds(5));
    later.join();
    fake_fail_device(false);
}

// A flush whose captures have ended and that has started its last copy does not give up on it, however long that takes, whichever
// engine moves it (block_timeout_ms is for what the host ring, the observes or the caller's work hold up); a GPU that fails is told of.
void a_flush_does_not_give_up_on_its_own_copy()
{
    for (const bool fails : {false, true})
        for (const uint32_t flags : {0u, (uint32_t)DMI_DRAIN_COPY_ENGINE, (uint32_t)DMI_DRAIN_KERNEL}) {
            Bench b(flags, fails ? 10000 : 1);
            CHECK(b.observe(16) == DMI_OK);         // (the sixteenth puts a probe behind them)
            CHECK(hipStreamSynchronize(b.stream) == hipSuccess);
            fake_hold_copies(true);
            std::thread later([&] {
                std::this_thread::sleep_for(std::chrono::milliseconds(60));
                if (fails) fake_fail_device(true);
                else fake_hold_copies(false);
            });
            const auto t0 = std::chrono::steady_clock::now();
            CHECK(dmi_drain(b.ring, DMI_DRAIN_FLUSH, nullptr) == (fails ? DMI_ERR_HIP : DMI_OK));
            CHECK(std::chrono::steady_clock::now() - t0 < std::chrono::seconds(5));
            later.join();
            if (!fails) CHECK(b.poll() == 16);
            fake_fail_device(false);
            fake_hold_copies(false);
        }
}

// What a flush still has to move when the captures are over goes by a drain kernel only if the producer's stream has nothing behind
// them: a kernel would contend with that for compute units, which the copy engine does not need.
void the_last_copy_leaves_the_compute_units_to_work_behind_the_captures()
{
    for (const bool work : {false, true}) {
        Bench b(0, 2000);
        std::atomic<bool> go{false};
        fake_enqueue(b.stream, [&] { while (!go.load()) std::this_thread::sleep_for(std::chrono::microseconds(20)); });
        CHECK(b.observe(16) == DMI_OK);         // (the sixteenth puts a probe behind them)
        if (work) b.close_gate();
        std::thread later([&] {
            std::this_thread::sleep_for(std::chrono::milliseconds(20));
            go.store(true);
        });
        const unsigned before = fake_all_drain_launches();
        CHECK(dmi_drain(b.ring, DMI_DRAIN_FLUSH, nullptr) == DMI_OK);
        later.join();
        CHECK(b.poll() == 16 && fake_all_drain_launches() - before == (work ? 0u : 1u));
    }
}

// Nor while the runtime will not say whether that stream is captured, which leaves no error, or while it is: it is not asked then.
void a_captured_stream_is_not_asked_for_its_state()
{
    for (const bool unanswered : {false, true}) {
        Bench b(0, 2000);
        CHECK(b.observe(16) == DMI_OK);
        CHECK(hipStreamSynchronize(b.stream) == hipSuccess);
        const unsigned before = fake_all_drain_launches();
        if (unanswered) fake_fail_capture_queries(1);
        else fake_begin_capture(b.stream);
        CHECK(dmi_drain(b.ring, DMI_DRAIN_FLUSH, nullptr) == DMI_OK);
        if (!unanswered) CHECK(fake_end_capture(b.stream).empty());
        CHECK(b.poll() == 16 && fake_all_drain_launches() == before && fake_queries_under_capture() == 0);
        CHECK(b.observe() == DMI_OK);
    }
}

// Notes are for a flush by the producer of a ring that may choose its engine: it knows how much is still to come and copies what is
// worth a copy.  All other drains move what an event has confirmed, and so does the flush of a ring that was asked for one engine by name.
void other_drains_do_not_copy_by_notes()
{
    constexpr uint64_t bytes = 600u << 10;
    auto noted = [](Bench &b) {                 // three records of which only notes tell, and two behind them
        for (int i = 0; i < 4; i++) CHECK(observe_bytes(b, bytes) == DMI_OK);
        CHECK(hipStreamSynchronize(b.stream) == hipSuccess);
        b.close_gate();
        CHECK(observe_bytes(b, bytes) == DMI_OK);
    };
    auto rest = [](Bench &b) {
        b.open_gate();
        CHECK(dmi_drain(b.ring, DMI_DRAIN_FLUSH, nullptr) == DMI_OK);
        CHECK(b.poll() == 5);
    };
    {
        Bench b(0, 200, 64u << 20, 64u << 20);
        noted(b);
        uint64_t moved = 1;
        for (const uint32_t how : {(uint32_t)DMI_DRAIN_NONBLOCK, 0u})
            CHECK(dmi_drain(b.ring, how, &moved) == DMI_OK && moved == 0);
        std::thread([&] { CHECK(dmi_drain(b.ring, DMI_DRAIN_FLUSH, &moved) == DMI_ERR_AGAIN && moved == 0); }).join();
        dmi_stats_t s;
        CHECK(dmi_get_stats(b.ring, &s) == DMI_OK && s.drained_bytes == s.captured_bytes);
        rest(b);
    }
    for (const uint32_t flags : {(uint32_t)DMI_DRAIN_COPY_ENGINE, (uint32_t)DMI_DRAIN_KERNEL}) {
        Bench b(flags, 200, 64u << 20, 64u << 20);
        noted(b);
        CHECK(dmi_drain(b.ring, DMI_DRAIN_FLUSH, nullptr) == DMI_ERR_AGAIN && b.poll() == 0);
        rest(b);
    }
    {   // a drain behind a flush that has copied by notes and given up: nothing of that again, and then the rest
        Bench b(0, 200, 64u << 20, 64u << 20);
        noted(b);
        uint64_t moved = 1;
        CHECK(dmi_drain(b.ring, DMI_DRAIN_FLUSH, nullptr) == DMI_ERR_AGAIN && b.poll() == 3);
        CHECK(dmi_drain(b.ring, 0, &moved) == DMI_OK && moved == 0 && b.poll() == 0);
        b.open_gate();
        CHECK(hipStreamSynchronize(b.stream) == hipSuccess);
        CHECK(dmi_drain(b.ring, 0, &moved) == DMI_OK && moved == 2 * bytes && b.poll() == 2);
    }
}

// The captures of a replayed step belong to the drain from dmi_step_end on: a flush while the step is open neither delivers what their
// notes already say nor counts it.
void a_flush_leaves_an_open_step_alone()
{
    constexpr uint64_t bytes = 600u << 10;
    Bench b(0, 2000, 64u << 20, 64u << 20);
    dmi_step_t *step = nullptr;
    CHECK(dmi_step_create(b.ring, 8, &step) == DMI_OK && dmi_step_capture_begin(step) == DMI_OK);
    fake_begin_capture(b.stream);
    const uint32_t rows = (uint32_t)((bytes - 128u) / 64u);
    dmi_tensor_t t = {b.data.data(), DMI_DTYPE_BF16, {rows, 32}, {32, 1}};
    const dmi_req_sel_t all = {1, 0, 0, rows, 1};
    const dmi_selection_t sel = {1, &all, nullptr, nullptr};
    const dmi_transform_t raw = {DMI_DTYPE_BF16, 0};
    for (uint32_t i = 0; i < 6; i++) CHECK(dmi_step_observe(step, i, &t, &sel, &raw, b.stream, nullptr) == DMI_OK);
    const std::vector<FakeTask> graph = fake_end_capture(b.stream);
    CHECK(dmi_step_seal(step) == DMI_OK);
    for (uint64_t id = 0; id < 3; id++) {
        CHECK(b.observe() == DMI_OK);           // (what is in front of the step is delivered)
        CHECK(dmi_step_begin(step, id, b.stream) == DMI_OK);
        fake_graph_launch(graph, b.stream);
        CHECK(hipStreamSynchronize(b.stream) == hipSuccess);
        uint64_t moved = 0;
        CHECK(dmi_drain(b.ring, DMI_DRAIN_FLUSH, &moved) == DMI_OK && moved == Bench::record() && b.poll() == 1);
        CHECK(dmi_drain(b.ring, DMI_DRAIN_FLUSH, &moved) == DMI_OK && moved == 0 && b.poll() == 0);
        CHECK(dmi_step_end(step, b.stream) == DMI_OK);
        CHECK(dmi_drain(b.ring, DMI_DRAIN_FLUSH, &moved) == DMI_OK && moved == 6 * bytes && b.poll() == 6);
        dmi_stats_t s;
        CHECK(dmi_get_stats(b.ring, &s) == DMI_OK && s.drained_bytes == s.captured_bytes);
        CHECK(dmi_release_host(b.ring, 7 * (id + 1)) == DMI_OK);
    }
    CHECK(dmi_step_destroy(step) == DMI_OK);
}

// What the captures of a step have noted that was destroyed before its dmi_step_end the counters never hear of: the drain stays behind
// the head that the host counts on, and the producer has the room that this says.
void a_step_destroyed_while_open_is_not_drained_by_its_notes()
{
    constexpr uint64_t bytes = 600u << 10;
    Bench b(0, 50, 64u << 20, 64u << 20);
    dmi_step_t *step = nullptr;
    CHECK(dmi_step_create(b.ring, 8, &step) == DMI_OK && dmi_step_capture_begin(step) == DMI_OK);
    fake_begin_capture(b.stream);
    const uint32_t rows = (uint32_t)((bytes - 128u) / 64u);
    dmi_tensor_t t = {b.data.data(), DMI_DTYPE_BF16, {rows, 32}, {32, 1}};
    const dmi_req_sel_t all = {1, 0, 0, rows, 1};
    const dmi_selection_t sel = {1, &all, nullptr, nullptr};
    const dmi_transform_t raw = {DMI_DTYPE_BF16, 0};
    for (uint32_t i = 0; i < 6; i++) CHECK(dmi_step_observe(step, i, &t, &sel, &raw, b.stream, nullptr) == DMI_OK);
    const std::vector<FakeTask> graph = fake_end_capture(b.stream);
    CHECK(dmi_step_seal(step) == DMI_OK);
    CHECK(dmi_step_begin(step, 0, b.stream) == DMI_OK);
    fake_graph_launch(graph, b.stream);
    CHECK(hipStreamSynchronize(b.stream) == hipSuccess);
    CHECK(dmi_step_destroy(step) == DMI_OK);
    for (int i = 0; i < 4; i++) {
        uint64_t moved = 0, room = 0;
        CHECK(dmi_drain(b.ring, DMI_DRAIN_FLUSH, &moved) == DMI_OK && moved == (i ? Bench::record() : 0u));
        CHECK(dmi_ring_free_bytes(b.ring, &room) == DMI_OK && room == 64u << 20);
        CHECK(b.observe() == DMI_OK);
    }
}

// The second launch is for a flush that copies by notes: not where the ring's last drain was none, or one by another thread.
void a_batch_goes_by_two_launches_only_for_flushes_that_copy_by_notes()
{
    constexpr uint32_t rows = 65536, width = 1024;
    const dmi_req_sel_t all = {1, 0, 0, rows, 1};
    const dmi_selection_t sel = {1, &all, nullptr, nullptr};
    const dmi_transform_t sums = {DMI_DTYPE_NONE, 7};
    const uint32_t points[8] = {0, 1, 2, 3, 4, 5, 6, 7};
    auto launches = [&](Bench &b) {
        const dmi_tensor_t t = {b.data.data(), DMI_DTYPE_BF16, {rows, width}, {width, 1}};
        const void *data[8];
        for (const void *&d : data) d = b.data.data();
        const size_t before = fake_capture_launches().size();
        CHECK(dmi_observe_batch(b.ring, 8, points, data, &t, &sel, &sums, 0, b.stream, nullptr) == DMI_OK);
        return fake_capture_launches().size() - before;
    };
    Bench b(0, 2000, 64u << 20, 64u << 20);
    CHECK(launches(b) == 2);
    std::thread([&] { CHECK(dmi_drain(b.ring, DMI_DRAIN_FLUSH, nullptr) == DMI_OK); }).join();
    CHECK(launches(b) == 1);
    CHECK(dmi_drain(b.ring, DMI_DRAIN_FLUSH, nullptr) == DMI_OK);
    CHECK(launches(b) == 2);
    CHECK(dmi_drain(b.ring, DMI_DRAIN_NONBLOCK, nullptr) == DMI_OK);
    CHECK(launches(b) == 1);
    CHECK(dmi_drain(b.ring, DMI_DRAIN_FLUSH, nullptr) == DMI_OK && b.poll() == 32);
    for (const uint32_t flags : {(uint32_t)DMI_DRAIN_COPY_ENGINE, (uint32_t)DMI_DRAIN_KERNEL, (uint32_t)DMI_BG_THREAD}) {
        Bench other(flags, 2000, 64u << 20, 64u << 20);
        for (int i = 0; i < 2; i++)
            CHECK(launches(other) == 1 && dmi_drain(other.ring, DMI_DRAIN_FLUSH, nullptr) == DMI_OK);
    }
}

// The batches of tests/test_gpu_batch_in_two.py do go by two launches: how many of their tensors the first captures.
void where_the_batches_of_the_gpu_test_are_cut()
{
    struct Shape { uint32_t n, n_reqs, each, width, dtype, sums, paged, first; };
    const Shape shapes[] = {{4, 32, 2048, 1024, DMI_DTYPE_FP32, 7, 0, 3},
                            {4, 65, 3001, 128, DMI_DTYPE_BF16, 7, 0, 1},
                            {4, 70, 930, 1024, DMI_DTYPE_FP32, 7, 0, 3},
                            {8, 20, 4001, 256, DMI_DTYPE_BF16, 5, 1, 4}};
    for (const Shape &q : shapes) {
        Bench b(0, 500, 64u << 20, 64u << 20);
        std::vector<dmi_req_sel_t> reqs(q.n_reqs);
        for (uint32_t i = 0; i < q.n_reqs; i++) reqs[i] = {70 + i, q.paged ? i : i * q.each, 0, q.each, 1};
        const dmi_selection_t sel = {q.n_reqs, reqs.data(), nullptr, nullptr};
        const dmi_transform_t sums = {DMI_DTYPE_NONE, q.sums};
        const uint32_t points[8] = {0, 1, 2, 3, 4, 5, 6, 7};
        const int32_t table = 0;
        const void *data[8];
        for (const void *&d : data) d = b.data.data();
        const size_t before = fake_capture_launches().size();
        if (q.paged) {
            dmi_paged_kv_t kv;
            memset(&kv, 0, sizeof kv);
            kv.dtype = q.dtype;
            kv.n_blocks = q.n_reqs * 256; kv.block_size = 16; kv.n_heads = 4; kv.head_dim = 128;
            kv.block_stride = 16 * 4 * 128; kv.slot_stride = 4 * 128; kv.head_stride = 128;
            kv.block_table_dev = &table; kv.block_table_stride = 256; kv.n_seqs = q.n_reqs;
            kv.n_heads_sel = 2; kv.heads_sel[0] = 1; kv.heads_sel[1] = 2;
            kv.base = data[0];
            CHECK(dmi_observe_paged_batch(b.ring, q.n, points, data, &kv, &sel, &sums, 0, b.stream, nullptr) == DMI_OK);
        } else {
            const dmi_tensor_t t = {data[0], q.dtype, {q.n_reqs * q.each, q.width}, {q.width, 1}};
            CHECK(dmi_observe_batch(b.ring, q.n, points, data, &t, &sel, &sums, 0, b.stream, nullptr) == DMI_OK);
        }
        const std::vector<unsigned> launches = fake_capture_launches();
        CHECK(launches.size() - before == 2 && launches[before] == q.first && launches[before + 1] == q.n - q.first);
    }
}

// A ring that was asked for one engine by name leaves no notes, and the rules that go by them do not keep its flush from copying behind
// the captures.
void a_ring_that_drains_by_kernel_copies_behind_the_captures()
{
    Bench b(DMI_DRAIN_KERNEL, 2000, 64u << 20, 64u << 20);
    for (unsigned k = 1; k <= 3; k++) {
        for (int i = 0; i < 8; i++) CHECK(observe_bytes(b, 600u << 10) == DMI_OK);
        CHECK(dmi_drain(b.ring, DMI_DRAIN_FLUSH, nullptr) == DMI_OK);
        CHECK(fake_drain_launches(b.stream) == k && b.poll() == 8);
    }
}

// A span that goes in several copies (of at most 64 MiB) goes by the copy engine to its end, also where what is left for the last of
// them is little.
void the_rest_of_a_long_copy_stays_with_its_engine()
{
    Bench b(0, 2000, 72u << 20, 72u << 20);
    CHECK(observe_bytes(b, 66ull << 20) == DMI_OK);
    CHECK(dmi_drain(b.ring, DMI_DRAIN_FLUSH, nullptr) == DMI_OK && b.poll() == 1);
    dmi_stats_t s;
    CHECK(dmi_get_stats(b.ring, &s) == DMI_OK && s.drain_batches == 2);
    CHECK(fake_all_drain_launches() == 0);
}

struct Scenario {
    const char *name;
    void (*run)();
};
const Scenario kScenarios[] = {
    {"the_rest_of_a_long_copy_stays_with_its_engine", the_rest_of_a_long_copy_stays_with_its_engine},
    {"a_ring_that_drains_by_kernel_copies_behind_the_captures", a_ring_that_drains_by_kernel_copies_behind_the_captures},
    {"where_the_batches_of_the_gpu_test_are_cut", where_the_batches_of_the_gpu_test_are_cut},
    {"a_batch_goes_by_two_launches_only_for_flushes_that_copy_by_notes",
     a_batch_goes_by_two_launches_only_for_flushes_that_copy_by_notes},
    {"a_step_destroyed_while_open_is_not_drained_by_its_notes", a_step_destroyed_while_open_is_not_drained_by_its_notes},
    {"a_flush_leaves_an_open_step_alone", a_flush_leaves_an_open_step_alone},
    {"other_drains_do_not_copy_by_notes", other_drains_do_not_copy_by_notes},
    {"the_last_copy_leaves_the_compute_units_to_work_behind_the_captures",
     the_last_copy_leaves_the_compute_units_to_work_behind_the_captures},
    {"a_captured_stream_is_not_asked_for_its_state", a_captured_stream_is_not_asked_for_its_state},
    {"a_flush_does_not_give_up_on_its_own_copy", a_flush_does_not_give_up_on_its_own_copy},
    {"commit_slots_wait_for_a_flush_that_gave_up", commit_slots_wait_for_a_flush_that_gave_up},
    {"a_failing_gpu_is_not_a_flush_that_takes_long", a_failing_gpu_is_not_a_flush_that_takes_long},
    {"a_batch_in_two_launches", a_batch_in_two_launches},
    {"noted_records_do_not_wait_for_the_captures_behind_them", noted_records_do_not_wait_for_the_captures_behind_them},
    {"a_small_noted_part_goes_with_the_rest", a_small_noted_part_goes_with_the_rest},
    {"waiting_drain_after_a_flush_that_gave_up", waiting_drain_after_a_flush_that_gave_up},
    {"polling_alone_sees_a_flush_that_gave_up", polling_alone_sees_a_flush_that_gave_up},
    {"captured_records_do_not_wait_for_work_behind_them", captured_records_do_not_wait_for_work_behind_them},
    {"records_with_a_probe_do_not_wait_for_work_behind_it", records_with_a_probe_do_not_wait_for_work_behind_it},
    {"a_flush_that_gives_up_delivers_what_was_captured", a_flush_that_gives_up_delivers_what_was_captured},
    {"a_flush_that_gives_up_delivers_what_gets_captured", a_flush_that_gives_up_delivers_what_gets_captured},
    {"a_flush_that_gives_up_leaves_room_to_the_producer", a_flush_that_gives_up_leaves_room_to_the_producer},
    {"an_unanswered_capture_query_leaves_no_error", an_unanswered_capture_query_leaves_no_error},
    {"spans_up_to_the_limit_go_behind_the_captures", spans_up_to_the_limit_go_behind_the_captures},
    {"other_rings_and_spans_do_not_go_behind_the_captures", other_rings_and_spans_do_not_go_behind_the_captures},
    {"other_threads_flushes_stay_off_the_producers_stream", other_threads_flushes_stay_off_the_producers_stream},
};

}  // namespace

int main(int argc, char **argv)
{
    const std::string want = argc > 1 ? argv[1] : "";
    for (const Scenario &s : kScenarios)
        if (want == s.name) {
            s.run();
            fprintf(stderr, "passed\n");
            return 0;
        }
    fprintf(stderr, "no scenario '%s'\n", want.c_str());
    return 2;
}
