// A ring without a drain thread, flushed from a thread of its own and now and then by the producer while it
// observes and a consumer polls, on the CPU stand-in runtime -- TEST INFRASTRUCTURE ONLY.  The producer's
// small flushes move their bytes on its stream, all others on the drain stream; waiting and non-blocking
// drains come in between.  Built with -fsanitize=thread or
// -fsanitize=address by tests/test_flush_behind_captures.py.
#include <hip/hip_runtime.h>

#include <atomic>
#include <chrono>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <thread>
#include <utility>
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

static void scenario(const char *name, uint32_t policy, uint32_t flags, uint64_t dev_bytes, uint64_t host_bytes,
                     uint32_t timeout_ms, int n_iter)
{
    fprintf(stderr, "scenario %s\n", name);
    dmi_ring_config_t cfg;
    memset(&cfg, 0, sizeof cfg);
    cfg.device_ring_bytes = dev_bytes;
    cfg.host_ring_bytes = host_bytes;
    cfg.flags = flags;
    cfg.max_reqs_per_observe = 64;
    cfg.block_timeout_ms = timeout_ms;
    dmi_ring_t *ring = nullptr;
    CHECK(dmi_ring_create(&cfg, &ring) == DMI_OK);
    dmi_policy_t pol = {policy, 1, 0};
    CHECK(dmi_set_policy(ring, &pol) == DMI_OK);
    hipStream_t stream, second;         // the producer changes over from one to the other now and then
    CHECK(hipStreamCreate(&stream) == hipSuccess && hipStreamCreate(&second) == hipSuccess);
    std::vector<uint16_t> data(64 * 512, 0x3F80);
    dmi_tensor_t t = {data.data(), DMI_DTYPE_BF16, {64, 512}, {512, 1}};
    std::vector<dmi_req_sel_t> one(16);
    for (uint32_t i = 0; i < 16; i++) one[i] = {100 + i, i, 0, 1, 1};
    const dmi_selection_t sel = {16, one.data(), nullptr, nullptr};
    const dmi_transform_t raw = {DMI_DTYPE_BF16, 0};

    std::atomic<bool> producer_done{false}, stop{false};
    std::atomic<uint64_t> seen{0}, seen_bytes{0};
    std::thread flusher([&] {
        for (unsigned k = 0; !producer_done.load(); k++) {
            uint64_t moved = 0;
            const uint32_t how = k % 3 == 0 ? DMI_DRAIN_NONBLOCK : k % 3 == 1 ? 0u : DMI_DRAIN_FLUSH;
            const dmi_status_t rc = dmi_drain(ring, how, &moved);
            CHECK(rc == DMI_OK || rc == DMI_ERR_AGAIN);
            if (k % 4 == 0) std::this_thread::sleep_for(std::chrono::microseconds(150));
        }
    });
    std::thread consumer([&] {
        std::vector<dmi_record_view_t> v(64);
        uint64_t last = UINT64_MAX;
        while (!stop.load()) {
            uint32_t n = 0;
            CHECK(dmi_poll_host(ring, v.data(), 64, &n) == DMI_OK);
            for (uint32_t i = 0; i < n; i++) {
                // the executor fills a record with a byte derived from its sequence number
                const uint8_t want = (uint8_t)(0x40u + (v[i].seq & 0x3Fu));
                const uint8_t *end = v[i].n1 ? static_cast<const uint8_t *>(v[i].p1) + v[i].n1 - 1
                                             : static_cast<const uint8_t *>(v[i].p0) + v[i].n0 - 1;
                CHECK(*end == want && (last == UINT64_MAX || v[i].seq > last));
                last = v[i].seq;
                seen_bytes += v[i].n0 + v[i].n1;
                seen++;
            }
            if (n) CHECK(dmi_release_host(ring, v[n - 1].seq) == DMI_OK);
            else std::this_thread::sleep_for(std::chrono::microseconds(30));
        }
    });
    for (int it = 0; it < n_iter; it++) {
        dmi_status_t rc = DMI_ERR_AGAIN;
        for (int tries = 0; rc == DMI_ERR_AGAIN && tries < 1000000; tries++)
            rc = dmi_observe(ring, 1, &t, &sel, &raw, (uint64_t)it, stream);
        CHECK(rc == DMI_OK);
        if (it % 7 == 3) {
            rc = dmi_drain(ring, DMI_DRAIN_FLUSH, nullptr);
            CHECK(rc == DMI_OK || rc == DMI_ERR_AGAIN);
        }
        if (it % 5 == 0) std::this_thread::sleep_for(std::chrono::microseconds(100));
        if (it % 23 == 22) {            // (the stand-in has no waits between streams: the captures so far have run)
            std::atomic<bool> reached{false};
            fake_enqueue(stream, [&] { reached.store(true); });
            while (!reached.load()) std::this_thread::yield();
            std::swap(stream, second);
        }
    }
    producer_done.store(true);
    flusher.join();
    dmi_status_t rc = DMI_ERR_AGAIN;
    for (int i = 0; rc == DMI_ERR_AGAIN && i < 100000; i++) rc = dmi_drain(ring, DMI_DRAIN_FLUSH, nullptr);
    CHECK(rc == DMI_OK);
    dmi_stats_t s;
    CHECK(dmi_get_stats(ring, &s) == DMI_OK);
    CHECK(s.captured_records + s.dropped_records == (uint64_t)n_iter && s.drained_bytes == s.captured_bytes);
    CHECK(s.dev_ring_high_water <= dev_bytes && s.host_ring_high_water <= host_bytes);
    for (int i = 0; seen.load() < s.captured_records && i < 100000; i++)
        std::this_thread::sleep_for(std::chrono::microseconds(100));
    CHECK(seen.load() == s.captured_records && seen_bytes.load() == s.captured_bytes);
    stop.store(true);
    consumer.join();
    CHECK(hipStreamSynchronize(stream) == hipSuccess && hipStreamSynchronize(second) == hipSuccess);
    CHECK(dmi_ring_destroy(ring) == DMI_OK);
    CHECK(hipStreamDestroy(stream) == hipSuccess && hipStreamDestroy(second) == hipSuccess);
}

// Sixteen observes have put their probe behind them; a flush while their stream is being captured adds
// nothing to the capture and delivers them all the same.
static void scenario_capture()
{
    fprintf(stderr, "scenario flush while the stream is captured\n");
    dmi_ring_config_t cfg;
    memset(&cfg, 0, sizeof cfg);
    cfg.device_ring_bytes = cfg.host_ring_bytes = 1u << 20;
    dmi_ring_t *ring = nullptr;
    CHECK(dmi_ring_create(&cfg, &ring) == DMI_OK);
    hipStream_t stream;
    CHECK(hipStreamCreate(&stream) == hipSuccess);
    std::vector<uint16_t> data(64 * 512, 0x3F80);
    dmi_tensor_t t = {data.data(), DMI_DTYPE_BF16, {64, 512}, {512, 1}};
    const dmi_req_sel_t one = {1, 2, 0, 1, 1};
    const dmi_selection_t sel = {1, &one, nullptr, nullptr};
    const dmi_transform_t raw = {DMI_DTYPE_BF16, 0};
    for (int i = 0; i < 16; i++) CHECK(dmi_observe(ring, 1, &t, &sel, &raw, 0, stream) == DMI_OK);
    fake_begin_capture(stream);
    uint64_t moved = 0;
    CHECK(dmi_drain(ring, DMI_DRAIN_FLUSH, &moved) == DMI_OK);
    CHECK(fake_end_capture(stream).empty());
    CHECK(moved == 16 * dmi_record_bytes(1, 1, 512, DMI_DTYPE_BF16, 0));
    dmi_record_view_t v[32];
    uint32_t n = 0;
    CHECK(dmi_poll_host(ring, v, 32, &n) == DMI_OK && n == 16);
    CHECK(dmi_ring_destroy(ring) == DMI_OK);
    CHECK(hipStreamDestroy(stream) == hipSuccess);
}

int main(int argc, char **argv)
{
    const int n = argc > 1 ? atoi(argv[1]) : 500;
    fake_set_jitter_us(30);
    const uint64_t rb = dmi_record_bytes(16, 16, 512, DMI_DTYPE_BF16, 0);
    scenario("block", DMI_POLICY_BLOCK, 0, 1u << 20, 2u << 20, 2000, n);
    scenario("block, small rings that wrap", DMI_POLICY_BLOCK, 0, 3 * rb + 640, 4 * rb + 1280, 2000, n);
    scenario("block, flushes that give up waiting", DMI_POLICY_BLOCK, 0, 1u << 20, 1u << 20, 1, n);
    scenario("drop-newest", DMI_POLICY_DROP_NEWEST, 0, 5 * rb, 6 * rb, 2000, n);
    scenario("block, copy engine by name", DMI_POLICY_BLOCK, DMI_DRAIN_COPY_ENGINE, 1u << 20, 2u << 20, 2000, n);
    scenario_capture();
    fprintf(stderr, "all scenarios passed\n");
    return 0;
}
