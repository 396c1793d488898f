// Which kernel a dense capture takes and over how many workgroups, as the host plans it -- TEST INFRASTRUCTURE ONLY.
//   plan_driver SRC_DTYPE WIDTH REQS ROWS_EACH OUT_DTYPE SUMMARY_MASK TENSORS KEEP STEP EVERY INDEXED
// KEEP: none; unknown (a keep vector of the caller's); or a string of 0 and 1, one per request (dmi_set_keep_mask).
// STEP: 1 if the launch sits in a replayable step.  EVERY: rows of the source to one listed.  Prints the fields that plan_grid() decides.
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <string>
#include <vector>

#include "dmi_ring.h"

using namespace dmi;
using namespace dmi::host;

#define CHECK(cond)                                                                                        \
    do {                                                                                                   \
        if (!(cond)) { fprintf(stderr, "CHECK failed: %s (%s)\n", #cond, dmi_last_error()); exit(3); }      \
    } while (0)

int main(int argc, char **argv)
{
    CHECK(argc == 12);
    auto num = [&](int i) { return (uint32_t)strtoul(argv[i], nullptr, 10); };
    const uint32_t dtype = num(1), width = num(2), n = num(3), each = num(4), nb = num(7);
    const std::string keep = argv[8];
    dmi_ring_config_t cfg;
    memset(&cfg, 0, sizeof cfg);
    cfg.device_ring_bytes = cfg.host_ring_bytes = 1u << 20;
    cfg.max_reqs_per_observe = 4096;
    dmi_ring_t *ring = nullptr;
    hipStream_t stream = nullptr;
    CHECK(dmi_ring_create(&cfg, &ring) == DMI_OK);
    CHECK(hipStreamCreate(&stream) == hipSuccess);

    std::vector<dmi_req_sel_t> reqs;
    for (uint32_t i = 0; i < n; i++) reqs.push_back({i, i * each * num(10), 0u, each, num(10)});
    const uint8_t *mask = nullptr;
    uint8_t callers[1] = {1};
    if (keep == "unknown") {
        mask = callers;
    } else if (keep != "none") {
        CHECK(keep.size() == n);
        std::vector<uint8_t> k;
        for (char c : keep) k.push_back(c == '1');
        CHECK(dmi_set_keep_mask(ring, k.data(), n, stream, &mask) == DMI_OK);
    }
    alignas(16) static uint8_t data[16];            // (nothing is read: only the plan is made)
    dmi_tensor_t t = {data, dtype, {(int64_t)n * each * num(10), (int64_t)width}, {(int64_t)width, 1}};
    static const int32_t index[1] = {0};
    dmi_selection_t sel = {n, reqs.data(), mask, num(11) ? index : nullptr};
    dmi_transform_t xf = {num(5), num(6)};
    Geometry geo;
    CaptureArgs a;
    Plan pl;
    PlanEnv env = plan_env(ring);
    env.cap = env.host_cap = 1ull << 40;
    CHECK(prep_dense(&t, &sel, geo, a) == DMI_OK);
    CHECK(plan_capture(env, 0, &sel, &xf, geo, a, pl, num(9) == 0) == DMI_OK);
    const uint32_t grid = plan_grid(a, nb);
    printf("grid=%u rows_kernel=%u wave_rows=%u read_once=%u decode=%u row_map=%u\n", grid, a.step_per_wave, a.wave_rows,
           a.read_once, pl.decode ? 1u : 0u, pl.row_map ? 1u : 0u);
    CHECK(hipStreamSynchronize(stream) == hipSuccess);
    CHECK(dmi_ring_destroy(ring) == DMI_OK);
    CHECK(hipStreamDestroy(stream) == hipSuccess);
    return 0;
}
