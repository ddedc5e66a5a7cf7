// Host-logic check of batches that are armed again (mock HIP runtime, under
// AddressSanitizer): a captured step holds the number of intact tetrahedra,
// so a run armed with another faulty set must capture its masked steps anew.
#include <cstdio>
#include <cstdlib>
#include <vector>

#include "../../include/hhgr.h"

extern int g_mock_captures, g_mock_launches;
extern double g_mock_res2;
static int fails = 0;
#define CHECK(c, ...)                          \
    do {                                       \
        if (!(c)) {                            \
            std::printf("FAIL: " __VA_ARGS__); \
            std::printf("\n");                 \
            fails++;                           \
        }                                      \
    } while (0)

int main() {
    g_mock_res2 = 1.0;  // every residual norm is 1: no member converges
    hhgr_desc d;
    hhgr_desc_default(&d);
    d.n_sub = 2;
    d.level = 4;
    d.general_geometry = 1;
    std::vector<double> xyz;
    for (int z = 0; z <= 2; z++)
        for (int y = 0; y <= 2; y++)
            for (int x = 0; x <= 2; x++) xyz.insert(xyz.end(), {x / 2.0, y / 2.0 + 0.01 * x, z / 2.0});
    std::vector<hhgr_ctx *> c(2, nullptr);
    std::vector<void *> ws;
    std::vector<double> v;
    for (auto &h : c) {
        size_t bytes = 0;
        CHECK(hhgr_workspace_bytes(&d, &bytes) == HHGR_OK, "workspace");
        ws.push_back(std::aligned_alloc(256, (bytes + 255) / 256 * 256));
        CHECK(hhgr_create(&d, ws.back(), bytes, nullptr, &h) == HHGR_OK, "create: %s", hhgr_last_error());
        CHECK(hhgr_set_geometry(h, xyz.data()) == HHGR_OK, "geometry: %s", hhgr_last_error());
        long long nd = 0;
        hhgr_sizes(h, &nd, nullptr, nullptr);
        v.assign(nd, 1.0);
        CHECK(hhgr_set_rhs(h, v.data(), HHGR_RHS_LOAD) == HHGR_OK, "rhs");
    }
    hhgr_batch *b = nullptr;
    CHECK(hhgr_batch_create(c.data(), 2, nullptr, &b) == HHGR_OK, "batch");
    const int sets[4][2] = {{3, 0}, {3, 17}, {17, 3}, {5, 0}}, count[4] = {1, 2, 2, 1};
    for (int r = 0; r < 4; r++) {
        const int cap0 = g_mock_captures, lau0 = g_mock_launches;
        CHECK(hhgr_batch_arm_dd(b, 0, sets[r], count[r], 1, 2) == HHGR_OK, "arm %d", r);
        CHECK(hhgr_batch_run(b, 1e-10, 4, nullptr) == HHGR_ENOCONV, "run %d: %s", r, hhgr_last_error());
        // the masked step beside the local cycles, and the plain step: two graphs
        CHECK(g_mock_captures - cap0 == 2, "armed run %d captured %d steps", r, g_mock_captures - cap0);
        CHECK(g_mock_launches - lau0 == 4, "armed run %d launched %d steps", r, g_mock_launches - lau0);
    }
    // a run that is not armed replays the plain step
    const int cap0 = g_mock_captures;
    CHECK(hhgr_batch_run(b, 1e-10, 4, nullptr) == HHGR_ENOCONV, "plain run: %s", hhgr_last_error());
    CHECK(g_mock_captures == cap0, "the plain run captured %d steps", g_mock_captures - cap0);
    hhgr_batch_destroy(b);
    for (auto h : c) hhgr_destroy(h);
    for (auto p : ws) std::free(p);
    std::printf("engine_batch_check: %s (%d failures)\n", fails ? "FAILED" : "ok", fails);
    return fails ? 1 : 0;
}
