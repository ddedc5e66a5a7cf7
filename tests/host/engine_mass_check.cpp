// hhgr_mass_apply with separate, equal and overlapping vectors (mock HIP
// runtime, under AddressSanitizer).  The mass launch is replaced by an
// operation that reads far-away entries, as the stencil does, so an input that
// the launch overwrites shows in the result.
#include <cstdio>
#include <cstdlib>
#include <vector>

#include "../../include/hhgr.h"
#include "hip/hip_runtime.h"

static int fails = 0;
static long long n = 0;

// (linked in place of hhgr::launch_mass_grid)
extern "C" void __wrap__ZN4hhgr16launch_mass_gridEP11mock_streamidPKdPd(hipStream_t, int, double, const double *x,
                                                                       double *y) {
    for (long long q = 0; q < n; q++) y[q] = x[q] + 3.0 * x[n - 1 - q];
}

int main() {
    hhgr_desc d;
    hhgr_desc_default(&d);
    d.n_sub = 1;
    d.level = 4;
    size_t bytes = 0;
    if (hhgr_workspace_bytes(&d, &bytes) != HHGR_OK) return 1;
    void *ws = std::aligned_alloc(256, (bytes + 255) / 256 * 256);
    hhgr_ctx *c = nullptr;
    if (hhgr_create(&d, ws, bytes, nullptr, &c) != HHGR_OK) return 1;
    hhgr_sizes(c, &n, nullptr, nullptr);
    for (long long shift : {0LL, 1LL, 100LL, n - 1, -1LL, -100LL, -(n - 1), n, -n}) {
        std::vector<double> buf(3 * n, -7.0);
        double *x = buf.data() + n, *y = x + shift;
        for (long long q = 0; q < n; q++) x[q] = 0.5 * q + 1.0;
        std::vector<double> in(x, x + n);
        if (hhgr_mass_apply(c, x, y) != HHGR_OK) fails++;
        for (long long q = 0; q < n; q++)
            if (y[q] != in[q] + 3.0 * in[n - 1 - q]) {
                std::printf("FAIL: shift %lld entry %lld\n", shift, q);
                fails++;
                break;
            }
    }
    hhgr_destroy(c);
    std::free(ws);
    std::printf("engine_mass_check: %s (%d failures)\n", fails ? "FAILED" : "ok", fails);
    return fails ? 1 : 0;
}
