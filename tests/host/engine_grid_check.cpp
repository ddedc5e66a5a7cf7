// Host-logic check of the engine's grid branches (mock HIP runtime and mock
// grid launchers, under AddressSanitizer): contexts of every kind on the cube
// through set-up, cycles, graphs, faults, recoveries, gradients, single
// operators, batches and the static solve.  Every launch's vectors are
// checked (mock_grid.hpp); the buffer that holds the solution after n cycles
// is the same with graphs, eagerly and in a batch.
#include <cstdio>
#include <cstdlib>
#include <vector>

#include "../../include/hhgr.h"
#include "mock_grid.hpp"

extern int g_mock_captures, g_mock_launches;
static int fails = 0;
#define CHECK(c, ...)                          \
    do {                                       \
        if (!(c)) {                            \
            std::printf("FAIL: " __VA_ARGS__); \
            std::printf(" (%s)\n", hhgr_last_error()); \
            fails++;                           \
        }                                      \
    } while (0)

struct Ctx {
    hhgr_desc d;
    hhgr_ctx *h = nullptr;
    void *ws = nullptr;
    size_t bytes = 0;
    long long n = 0, ne = 0;
    int nt = 0;
    std::vector<double> v, k;
    explicit Ctx(const hhgr_desc &desc) : d(desc) {
        CHECK(hhgr_workspace_bytes(&d, &bytes) == HHGR_OK, "workspace");
        ws = std::aligned_alloc(256, (bytes + 255) / 256 * 256);
        mockgrid::spaces.push_back({(const char *)ws, bytes});
        CHECK(hhgr_create(&d, ws, bytes, nullptr, &h) == HHGR_OK, "create");
        hhgr_sizes(h, &n, &nt, &ne);
        v.assign(n, 1.0);
        reg(v);
        if (d.variable_coeff) {
            k.assign(ne, 1.0);
            reg(k);
            CHECK(hhgr_set_coeff(h, k.data()) == HHGR_OK, "coeff");
        }
        CHECK(hhgr_set_rhs(h, v.data(), HHGR_RHS_LOAD) == HHGR_OK, "rhs");
    }
    ~Ctx() {
        hhgr_destroy(h);
        std::free(ws);
        mockgrid::spaces.clear();
    }
    Ctx(const Ctx &) = delete;
    static void reg(const std::vector<double> &x) { mockgrid::spaces.push_back({(const char *)x.data(), x.size() * sizeof(double)}); }
    const char *where() {
        CHECK(hhgr_get_solution(h, v.data()) == HHGR_OK, "get");
        return (const char *)mockgrid::last_solution;
    }
};

static hhgr_desc desc(int n_sub, int level, int precision, int vk, int pre, int post) {
    hhgr_desc d;
    hhgr_desc_default(&d);
    d.n_sub = n_sub;
    d.level = level;
    d.precision = precision;
    d.variable_coeff = vk;
    d.nu_pre = pre;
    d.nu_post = post;
    return d;
}

static void buffers(const hhgr_desc &d) {
    // offsets of the solution in the workspace after 0, 1, 2, 3 and 5 cycles
    std::vector<long long> at[3];
    for (int mode = 0; mode < 3; mode++) {  // eager, graph, batch
        Ctx c(d);
        hhgr_batch *b = nullptr;
        if (mode == 1) CHECK(hhgr_set_graph(c.h, 1) == HHGR_OK, "graph");
        if (mode == 2) CHECK(hhgr_batch_create(&c.h, 1, nullptr, &b) == HHGR_OK, "batch");
        for (int n : {0, 1, 1, 1, 2}) {
            if (mode == 2)
                CHECK(n == 0 || hhgr_batch_run(b, 1e-10, n, nullptr) == HHGR_ENOCONV, "batch run");
            else
                CHECK(hhgr_vcycle(c.h, n, nullptr) == HHGR_OK, "cycles");
            at[mode].push_back(c.where() - (const char *)c.ws);
        }
        if (b) hhgr_batch_destroy(b);
    }
    CHECK(at[0] == at[1] && at[0] == at[2], "buffers of n_sub %d level %d precision %d vk %d V(%d,%d)", d.n_sub, d.level,
          d.precision, d.variable_coeff, d.nu_pre, d.nu_post);
}

static void everything(const hhgr_desc &d) {
    Ctx c(d);
    double rr = 0.0;
    const int t2[2] = {c.nt - 1, 2}, t1[1] = {4};
    CHECK(hhgr_set_rhs(c.h, c.v.data(), HHGR_RHS_NODAL_F) == HHGR_OK, "nodal");
    const size_t N = (size_t)d.n_sub << d.level;
    std::vector<double> g((N + 1) * (N + 1) * (N + 1), 0.5), df(c.n), dk(c.ne), out(c.n);
    for (auto *x : {&g, &df, &dk, &out}) Ctx::reg(*x);
    CHECK(hhgr_set_rhs(c.h, g.data(), HHGR_RHS_DIRICHLET) == HHGR_OK, "dirichlet");
    CHECK(hhgr_set_solution(c.h, c.v.data()) == HHGR_OK && hhgr_set_solution(c.h, nullptr) == HHGR_OK, "solution");
    CHECK(hhgr_vcycle(c.h, 3, &rr) == HHGR_OK && hhgr_vcycle(c.h, 0, &rr) == HHGR_OK, "cycles");
    const int recover = d.max_faults > 1;
    CHECK(hhgr_inject_fault(c.h, t2[0]) == HHGR_OK, "fault");
    if (recover) {
        CHECK(hhgr_recover_local(c.h, t2[0], 2, &rr) == HHGR_OK && hhgr_recover_local(c.h, t2[1], 2, &rr) == HHGR_OK, "local");
        CHECK(hhgr_recover_dd(c.h, t2, 2, 2, 3) == HHGR_OK, "dd");
        CHECK(hhgr_recover_dn(c.h, t2, 2, 3, 2) == HHGR_OK, "dn");
        CHECK(hhgr_vcycle(c.h, 1, &rr) == HHGR_OK, "cycle after dn");
        CHECK(hhgr_recover_dn(c.h, t1, 1, 0, 1) == HHGR_OK, "dn without rounds");
    } else {
        CHECK(hhgr_recover_dn(c.h, t2, 2, 1, 1) == HHGR_EINVAL, "dn refused");
    }
    CHECK(hhgr_adjoint_grad(c.h, c.v.data(), 1e-10, 3, df.data(), d.variable_coeff ? dk.data() : nullptr) == HHGR_ENOCONV,
          "adjoint");
    CHECK(hhgr_mass_apply(c.h, c.v.data(), out.data()) == HHGR_OK, "mass");
    for (int op : {0, 1, 2, 3}) CHECK(hhgr_debug_op(c.h, op, d.level, c.v.data(), c.v.data(), out.data()) == HHGR_OK, "op %d", op);
    CHECK(hhgr_debug_op(c.h, 4, d.level, c.v.data(), nullptr, out.data()) == HHGR_OK, "op 4");
    CHECK(hhgr_debug_op(c.h, 5, d.level, c.v.data(), c.v.data(), out.data()) == HHGR_OK, "op 5");
    CHECK(hhgr_debug_op(c.h, 6, 2, c.v.data(), nullptr, out.data()) == HHGR_OK, "op 6");
    CHECK(hhgr_debug_op(c.h, 7, 2, c.v.data(), nullptr, out.data()) == (d.variable_coeff || d.n_sub > 2 ? HHGR_EINVAL : HHGR_OK),
          "op 7");
    const bool fused = !d.variable_coeff && d.precision == HHGR_FP64;
    CHECK(hhgr_debug_op(c.h, 9, d.level, c.v.data(), c.v.data(), out.data()) == (fused ? HHGR_OK : HHGR_EINVAL), "op 9");
    CHECK(hhgr_set_fused_sweeps(c.h, d.level, 1) == (d.variable_coeff ? HHGR_EINVAL : HHGR_OK), "fused sweeps");
    CHECK(hhgr_autotune(c.h, nullptr) == HHGR_OK, "autotune");
    CHECK(hhgr_set_tuning(c.h, 0, 512, 0, 4) == HHGR_OK, "tuning");
    long long launches = 0;
    double ms = 0.0, by = 0.0;
    CHECK(hhgr_kernel_timing(c.h, 1) == HHGR_OK && hhgr_vcycle(c.h, 2, nullptr) == HHGR_OK &&
              hhgr_kernel_stats(c.h, &launches, &ms, &by) == HHGR_OK && hhgr_kernel_timing(c.h, 0) == HHGR_OK,
          "timing");
    CHECK(d.nu_pre == 0 || (launches > 0 && by >= 8.0 * c.n), "timed launches %lld", launches);
    CHECK(hhgr_vcycle(c.h, 1, &rr) == HHGR_OK, "cycle at the end");
}

int main() {
    g_mock_res2 = 1.0;  // every residual norm is 1: nothing converges
    const int nus[][2] = {{2, 1}, {1, 1}, {3, 2}, {0, 2}, {2, 0}};
    for (auto &nu : nus)
        for (int precision : {HHGR_FP64, HHGR_MIXED})
            for (int vk : {0, 1})
                for (int level : {3, 4, 5}) buffers(desc(1, level, precision, vk, nu[0], nu[1]));
    for (int precision : {HHGR_FP64, HHGR_MIXED})
        for (int vk : {0, 1}) {
            everything(desc(2, 4, precision, vk, 2, 1));
            everything(desc(1, 4, precision, vk, 0, 1));
            everything(desc(3, 3, precision, vk, 1, 0));
            hhgr_desc d = desc(1, 5, precision, vk, 1, 2);
            d.max_faults = vk ? 2 : 0;
            everything(d);
        }
    {
        // batches: two members, one armed with one and then with two tetrahedra
        Ctx a(desc(2, 4, HHGR_FP64, 0, 2, 1));
        const auto first = mockgrid::spaces;
        Ctx b(desc(1, 5, HHGR_MIXED, 0, 2, 1));
        hhgr_ctx *hs[2] = {a.h, b.h};
        hhgr_batch *bt = nullptr;
        CHECK(hhgr_batch_create(hs, 2, nullptr, &bt) == HHGR_OK, "batch");
        const int sets[3][2] = {{3, 0}, {3, 17}, {5, 0}}, count[3] = {1, 2, 1};
        for (int r = 0; r < 3; r++) {
            CHECK(hhgr_batch_arm_dd(bt, 0, sets[r], count[r], r, 2) == HHGR_OK, "arm %d", r);
            CHECK(hhgr_batch_run(bt, 1e-10, 4, nullptr) == HHGR_ENOCONV, "armed run %d", r);
        }
        const int cap0 = g_mock_captures;
        for (int r = 0; r < 6; r++) CHECK(hhgr_batch_run(bt, 1e-10, 5, nullptr) == HHGR_ENOCONV, "run %d", r);
        CHECK(g_mock_captures - cap0 <= 2, "six plain runs captured %d steps", g_mock_captures - cap0);
        hhgr_batch_destroy(bt);
    }
    {
        hhgr_desc d = desc(2, 5, HHGR_FP64, 0, 2, 1);
        std::vector<double> rhs(63 * 63 * 63, 1.0), u(rhs);
        hhgr_report rep{0, 0.0, nullptr, 0};
        mockgrid::spaces.push_back({(const char *)0, ~(size_t)0 >> 1});  // (the static scratch)
        for (int kind : {HHGR_RHS_LOAD, HHGR_RHS_NODAL_F})
            CHECK(hhgr_solve_static(&d, rhs.data(), kind, 1e-8, 4, u.data(), &rep, nullptr) == HHGR_ENOCONV && rep.cycles == 4,
                  "static");
        mockgrid::spaces.clear();
    }
    fails += mockgrid::fails;
    std::printf("engine_grid_check: %s (%d failures, %lld grid launches)\n", fails ? "FAILED" : "ok", fails, mockgrid::launches);
    return fails ? 1 : 0;
}
