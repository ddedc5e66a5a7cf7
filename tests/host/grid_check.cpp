// CPU check of the structured-grid marching kernels (grid.hip) compiled for
// the host against the device-code emulation in mockgrid/: for several grid
// sizes and tile shapes, every built start and tail, FP64 and FP32, with and
// without frozen nodes, one sweep launch against plain sweeps,
// interpolation, residual and restriction written here node by node; the
// residual, mass and coarsest-level kernels likewise.  Buffers are exact-size
// vectors under AddressSanitizer, and LDS starts as NaN.
#define _USE_MATH_DEFINES
#include <cmath>
#include <cstdio>
#include <random>
#include <vector>

#include "../../paper_1506_06185_amd/csrc/grid.hpp"

namespace hhgr {
alignas(16) unsigned char grid_lds[kMockLds];
}
namespace hhgr {
// (another file's kernel, checked on the GPU)
template <typename T>
void launch_coarse_pcg_sine(hipStream_t, int, const int *, const double *, const double *, const T *, T *, double, int) {}
template void launch_coarse_pcg_sine<double>(hipStream_t, int, const int *, const double *, const double *,
                                             const double *, double *, double, int);
template void launch_coarse_pcg_sine<float>(hipStream_t, int, const int *, const double *, const double *,
                                            const float *, float *, double, int);
}  // namespace hhgr
using namespace hhgr;

static int fails = 0, cases = 0;

struct Ref {
    int N, P;
    long long S;
    explicit Ref(int n) : N(n), P(grid_pitch(n)), S(grid_plane(n)) {}
    long long at(int x, int y, int z) const { return x + (long long)P * y + S * z; }
};

template <typename T>
static std::vector<T> random_grid(int N, std::mt19937 &g) {
    Ref r(N);
    std::uniform_real_distribution<double> d(-1.0, 1.0);
    std::vector<T> v(grid_len(N), T(0));
    for (int z = 1; z < N; z++)
        for (int y = 1; y < N; y++)
            for (int x = 1; x < N; x++) v[r.at(x, y, z)] = (T)d(g);
    return v;
}

// edge weights in node order -> split by colour
template <typename T>
static std::vector<T> split(const Ref &r, const std::vector<T> &w) {
    const long long L = grid_len(r.N);
    std::vector<T> o(3 * L, T(0));
    for (int a = 0; a < 3; a++)
        for (int z = 0; z < r.N; z++)
            for (int y = 0; y < r.N; y++)
                for (int x = 0; x < r.N; x++)
                    o[a * L + (((x + y + z) & 1) ? L / 2 : 0) + (x >> 1) + (long long)(r.P / 2) * (y + (long long)r.N * z)] =
                        w[a * L + r.at(x, y, z)];
    return o;
}

template <typename T>
static void run_case(int N, int ns, int start, int tail, bool mask, int vp, int vy, int vz, unsigned seed, bool vk = false) {
    std::mt19937 g(seed);
    const Ref r(N), rc(N / 2);
    const std::vector<T> u = random_grid<T>(N, g), b = random_grid<T>(N, g);
    std::vector<T> e = random_grid<T>(N / 2, g);
    std::vector<unsigned char> fz(grid_len(N), 0);
    if (mask)
        for (int z = 1; z < N; z++)
            for (int y = 1; y < N; y++)
                for (int x = 1; x < N; x++) fz[r.at(x, y, z)] = x >= y && y >= z && x <= N / 2;
    if (mask && start == kGridProlong)
        for (int z = 0; z <= N / 2; z++)
            for (int y = 0; y < N / 2; y++)
                for (int x = 0; x < N / 2; x++)
                    if (x >= y && y >= z && x <= N / 4) e[rc.at(x, y, z)] = T(0);
    const double h = 1.0 / N, omega = 1.25;
    // reference
    std::vector<double> w(u.begin(), u.end());
    auto frozen = [&](long long i) { return mask && fz[i]; };
    if (start == kGridFromZero)
        for (auto &x : w) x = 0.0;
    if (mask && start == kGridFromZero)
        for (auto &x : w) x = 0.0;
    if (start == kGridProlong)
        for (int z = 1; z < N; z++)
            for (int y = 1; y < N; y++)
                for (int x = 1; x < N; x++)
                    w[r.at(x, y, z)] += 0.5 * ((double)e[rc.at(x / 2, y / 2, z / 2)] +
                                               (double)e[rc.at((x + 1) / 2, (y + 1) / 2, (z + 1) / 2)]);
    // edge weights: random around h, or h
    std::vector<T> ew(3 * grid_len(N), T(0));
    std::uniform_real_distribution<double> wd(0.2, 3.0);
    if (vk)
        for (auto &x : ew) x = (T)(h * wd(g));
    const long long L = grid_len(N);
    auto diag = [&](long long i) {
        return vk ? (double)ew[i] + ew[i - 1] + ew[L + i] + ew[L + i - r.P] + ew[2 * L + i] + ew[2 * L + i - r.S] : 6.0 * h;
    };
    auto rr = [&](long long i) {
        if (vk)
            return (double)b[i] - (diag(i) * w[i] - (ew[i] * w[i + 1] + ew[i - 1] * w[i - 1] + ew[L + i] * w[i + r.P] +
                                                     ew[L + i - r.P] * w[i - r.P] + ew[2 * L + i] * w[i + r.S] +
                                                     ew[2 * L + i - r.S] * w[i - r.S]));
        return (double)b[i] - h * (6.0 * w[i] - (w[i - 1] + w[i + 1] + w[i - r.P] + w[i + r.P] + w[i - r.S] + w[i + r.S]));
    };
    for (int q = 0; q < 2 * ns; q++)
        for (int z = 1; z < N; z++)
            for (int y = 1; y < N; y++)
                for (int x = 1; x < N; x++)
                    if (((x + y + z) & 1) == (q & 1) && !frozen(r.at(x, y, z))) w[r.at(x, y, z)] += omega / diag(r.at(x, y, z)) * rr(r.at(x, y, z));
    std::vector<double> res(w.size(), 0.0);
    double norm = 0.0;
    for (int z = 1; z < N; z++)
        for (int y = 1; y < N; y++)
            for (int x = 1; x < N; x++)
                if (!frozen(r.at(x, y, z))) {
                    const double v = rr(r.at(x, y, z));
                    res[r.at(x, y, z)] = v;
                    norm += v * v;
                }
    // launch
    GridTiles t = grid_tiles_of(N, ns, tail, vp, vy, vz);
    std::vector<T> v(grid_len(N), T(0)), bc(grid_len(N / 2), T(0));
    std::vector<double> part(t.blocks(), -1.0);
    GridSweep<T> gs;
    gs.N = N;
    gs.h = h;
    gs.omega = omega;
    gs.u = u.data();
    gs.v = v.data();
    gs.b = b.data();
    gs.ec = e.data();
    gs.bc = bc.data();
    gs.frz = mask ? fz.data() : nullptr;
    gs.partial = part.data();
    const std::vector<T> es = split(r, ew);
    gs.w = vk ? es.data() : nullptr;
    gs.wstride = L;
    if constexpr (sizeof(T) == 8)
        grid_ops()->sweep64(nullptr, ns, start, tail, t, gs);
    else
        grid_ops()->sweep32(nullptr, ns, start, tail, t, gs);
    const double tol = sizeof(T) == 8 ? 1e-13 : 3e-5;
    double err = 0.0;
    for (size_t i = 0; i < w.size(); i++) err = std::max(err, std::fabs(w[i] - (double)v[i]) / (std::isfinite((double)v[i]) ? 1.0 : 0.0));
    bool ok = err < tol * 4.0;
    double erc = 0.0, ern = 0.0;
    if (tail == kGridRestrict) {
        static const int d[7][3] = {{1, 0, 0}, {0, 1, 0}, {0, 0, 1}, {1, 1, 0}, {0, 1, 1}, {1, 0, 1}, {1, 1, 1}};
        for (int z = 0; z <= N / 2; z++)
            for (int y = 0; y < N / 2; y++)
                for (int x = 0; x < N / 2; x++) {
                    double s = 0.0;
                    const bool in = x > 0 && y > 0 && z > 0 && z < N / 2;
                    const long long i = r.at(2 * x, 2 * y, 2 * z);
                    if (in && frozen(i)) continue;  // a frozen coarse node is never read
                    if (in) {
                        s = res[i];
                        for (auto &o : d) {
                            const long long q = o[0] + (long long)r.P * o[1] + r.S * o[2];
                            s += 0.5 * (res[i + q] + res[i - q]);
                        }
                    }
                    erc = std::max(erc, std::fabs(s - (double)bc[rc.at(x, y, z)]));
                }
        ok = ok && erc < tol * 20.0;
    }
    if (tail == kGridNorm) {
        double s = 0.0;
        for (double x : part) s += x;
        ern = std::fabs(s - norm) / norm;
        ok = ok && ern < tol * 10.0;
    }
    cases++;
    if (!ok) {
        std::printf("FAIL vk=%d N=%d ns=%d start=%d tail=%d mask=%d tile %d %d %d word %zu: u %.2e bc %.2e norm %.2e\n", vk, N, ns, start,
                    tail, mask, vp, vy, vz, sizeof(T), err, erc, ern);
        fails++;
    }
}

static void check(bool ok, const char *what, int N, double err) {
    cases++;
    if (!ok) {
        std::printf("FAIL %s N=%d: %.2e\n", what, N, err);
        fails++;
    }
}

static void run_residual(int N, bool add, bool mask, bool vk, int vp, int vy, int vz, unsigned seed) {
    std::mt19937 g(seed);
    const Ref r(N);
    const std::vector<double> u = random_grid<double>(N, g), b = random_grid<double>(N, g);
    const std::vector<float> e = random_grid<float>(N, g);
    std::vector<unsigned char> fz(grid_len(N), 0);
    if (mask)
        for (int z = 1; z < N; z++)
            for (int y = 1; y < N; y++)
                for (int x = 1; x < N; x++) fz[r.at(x, y, z)] = x >= y && y >= z;
    GridResidual q;
    const GridTiles t = grid_tiles_of(N, 0, kGridResidual, vp, vy, vz);
    std::vector<double> v(grid_len(N), 0.0), r64(grid_len(N), 0.0), part(t.blocks(), -1.0);
    std::vector<float> r32(grid_len(N), 0.0f);
    q.N = N;
    q.h = 1.0 / N;
    q.u = u.data();
    q.b = b.data();
    q.e = add ? e.data() : nullptr;
    q.v = v.data();
    q.r64 = r64.data();
    q.r32 = r32.data();
    q.frz = mask ? fz.data() : nullptr;
    q.partial = part.data();
    const long long L = grid_len(N);
    std::vector<double> ew(3 * L, 0.0);
    std::uniform_real_distribution<double> wd(0.2, 3.0);
    for (auto &x : ew) x = vk ? wd(g) / N : 1.0 / N;
    const std::vector<double> es = split(r, ew);
    q.w = vk ? es.data() : nullptr;
    q.wstride = L;
    grid_ops()->residual(nullptr, t, q);
    std::vector<double> w(u);
    if (add)
        for (size_t i = 0; i < w.size(); i++) w[i] += (double)e[i];
    double err = 0.0, norm = 0.0, sum = 0.0;
    for (int z = 0; z < N; z++)
        for (int y = 0; y < N; y++)
            for (int x = 0; x < N; x++) {
                const long long i = r.at(x, y, z);
                double s = 0.0;
                if (x && y && z && !fz[i])
                    s = b[i] + ew[i - 1] * (w[i - 1] - w[i]) + ew[i] * (w[i + 1] - w[i]) + ew[L + i - r.P] * (w[i - r.P] - w[i]) +
                        ew[L + i] * (w[i + r.P] - w[i]) + ew[2 * L + i - r.S] * (w[i - r.S] - w[i]) + ew[2 * L + i] * (w[i + r.S] - w[i]);
                norm += s * s;
                err = std::max({err, std::fabs(s - r64[i]), std::fabs((float)s - r32[i]) * 1e-7, add ? std::fabs(w[i] - v[i]) : 0.0});
            }
    for (double x : part) sum += x;
    check(err < 1e-13 && std::fabs(sum - norm) < 1e-12 * norm, "residual", N, err);
}

static void run_mass(int N, unsigned seed) {
    std::mt19937 g(seed);
    const Ref r(N);
    const std::vector<double> f = random_grid<double>(N, g);
    const int n = N - 1;
    std::vector<double> user((size_t)n * n * n), out(user.size()), back(grid_len(N), 0.0), part(1 << 16, 0.0);
    grid_ops()->to_user(nullptr, N, f.data(), user.data());
    const int nb = grid_ops()->mass_load(nullptr, N, 1.0 / N, user.data(), back.data(), part.data());
    grid_ops()->mass_user(nullptr, N, 1.0 / N, f.data(), out.data());
    double err = 0.0, norm = 0.0, sum = 0.0, big = 0.0;
    for (int q = 0; q < nb; q++) sum += part[q];
    const double h3 = 1.0 / ((double)N * N * N);
    for (int z = 1; z < N; z++)
        for (int y = 1; y < N; y++)
            for (int x = 1; x < N; x++) {
                const long long i = r.at(x, y, z);
                auto two = [&](long long d) { return f[i + d] + f[i - d]; };
                const double s = h3 * (0.4 * f[i] + (two(1) + two(r.P) + two(r.S) + two(1 + r.P + r.S)) / 20.0 +
                                       (two(1 + r.P) + two(r.P + r.S) + two(1 + r.S)) / 30.0);
                const long long k = (x - 1) + (long long)n * ((y - 1) + (long long)n * (z - 1));
                norm += s * s;
                big = std::max(big, std::fabs(s));
                err = std::max({err, std::fabs(s - back[i]), std::fabs(s - out[k]), std::fabs(user[k] - f[i])});
            }
    check(err < 1e-14 * big && std::fabs(sum - norm) < 1e-12 * norm, "mass", N, err);
}

// the one-workgroup cycle against the same cycle of separate launches
static std::vector<double> launches(int N, int Nc, int pre, int post, const std::vector<double> &b, std::vector<double> u,
                                    const std::vector<double> &st) {
    const GridOps &o = *grid_ops();
    if (N == Nc) {
        o.coarse64(nullptr, N, st.data(), b.data(), u.data());
        return u;
    }
    std::vector<double> v(u.size(), 0.0), bc(grid_len(N / 2), 0.0), r(u.size(), 0.0);
    GridSweep<double> g;
    g.N = N;
    g.h = 1.0 / N;
    g.omega = 1.25;
    g.b = b.data();
    auto sweep = [&](int start) {
        g.u = u.data();
        g.v = v.data();
        o.sweep64(nullptr, 1, start, kGridPlain, grid_tiles_of(N, 1, kGridPlain, 4, 8, 8), g);
        u.swap(v);
    };
    for (int k = 0; k < pre; k++) sweep(kGridFromU);
    o.plain_residual64(nullptr, N, 1.0 / N, u.data(), b.data(), nullptr, 0, r.data());
    o.plain_restrict64(nullptr, N, r.data(), bc.data());
    const std::vector<double> e = launches(N / 2, Nc, pre, post, bc, std::vector<double>(bc.size(), 0.0), st);
    o.plain_prolong64(nullptr, N, u.data(), e.data(), v.data());
    u.swap(v);
    for (int k = 0; k < post; k++) sweep(kGridFromU);
    return u;
}

static void run_tail(int N, int Nc, int pre, int post, bool finest, unsigned seed) {
    std::mt19937 g(seed);
    const std::vector<double> b = random_grid<double>(N, g);
    std::vector<double> u = random_grid<double>(N, g), st((Nc - 1) * Nc);
    for (int i = 0; i < Nc - 1; i++) {
        for (int j = 0; j < Nc - 1; j++) st[i * (Nc - 1) + j] = std::sqrt(2.0 / Nc) * std::sin(M_PI * (i + 1) * (j + 1) / Nc);
        st[(Nc - 1) * (Nc - 1) + i] = 2.0 - 2.0 * std::cos(M_PI * (i + 1) / Nc);
    }
    const std::vector<double> w = launches(N, Nc, pre, post, b, finest ? u : std::vector<double>(u.size(), 0.0), st);
    std::vector<double> r(u.size(), 0.0);
    grid_ops()->plain_residual64(nullptr, N, 1.0 / N, w.data(), b.data(), nullptr, 0, r.data());
    double norm = -1.0, ref = 0.0, err = 0.0;
    for (double x : r) ref += x * x;
    grid_ops()->tail64(nullptr, N, Nc, pre, post, 1.0 / N, 1.25, st.data(), b.data(), u.data(), finest ? &norm : nullptr);
    for (size_t i = 0; i < u.size(); i++) err = std::max(err, std::isfinite(u[i]) ? std::fabs(u[i] - w[i]) : 1.0);
    check(err < 1e-11 && (!finest || std::fabs(norm - ref) < 1e-10 * ref), "tail", N, err);
}

int main() {
    const int shapes[][4] = {{16, 8, 16, 16}, {16, 3, 6, 4}, {24, 5, 8, 10}, {8, 4, 8, 8}, {8, 2, 2, 2}};
    const int kinds[][3] = {{1, 0, 0}, {1, 0, 1}, {1, 0, 2}, {1, 1, 0}, {1, 1, 1}, {1, 2, 0}, {1, 2, 2}, {2, 1, 0}, {2, 1, 1}};
    unsigned seed = 1;
    for (auto &sh : shapes) {
        for (auto &k : kinds) {
            run_case<double>(sh[0], k[0], k[1], k[2], false, sh[1], sh[2], sh[3], seed++);
            run_case<double>(sh[0], k[0], k[1], k[2], true, sh[1], sh[2], sh[3], seed++);
            if (k[0] == 1) run_case<double>(sh[0], 1, k[1], k[2], (seed & 1) != 0, sh[1], sh[2], sh[3], seed, true), seed++;
            if (k[2] != kGridNorm) run_case<float>(sh[0], k[0], k[1], k[2], (seed & 1) != 0, sh[1], sh[2], sh[3], seed++);
        }
        for (int q = 0; q < 8; q++) run_residual(sh[0], q & 1, (q >> 1) & 1, q >> 2, sh[1], sh[2], sh[3], seed++);
    }
    run_tail(16, 8, 2, 1, false, seed++);
    run_tail(16, 4, 2, 1, true, seed++);
    run_tail(8, 4, 1, 2, true, seed++);
    run_tail(8, 4, 0, 1, false, seed++);
    run_mass(8, seed++);
    run_mass(24, seed++);
    // every chosen tiling fits a workgroup, from the smallest grid to the largest of one GPU
    for (int N : {8, 12, 16, 24, 48, 64, 96, 128, 192, 256, 384, 512, 768})
        for (auto &k : kinds) {
            const GridTiles t = grid_ops()->tiles(N, k[0], k[1], k[2], 8, false);
            const bool ok = grid_threads(t) <= 1024 && t.ntx * t.vp >= N / 2 && t.nty * t.vy >= N && t.ntz * t.vz >= N &&
                            t.blocks() <= std::max(N * N / 4, 65536);
            check(ok, "tiles", N, t.blocks());
        }
    std::printf("grid_check: %s (%d cases, %d failures)\n", fails ? "FAILED" : "ok", cases, fails);
    return fails ? 1 : 0;
}
