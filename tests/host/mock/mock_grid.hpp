// Host stand-in for the structured-grid launchers of grid.hpp (test use only),
// so that the engine's grid branches run on the CPU: the kernels are skipped,
// but every vector of a launch must lie in a registered workspace, be large
// enough and not overlap the vectors that the launch reads.  Residual sums are
// g_mock_res2.
#pragma once
#include <cstdio>
#include <cstdlib>
#include <utility>
#include <vector>

#include "../../../paper_1506_06185_amd/csrc/grid.hpp"
#include "../../../paper_1506_06185_amd/csrc/kernels.hpp"

extern double g_mock_res2;

namespace mockgrid {

inline std::vector<std::pair<const char *, size_t>> spaces;  // workspaces and user vectors
inline const void *last_solution = nullptr;                  // grid that to_user read last
inline long long launches = 0;
inline int fails = 0;

template <typename T>
void range(const T *p, long long n, const char *what) {
    const char *a = (const char *)p, *b = a + n * (long long)sizeof(T);
    for (auto &s : spaces)
        if (a >= s.first && b <= s.first + s.second) return;
    std::printf("FAIL: %s outside every workspace\n", what);
    fails++;
}
template <typename T, typename U>
void apart(const T *p, long long n, const U *q, long long m, const char *what) {
    const char *a = (const char *)p, *b = a + n * (long long)sizeof(T), *c = (const char *)q, *d = c + m * (long long)sizeof(U);
    if (a < d && c < b) {
        std::printf("FAIL: %s overlap\n", what);
        fails++;
    }
}

using namespace hhgr;

inline GridTiles tiles(int N, int, int, int, int, bool) {
    GridTiles t;
    t.vp = N / 2;
    t.vy = t.vz = N;
    t.tp = N / 2 + 1;
    t.ty = N + 1;
    t.ntx = t.nty = t.ntz = 1;
    return t;
}
template <typename T>
void sweep(hipStream_t, int ns, int start, int tail, const GridTiles &t, const GridSweep<T> &g) {
    launches++;
    const long long L = grid_len(g.N), Lc = grid_len(g.N / 2);
    range(g.v, L, "sweep v");
    range(g.b, L, "sweep b");
    apart(g.v, L, g.b, L, "sweep v and b");
    if (start != kGridFromZero) {
        range(g.u, L, "sweep u");
        apart(g.v, L, g.u, L, "sweep v and u");
    }
    if (start == kGridProlong) range(g.ec, Lc, "sweep ec");
    if (tail == kGridRestrict) {
        range(g.bc, Lc, "sweep bc");
        apart(g.bc, Lc, g.v, L, "sweep bc and v");
    }
    if (tail == kGridNorm) {
        range(g.partial, t.blocks(), "sweep partial");
        for (int q = 0; q < t.blocks(); q++) g.partial[q] = q ? 0.0 : g_mock_res2;
    }
    if (g.frz) range(g.frz, L, "sweep frz");
    if (g.w) range(g.w, 3 * L, "sweep w");
    if (g.code) range(g.code, 3 * L, "sweep code");
    // (the variants that grid.hip builds)
    const bool two = ns == 2 && start == kGridFromZero && !g.w && !g.code && tail != kGridNorm;
    const bool one = ns == 1 && (tail != kGridNorm || (sizeof(T) == 8 && start != kGridFromZero && !g.code)) &&
                     !(start == kGridProlong && tail == kGridRestrict) && !(g.code && (sizeof(T) != 8 || !g.frz || g.w));
    if (!(two || one) || t.blocks() < 1) {
        std::printf("FAIL: no such sweep: ns %d start %d tail %d\n", ns, start, tail);
        fails++;
    }
}
inline void residual(hipStream_t, const GridTiles &t, const GridResidual &g) {
    launches++;
    const long long L = grid_len(g.N);
    range(g.u, L, "residual u");
    range(g.b, L, "residual b");
    if (g.e) {
        range(g.e, L, "residual e");
        range(g.v, L, "residual v");
        apart(g.v, L, g.u, L, "residual v and u");
    }
    if (g.r32) {
        range(g.r32, L, "residual r32");
        if (g.e) apart(g.r32, L, g.e, L, "residual r32 and e");
    }
    if (g.frz) range(g.frz, L, "residual frz");
    if (g.w) range(g.w, 3 * L, "residual w");
    if (g.partial) {
        range(g.partial, t.blocks(), "residual partial");
        for (int q = 0; q < t.blocks(); q++) g.partial[q] = q ? 0.0 : g_mock_res2;
    }
}
template <typename T>
void plain_residual(hipStream_t, int N, double, const T *u, const T *b, const T *w, long long, T *r) {
    const long long L = grid_len(N);
    range(u, L, "plain u"), range(b, L, "plain b"), range(r, L, "plain r"), apart(r, L, u, L, "plain r and u");
    if (w) range(w, 3 * L, "plain w");
}
inline void plain_residual_intact(hipStream_t, int N, double, const double *u, const double *b, const double *w,
                                  const unsigned char *code, long long, const unsigned char *frz, double *r) {
    const long long L = grid_len(N);
    range(u, L, "plain u"), range(b, L, "plain b"), range(r, L, "plain r"), range(frz, L, "plain frz");
    if (w) range(w, 3 * L, "plain w");
    if (code) range(code, 3 * L, "plain code");
    if ((w != nullptr) == (code != nullptr)) fails++;
}
inline void plain_prolong_intact(hipStream_t, int N, const double *u, const double *ec, const unsigned char *frz, double *v) {
    range(u, grid_len(N), "prolong u"), range(ec, grid_len(N / 2), "prolong ec"), range(v, grid_len(N), "prolong v");
    range(frz, grid_len(N), "prolong frz");
}
template <typename T>
void plain_restrict(hipStream_t, int N, const T *r, T *bc) {
    range(r, grid_len(N), "restrict r"), range(bc, grid_len(N / 2), "restrict bc");
}
template <typename T>
void plain_prolong(hipStream_t, int N, const T *u, const T *ec, T *v) {
    range(u, grid_len(N), "prolong u"), range(ec, grid_len(N / 2), "prolong ec"), range(v, grid_len(N), "prolong v");
    apart(u, grid_len(N), v, grid_len(N), "prolong u and v");
}
template <typename T>
void coarse(hipStream_t, int N, const double *st, const T *b, T *u) {
    range(st, (long long)(N - 1) * N, "coarse st"), range(b, grid_len(N), "coarse b"), range(u, grid_len(N), "coarse u");
}
template <typename T>
void coarse_pcg(hipStream_t, int N, const int *ord, const double *val, const double *st, const T *b, T *u, double, int) {
    const long long n = (long long)(N - 1) * (N - 1) * (N - 1);
    range(ord, n, "pcg ord"), range(val, 7 * n, "pcg val"), range(st, (long long)(N - 1) * N, "pcg st");
    range(b, grid_len(N), "pcg b"), range(u, grid_len(N), "pcg u");
}
inline bool tail_fits(int N, int Nc) { return N <= 16 && Nc <= 8 && N > Nc && (N / 2 == Nc || (N == 16 && N / 4 == Nc)); }
template <typename T>
void tail(hipStream_t, int N, int Nc, int, int, double, double, const double *st, const T *b, T *u, double *norm) {
    launches++;
    range(st, (long long)(Nc - 1) * Nc, "tail st"), range(b, grid_len(N), "tail b"), range(u, grid_len(N), "tail u");
    if (norm) *norm = g_mock_res2;
}
inline int from_user(hipStream_t, int N, const double *user, double *grid, double *partial) {
    const long long n = N - 1;
    const int nb = (int)((n * n + 3) / 4);
    range(user, n * n * n, "from_user user"), range(grid, grid_len(N), "from_user grid");
    if (partial) {
        range(partial, nb, "from_user partial");
        for (int q = 0; q < nb; q++) partial[q] = q ? 0.0 : 1.0;
    }
    return nb;
}
inline void to_user(hipStream_t, int N, const double *grid, double *user) {
    const long long n = N - 1;
    range(user, n * n * n, "to_user user"), range(grid, grid_len(N), "to_user grid");
    last_solution = grid;
}
inline int mass_load(hipStream_t, int N, double, const double *f, double *grid, double *partial) {
    const long long n = N - 1;
    range(f, n * n * n, "mass_load f"), range(grid, grid_len(N), "mass_load grid"), range(partial, 4, "mass_load partial");
    for (int q = 0; q < 4; q++) partial[q] = q ? 0.0 : 1.0;
    return 4;
}
inline void mass_user(hipStream_t, int N, double, const double *grid, double *user) {
    const long long n = N - 1;
    range(user, n * n * n, "mass_user user"), range(grid, grid_len(N), "mass_user grid");
}
inline void weights(hipStream_t, int N, double, const double *k, double *w, float *w32, long long ws) {
    range(k, 6LL * N * N * N, "weights k"), range(w, 3 * ws, "weights w");
    if (w32) range(w32, 3 * ws, "weights w32");
}
// slots that a launch over closures reaches: those of its containers
inline void closures(const GridClosures &c, const double *vec, const char *what) {
    for (int v = 0; v < c.nvol; v++) {
        const VolDesc &d = c.vd[v];
        long long hi = 0;
        for (int e = 0; e < c.nlist; e++) {
            const int i = (int)(c.list[e] & 1023u), j = (int)((c.list[e] >> 10) & 1023u), k = (int)(c.list[e] >> 20);
            const int2 r = c.rowC[k * c.M - k * (k - 1) / 2 + j];
            hi = std::max<long long>(hi, (((i + k) & 1) ? r.y : r.x) + (i >> 1));
        }
        range(vec + d.w, hi + 1, what);
    }
    range(c.list, c.nlist, "closure list"), range(c.vd, c.nvol, "closure containers");
}
inline void closure_weights(hipStream_t, const GridClosures &c, const double *w, long long ws, double *w0, double *w1, double *w2) {
    range(w, 3 * ws, "closure_weights w");
    for (double *s : {w0, w1, w2}) closures(c, s, "closure weights");
}
inline void master_weights(hipStream_t, int n, const int *xyz, int, const double *w, long long ws, double *wi) {
    range(xyz, 3LL * n, "master xyz"), range(w, 3 * ws, "master w"), range(wi, 6LL * n, "master wi");
}
inline void intact_weights(hipStream_t, const GridClosures &c, int n_sub, double, const double *k, const unsigned char *faulty,
                           double *w, unsigned char *code, long long ws) {
    if ((w != nullptr) == (code != nullptr) || (w && !k)) {
        std::printf("FAIL: intact_weights takes k and w, or code\n");
        fails++;
    }
    if (w) range(w, 3 * ws, "intact w"), range(k, 6LL * c.N * c.N * c.N, "intact k");
    if (code) range(code, 3 * ws, "intact code");
    if (faulty) range(faulty, 6LL * n_sub * n_sub * n_sub, "intact faulty");
    range(c.list, c.nlist, "closure list"), range(c.vd, c.nvol, "closure containers");
}
inline void grad_k(hipStream_t, int N, double, const double *u, const double *lam, double *out) {
    range(u, grid_len(N), "grad u"), range(lam, grid_len(N), "grad lam"), range(out, 6LL * N * N * N, "grad out");
    apart(u, grid_len(N), lam, grid_len(N), "grad u and lam");
}
inline void to_closures(hipStream_t, const GridLocal &c, int, const double *gu, double *u, const double *gb, double *b) {
    range(gu, grid_len(c.N), "to_closures u");
    range(u, c.stride * c.tets.n, "to_closures vec u");
    if (c.tets.n < 1 || c.tets.n > 8) fails++;
    if (!gb) return;
    range(gb, grid_len(c.N), "to_closures b");
    range(b, c.stride * c.tets.n, "to_closures vec b");
    apart(u, c.stride * c.tets.n, b, c.stride * c.tets.n, "to_closures vecs");
}
inline void from_closures(hipStream_t, const GridLocal &c, const double *vec, double *grid) {
    range(grid, grid_len(c.N), "from_closures grid");
    range(vec, c.stride * c.tets.n, "from_closures vec");
}
inline void neumann(hipStream_t, int n, const int *xyz, int N, const double *wi, const unsigned char *gamma, const double *u,
                    double *b, double *save) {
    range(xyz, 3LL * n, "neumann xyz"), range(wi, 6LL * n, "neumann wi"), range(gamma, n, "neumann gamma");
    range(u, grid_len(N), "neumann u"), range(b, grid_len(N), "neumann b"), range(save, n, "neumann save");
}
inline void neumann_end(hipStream_t, int n, const int *, int N, const unsigned char *gamma, const double *save, double *b) {
    range(gamma, n, "neumann gamma"), range(b, grid_len(N), "neumann b"), range(save, n, "neumann save");
}
inline void zero_tets(hipStream_t, int N, int, const GridTets &t, double *grid) {
    range(grid, grid_len(N), "zero_tets grid");
    if (t.n < 1 || t.n > 8) fails++;
}
inline void freeze_tets(hipStream_t, int N, int, const GridTets &t, unsigned char *frz) {
    range(frz, (grid_len(N) + 3) / 4 * 4, "freeze frz");
    if (t.n < 1 || t.n > 8) fails++;
}
inline void freeze_inside(hipStream_t s, int N, int m, const GridTets &t, int n, const int *xyz, const unsigned char *frozen,
                          unsigned char *frz) {
    freeze_tets(s, N, m, t, frz);
    range(xyz, 3LL * n, "freeze xyz"), range(frozen, n, "freeze frozen");
}

inline const GridOps ops = {tiles,
                            sweep<double>,
                            sweep<float>,
                            residual,
                            plain_residual<double>,
                            plain_residual<float>,
                            plain_residual_intact,
                            plain_prolong_intact,
                            plain_restrict<double>,
                            plain_restrict<float>,
                            plain_prolong<double>,
                            plain_prolong<float>,
                            coarse<double>,
                            coarse<float>,
                            coarse_pcg<double>,
                            coarse_pcg<float>,
                            tail_fits,
                            tail<double>,
                            tail<float>,
                            from_user,
                            to_user,
                            mass_load,
                            mass_user,
                            weights,
                            closure_weights,
                            master_weights,
                            intact_weights,
                            grad_k,
                            to_closures,
                            from_closures,
                            neumann,
                            neumann_end,
                            zero_tets,
                            freeze_tets,
                            freeze_inside};

}  // namespace mockgrid

namespace hhgr {
const GridOps *grid_ops() { return &mockgrid::ops; }
}  // namespace hhgr
