// CPU check of the structured-grid kernels around the sweeps (grid.hip in the
// device-code emulation of mockgrid/, under AddressSanitizer, LDS starting as
// NaN): sweeps and residuals with element counts at the edges, edge weights
// from k and their slot-space copies, the intact side's weights, nodes of
// single tetrahedra, closures, Neumann data, dJ/dk, the FP32 one-workgroup
// cycle, and every chosen tiling of the variants with edge weights, of FP32
// and of the residual.  References are written here from the definitions.
#define _USE_MATH_DEFINES
#include <cmath>
#include <cstdio>
#include <functional>
#include <random>
#include <vector>

#include "../../paper_1506_06185_amd/csrc/grid.hpp"
#include "../../paper_1506_06185_amd/csrc/kernels.hpp"
#include "../../paper_1506_06185_amd/csrc/topology.hpp"

namespace hhgr {
alignas(16) unsigned char grid_lds[kMockLds];
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
static void check(bool ok, const char *what, int a, int b, double err = 0.0) {
    cases++;
    if (!ok) {
        std::printf("FAIL %s %d %d: %.2e\n", what, a, b, err);
        fails++;
    }
}

static const int kOrder[6][3] = {{0, 1, 2}, {0, 2, 1}, {1, 0, 2}, {1, 2, 0}, {2, 0, 1}, {2, 1, 0}};

struct Grid {
    int N, P;
    long long S;
    explicit Grid(int n) : N(n), P(grid_pitch(n)), S(grid_plane(n)) {}
    long long at(int x, int y, int z) const { return x + (long long)P * y + S * z; }
    // place of an edge weight in its array
    long long w(int x, int y, int z) const {
        return (((x + y + z) & 1) ? grid_len(N) / 2 : 0) + (x >> 1) + (long long)(P / 2) * (y + (long long)N * z);
    }
};

template <typename T>
static std::vector<T> random_grid(int N, std::mt19937 &g) {
    Grid r(N);
    std::uniform_real_distribution<double> d(-1.0, 1.0);
    std::vector<T> v(grid_len(N), T(0));
    for (int z = 1; z < N; z++)
        for (int y = 1; y < N; y++)
            for (int x = 1; x < N; x++) v[r.at(x, y, z)] = (T)d(g);
    return v;
}

// position of a point in a subcube of m cells relative to a tetrahedron with
// axis order a, b, c: 0 outside the closure, 1 on its boundary, 2 inside
static int where(const Topology &tp, int t, int m, int x, int y, int z) {
    const int X[3] = {x, y, z};
    int d[3];
    for (int q = 0; q < 3; q++) d[q] = X[q] - m * tp.V0[t][q];
    const int a = d[tp.perm[t][0]], b = d[tp.perm[t][1]], c = d[tp.perm[t][2]];
    if (m < a || a < b || b < c || c < 0) return 0;
    return m > a && a > b && b > c && c > 0 ? 2 : 1;
}

// macro tetrahedron of fine element (cell, order q): its centroid is inside
static int tet_of(const Topology &tp, int m, int cx, int cy, int cz, int q) {
    double X[3] = {(double)cx, (double)cy, (double)cz};
    X[kOrder[q][0]] += 0.75;
    X[kOrder[q][1]] += 0.5;
    X[kOrder[q][2]] += 0.25;
    for (int t = 0; t < tp.n_tets; t++) {
        double d[3];
        bool in = true;
        for (int k = 0; k < 3; k++) {
            d[k] = X[k] - m * tp.V0[t][k];
            in = in && d[k] > 0.0 && d[k] < m;
        }
        if (in && d[tp.perm[t][0]] > d[tp.perm[t][1]] && d[tp.perm[t][1]] > d[tp.perm[t][2]]) return t;
    }
    return -1;
}

// sum over the elements that have the edge (x, y, z) + axis on their path
static double edge(int N, int x, int y, int z, int axis, const std::function<double(int, int, int, int)> &f) {
    double s = 0.0;
    for (int dd = 0; dd < 8; dd++) {
        const int dl[3] = {dd & 1, (dd >> 1) & 1, (dd >> 2) & 1};
        if (dl[axis]) continue;
        const int c[3] = {x - dl[0], y - dl[1], z - dl[2]};
        if (c[0] < 0 || c[1] < 0 || c[2] < 0 || c[0] >= N || c[1] >= N || c[2] >= N) continue;
        const int ns = dl[0] + dl[1] + dl[2];
        for (int q = 0; q < 6; q++) {
            bool on = kOrder[q][ns] == axis;
            for (int k = 0; k < ns; k++) on = on && dl[kOrder[q][k]];
            if (on) s += f(c[0], c[1], c[2], q);
        }
    }
    return s;
}

struct Mesh {
    Topology tp;
    int l;
    std::vector<VolDesc> all;
    std::vector<int> info;
    std::vector<int2> rowC;
    const TopoLevel &T() const { return tp.lev[l]; }
    Mesh(int n_sub, int level) : l(level) {
        const std::string e = tp.build(n_sub, level, 2);
        check(e.empty(), "topology", n_sub, level);
        for (int t = 0; t < tp.n_tets; t++) {
            all.push_back(VolDesc{(long long)t * T().C_pad, (long long)t * T().C_pad, t, 0});
            for (int a = 0; a < 3; a++) info.push_back(tp.V0[t][a]);
            for (int a = 0; a < 3; a++) info.push_back(tp.perm[t][a]);
        }
        for (auto &r : T().rowC) rowC.push_back(int2{r[0], r[1]});
    }
    GridLocal finest(const std::vector<int> &ft) const {
        GridLocal g;
        g.tets = tets(ft);
        g.stride = T().C_pad;
        g.rowC = rowC.data();
        g.M = T().M;
        g.N = T().N;
        return g;
    }
    GridClosures closures(const std::vector<VolDesc> &vd) const {
        GridClosures g;
        g.vd = vd.data();
        g.nvol = (int)vd.size();
        g.list = T().flist.data();
        g.nlist = (int)T().flist.size();
        g.rowC = rowC.data();
        g.tetinfo = info.data();
        g.M = T().M;
        g.N = T().N;
        return g;
    }
    GridTets tets(const std::vector<int> &ft) const {
        GridTets g;
        g.n = (int)ft.size();
        for (int q = 0; q < g.n; q++)
            for (int a = 0; a < 3; a++) {
                g.info[q][a] = tp.V0[ft[q]][a];
                g.info[q][3 + a] = tp.perm[ft[q]][a];
            }
        return g;
    }
    // local containers, one after the other
    std::vector<VolDesc> local(const std::vector<int> &ft) const {
        std::vector<VolDesc> v;
        for (size_t f = 0; f < ft.size(); f++)
            v.push_back(VolDesc{(long long)f * T().C_pad, (long long)ft[f] * T().C_pad, ft[f], 0});
        return v;
    }
    void node(int t, unsigned e, int &x, int &y, int &z, long long &slot) const {
        const int i = (int)(e & 1023u), j = (int)((e >> 10) & 1023u), k = (int)(e >> 20), m = T().m;
        int X[3] = {m * tp.V0[t][0] + k, m * tp.V0[t][1] + k, m * tp.V0[t][2] + k};
        X[tp.perm[t][0]] += i + j;
        X[tp.perm[t][1]] += j;
        x = X[0], y = X[1], z = X[2];
        slot = T().lay.index(i, j, k);
    }
};

// weights, intact weights, closures, tetrahedra, Neumann data
static void run_mesh(int n_sub, int level, const std::vector<int> &ft, unsigned seed) {
    std::mt19937 g(seed);
    const Mesh M(n_sub, level);
    const TopoLevel &T = M.T();
    const int N = T.N, m = T.m;
    const Grid r(N);
    const long long L = grid_len(N);
    const GridOps &o = *grid_ops();
    std::uniform_real_distribution<double> kd(0.1, 4.0);
    std::vector<double> k(6 * (size_t)N * N * N);
    for (auto &v : k) v = kd(g);
    std::vector<unsigned char> faulty(M.tp.n_tets, 0);
    for (int t : ft) faulty[t] = 1;
    const double h = 1.0 / N;
    // from k, in FP64 and rounded
    std::vector<double> w(3 * L, -1.0);
    std::vector<float> w32(3 * L, -1.0f);
    o.weights(nullptr, N, h, k.data(), w.data(), w32.data(), L);
    auto kval = [&](int cx, int cy, int cz, int q) { return k[6 * (cx + (size_t)N * (cy + (size_t)N * cz)) + q]; };
    auto read = [&](int a, int x, int y, int z) {  // an edge with an interior end
        const int X[3] = {x, y, z};
        bool in = X[a] < N;
        for (int b = 0; b < 3; b++) in = in && (b == a || (X[b] > 0 && X[b] < N));
        return in;
    };
    double e1 = 0.0, e2 = 0.0;
    for (int z = 0; z < N; z++)
        for (int y = 0; y < N; y++)
            for (int x = 0; x < N; x++)
                for (int a = 0; a < 3; a++) {
                    const double v = read(a, x, y, z) ? edge(N, x, y, z, a, kval) * h / 6.0 : 0.0;
                    e1 = std::max(e1, std::fabs(v - w[a * L + r.w(x, y, z)]));
                    e2 = std::max(e2, std::fabs((double)(float)v - (double)w32[a * L + r.w(x, y, z)]));
                }
    check(e1 < 1e-15 && e2 == 0.0, "weights", N, 0, e1);
    // slot-space copies
    std::vector<double> s0(T.n_slots, -1.0), s1(T.n_slots, -1.0), s2(T.n_slots, -1.0), wi(6 * (size_t)T.n_ifc, -1.0);
    o.closure_weights(nullptr, M.closures(M.all), w.data(), L, s0.data(), s1.data(), s2.data());
    o.master_weights(nullptr, T.n_ifc, &T.ifc_X[0][0], N, w.data(), L, wi.data());
    bool same = true;
    for (int t = 0; t < M.tp.n_tets; t++)
        for (unsigned e : T.flist) {
            int x, y, z;
            long long sl;
            M.node(t, e, x, y, z, sl);
            sl += (long long)t * T.C_pad;
            const std::vector<double> *s[3] = {&s0, &s1, &s2};
            for (int b = 0; b < 3; b++) {
                const int a = M.tp.perm[t][b];
                same = same && (*s[b])[sl] == (read(a, x, y, z) ? w[a * L + r.w(x, y, z)] : 0.0);
            }
        }
    for (int t = 0; t < T.n_ifc; t++)
        for (int a = 0; a < 3; a++) {
            int X[3] = {T.ifc_X[t][0], T.ifc_X[t][1], T.ifc_X[t][2]};
            same = same && wi[(size_t)(2 * a) * T.n_ifc + t] == w[a * L + r.w(X[0], X[1], X[2])];
            X[a]--;
            same = same && wi[(size_t)(2 * a + 1) * T.n_ifc + t] == w[a * L + r.w(X[0], X[1], X[2])];
        }
    check(same, "slot weights", N, 0);
    // the intact side's weights, and all elements again
    const std::vector<VolDesc> loc = M.local(ft);
    std::vector<double> wd(w);
    std::vector<unsigned char> code(3 * L, 6);
    for (int back = 0; back < 2; back++) {
        const unsigned char *fl = back ? nullptr : faulty.data();
        o.intact_weights(nullptr, M.closures(loc), n_sub, h, k.data(), fl, wd.data(), nullptr, L);
        o.intact_weights(nullptr, M.closures(loc), n_sub, h, nullptr, fl, nullptr, code.data(), L);
        double e = 0.0;
        bool ok = true;
        for (int z = 0; z < N; z++)
            for (int y = 0; y < N; y++)
                for (int x = 0; x < N; x++)
                    for (int a = 0; a < 3; a++) {
                        if (!read(a, x, y, z)) continue;
                        const long long i = a * L + r.w(x, y, z);
                        auto left = [&](int cx, int cy, int cz, int q) {
                            return fl && fl[tet_of(M.tp, m, cx, cy, cz, q)] ? 0.0 : 1.0;
                        };
                        auto sum = [&](int cx, int cy, int cz, int q) { return left(cx, cy, cz, q) * kval(cx, cy, cz, q); };
                        ok = ok && code[i] == (unsigned char)edge(N, x, y, z, a, left);
                        e = std::max(e, std::fabs(wd[i] - edge(N, x, y, z, a, sum) * h / 6.0));
                    }
        check(ok && e < 1e-15, "intact weights", N, back, e);
        if (back) {
            bool bits = true;
            for (long long q = 0; q < 3 * L; q++) bits = bits && wd[q] == w[q];
            check(bits, "weights restored", N, 0);
        } else {
            // a plain residual with the counts equals one with the weights they stand for
            const std::vector<double> u = random_grid<double>(N, g), b = random_grid<double>(N, g);
            std::vector<double> wc(3 * L, 0.0), ra(L, 0.0), rb(L, 0.0);
            for (long long q = 0; q < 3 * L; q++) wc[q] = code[q] * (h / 6.0);
            o.plain_residual64(nullptr, N, h, u.data(), b.data(), wc.data(), L, ra.data());
            std::vector<unsigned char> fz(L);
            for (auto &x : fz) x = (unsigned char)(g() % 4 == 0);
            o.plain_residual_intact(nullptr, N, h, u.data(), b.data(), nullptr, code.data(), L, fz.data(), rb.data());
            double d = 0.0;
            for (long long q = 0; q < L; q++) d = std::max(d, std::fabs((fz[q] ? 0.0 : ra[q]) - rb[q]));
            o.plain_residual_intact(nullptr, N, h, u.data(), b.data(), wc.data(), nullptr, L, fz.data(), rb.data());
            for (long long q = 0; q < L; q++) d = std::max(d, std::fabs((fz[q] ? 0.0 : ra[q]) - rb[q]));
            const std::vector<double> ec = random_grid<double>(N / 2, g);
            o.plain_prolong64(nullptr, N, u.data(), ec.data(), ra.data());
            o.plain_prolong_intact(nullptr, N, u.data(), ec.data(), fz.data(), rb.data());
            for (int z = 1; z < N; z++)
                for (int y = 1; y < N; y++)
                    for (int x = 1; x < N; x++) {
                        const long long i = r.at(x, y, z);
                        d = std::max(d, std::fabs((fz[i] ? u[i] : ra[i]) - rb[i]));
                    }
            check(d < 1e-14, "plain residual and correction of an intact side", N, 0, d);
        }
    }
    // single tetrahedra
    std::vector<double> u(L, 1.0);
    std::vector<unsigned char> fc(L, 9), fi(L, 9), fm(T.n_ifc);
    for (auto &v : fm) v = (unsigned char)(g() & 1);
    o.zero_tets(nullptr, N, m, M.tets(ft), u.data());
    o.freeze_tets(nullptr, N, m, M.tets(ft), fc.data());
    o.freeze_inside(nullptr, N, m, M.tets(ft), T.n_ifc, &T.ifc_X[0][0], fm.data(), fi.data());
    std::vector<unsigned char> master(L, 0);
    for (int t = 0; t < T.n_ifc; t++)
        if (fm[t]) master[r.at(T.ifc_X[t][0], T.ifc_X[t][1], T.ifc_X[t][2])] = 1;
    bool ok = true;
    long long outside = 0;
    std::vector<char> seen(L, 0);
    for (int z = 0; z <= N; z++)
        for (int y = 0; y < N; y++)
            for (int x = 0; x < N; x++) {
                int in = 0;
                for (int t : ft) in = std::max(in, where(M.tp, t, m, x, y, z));
                const long long i = r.at(x, y, z);
                seen[i] = 1;
                ok = ok && u[i] == (in == 2 ? 0.0 : 1.0) && fc[i] == (in ? 1 : 0) && fi[i] == (in == 2 || master[i] ? 1 : 0);
            }
    for (long long i = 0; i < L; i++)
        if (!seen[i] && (u[i] != 1.0 || fc[i] || fi[i])) outside++;
    check(ok && outside == 0, "tetrahedra", N, (int)outside);
    // closures of the faulty tetrahedra there and back
    const std::vector<double> v = random_grid<double>(N, g);
    std::vector<double> a(ft.size() * T.C_pad, 5.0), b(a), c(a), back(L, 0.0);
    const std::vector<double> v2 = random_grid<double>(N, g);
    std::vector<double> a2(a);
    o.to_closures(nullptr, M.finest(ft), kInteriorCopy, v.data(), a.data(), nullptr, nullptr);
    o.to_closures(nullptr, M.finest(ft), kInteriorZero, v.data(), b.data(), v2.data(), a2.data());
    o.to_closures(nullptr, M.finest(ft), kInteriorKeep, v.data(), c.data(), nullptr, nullptr);
    o.from_closures(nullptr, M.finest(ft), a.data(), back.data());
    ok = true;
    for (size_t f = 0; f < ft.size(); f++)
        for (unsigned e : T.flist) {
            int x, y, z;
            long long sl;
            M.node(ft[f], e, x, y, z, sl);
            sl += (long long)f * T.C_pad;
            const bool in = where(M.tp, ft[f], m, x, y, z) == 2;
            const double val = x > 0 && y > 0 && z > 0 && x < N && y < N && z < N ? v[r.at(x, y, z)] : 0.0;
            const double val2 = x > 0 && y > 0 && z > 0 && x < N && y < N && z < N ? v2[r.at(x, y, z)] : 0.0;
            ok = ok && a[sl] == val && a2[sl] == (in ? val2 : 5.0) && b[sl] == (in ? 0.0 : val) && c[sl] == (in ? 5.0 : val);
            if (in) ok = ok && back[r.at(x, y, z)] == val;
        }
    double inside = 0.0;
    for (double x : back) inside += x != 0.0;
    check(ok && inside == (double)ft.size() * T.ilist.size(), "closures", N, (int)inside);
    // Neumann data at flagged masters
    std::vector<unsigned char> gamma(T.n_ifc);
    for (auto &x : gamma) x = (unsigned char)(g() % 3 == 0);
    std::vector<double> rhs = random_grid<double>(N, g), rhs0(rhs), save(T.n_ifc, 0.0);
    o.neumann(nullptr, T.n_ifc, &T.ifc_X[0][0], N, wi.data(), gamma.data(), v.data(), rhs.data(), save.data());
    double e = 0.0;
    std::vector<char> changed(L, 0);
    for (int t = 0; t < T.n_ifc; t++) {
        const int x = T.ifc_X[t][0], y = T.ifc_X[t][1], z = T.ifc_X[t][2];
        const long long i = r.at(x, y, z);
        if (!gamma[t]) continue;
        changed[i] = 1;
        const double s = w[r.w(x, y, z)] * (v[i] - v[i + 1]) + w[r.w(x - 1, y, z)] * (v[i] - v[i - 1]) +
                         w[L + r.w(x, y, z)] * (v[i] - v[i + r.P]) + w[L + r.w(x, y - 1, z)] * (v[i] - v[i - r.P]) +
                         w[2 * L + r.w(x, y, z)] * (v[i] - v[i + r.S]) + w[2 * L + r.w(x, y, z - 1)] * (v[i] - v[i - r.S]);
        e = std::max(e, std::fabs(s - rhs[i]));
    }
    for (long long i = 0; i < L; i++)
        if (!changed[i] && rhs[i] != rhs0[i]) e = 1.0;
    o.neumann_end(nullptr, T.n_ifc, &T.ifc_X[0][0], N, gamma.data(), save.data(), rhs.data());
    check(e < 1e-14 && rhs == rhs0, "neumann", N, 0, e);
    // dJ/dk
    const std::vector<double> lam = random_grid<double>(N, g);
    std::vector<double> dk(6 * (size_t)N * N * N, -1.0);
    o.grad_k(nullptr, N, h, v.data(), lam.data(), dk.data());
    e = 0.0;
    for (int z = 0; z < N; z++)
        for (int y = 0; y < N; y++)
            for (int x = 0; x < N; x++)
                for (int q = 0; q < 6; q++) {
                    int X[3] = {x, y, z};
                    double s = 0.0;
                    for (int k2 = 0; k2 < 3; k2++) {
                        const long long i = r.at(X[0], X[1], X[2]);
                        X[kOrder[q][k2]]++;
                        const long long j = r.at(X[0], X[1], X[2]);
                        s += (lam[i] - lam[j]) * (v[i] - v[j]);
                    }
                    e = std::max(e, std::fabs(dk[6 * (x + (size_t)N * (y + (size_t)N * z)) + q] + h / 6.0 * s));
                }
    check(e < 1e-14, "grad_k", N, 0, e);
}

// one sweep with element counts (frozen nodes, tiles) against the same sweep
// with the weights they stand for
static void run_code(int N, int start, int tail, int vp, int vy, int vz, unsigned seed) {
    std::mt19937 g(seed);
    const Grid r(N);
    const long long L = grid_len(N), Lc = grid_len(N / 2);
    const std::vector<double> u = random_grid<double>(N, g), b = random_grid<double>(N, g), ec = random_grid<double>(N / 2, g);
    std::vector<unsigned char> code(3 * L), fz(L, 0);
    for (auto &c : code) c = (unsigned char)(1 + g() % 6);
    for (int z = 1; z < N; z++)
        for (int y = 1; y < N; y++)
            for (int x = 1; x < N; x++) fz[r.at(x, y, z)] = x > y && y > z && x < N / 2;
    std::vector<double> w(3 * L);
    for (long long q = 0; q < 3 * L; q++) w[q] = code[q] / 6.0 / N;
    std::vector<double> out[2], bc[2];
    for (int k = 0; k < 2; k++) {
        out[k].assign(L, 0.0);
        bc[k].assign(Lc, 0.0);
        GridSweep<double> s;
        s.N = N;
        s.h = 1.0 / N;
        s.omega = 1.25;
        s.u = u.data();
        s.v = out[k].data();
        s.b = b.data();
        s.ec = ec.data();
        s.bc = bc[k].data();
        s.frz = fz.data();
        s.w = k ? nullptr : w.data();
        s.code = k ? code.data() : nullptr;
        s.wstride = L;
        grid_ops()->sweep64(nullptr, 1, start, tail, grid_tiles_of(N, 1, tail, vp, vy, vz), s);
    }
    double e = 0.0;
    for (long long q = 0; q < L; q++)
        if (fz[q] && start != kGridFromZero && out[1][q] != u[q]) e = 1.0;  // frozen nodes keep their values
    for (long long q = 0; q < L; q++) e = std::max(e, std::isfinite(out[1][q]) ? std::fabs(out[0][q] - out[1][q]) : 1.0);
    for (long long q = 0; q < Lc; q++) e = std::max(e, std::isfinite(bc[1][q]) ? std::fabs(bc[0][q] - bc[1][q]) : 1.0);
    // (values up to the right-hand side over the smallest diagonal, N)
    check(e < 1e-13 * N * N, "sweep with counts", N, 10 * start + tail, e);
}

// the FP32 one-workgroup cycle against the FP64 one
static void run_tail32(int N, int Nc, int pre, int post, unsigned seed) {
    std::mt19937 g(seed);
    const std::vector<double> b = random_grid<double>(N, g);
    std::vector<double> u(b.size(), 0.0), st((Nc - 1) * Nc);
    std::vector<float> b32(b.begin(), b.end()), u32(b.size(), 0.0f);
    for (int i = 0; i < Nc - 1; i++) {
        for (int j = 0; j < Nc - 1; j++) st[i * (Nc - 1) + j] = std::sqrt(2.0 / Nc) * std::sin(M_PI * (i + 1) * (j + 1) / Nc);
        st[(Nc - 1) * (Nc - 1) + i] = 2.0 - 2.0 * std::cos(M_PI * (i + 1) / Nc);
    }
    grid_ops()->tail64(nullptr, N, Nc, pre, post, 1.0 / N, 1.25, st.data(), b.data(), u.data(), nullptr);
    grid_ops()->tail32(nullptr, N, Nc, pre, post, 1.0 / N, 1.25, st.data(), b32.data(), u32.data(), nullptr);
    double e = 0.0, big = 0.0;
    for (size_t q = 0; q < u.size(); q++) {
        e = std::max(e, std::isfinite(u32[q]) ? std::fabs(u[q] - u32[q]) : 1e9);
        big = std::max(big, std::fabs(u[q]));
    }
    // a few hundred roundings of 6e-8 each
    check(e < 1e-5 * big, "FP32 tail", N, Nc, e / big);
}

int main() {
    run_mesh(1, 3, {0}, 1);
    run_mesh(1, 4, {0, 1, 2, 3, 4, 5}, 2);
    run_mesh(1, 5, {3}, 5);
    run_mesh(2, 3, {9, 25, 8, 47}, 3);
    run_mesh(3, 3, {78, 37, 79}, 4);
    const int shapes[][4] = {{16, 8, 16, 16}, {16, 3, 6, 4}, {24, 5, 8, 10}, {8, 2, 2, 2}};
    const int kinds[][2] = {{kGridFromU, kGridPlain}, {kGridFromU, kGridRestrict}, {kGridFromZero, kGridPlain},
                            {kGridFromZero, kGridRestrict}, {kGridProlong, kGridPlain}};
    unsigned seed = 10;
    for (auto &s : shapes)
        for (auto &k : kinds) run_code(s[0], k[0], k[1], s[1], s[2], s[3], seed++);
    run_tail32(16, 8, 2, 1, seed++);
    run_tail32(16, 4, 1, 2, seed++);
    run_tail32(8, 4, 0, 1, seed++);
    run_tail32(12, 6, 2, 1, seed++);
    // chosen tilings: every size of one GPU, FP32 and FP64, with and without
    // edge weights, and the residual
    for (int n : {1, 2, 3})
        for (int N = 8 * n; N <= 1024; N *= 2)
            for (int word : {4, 8})
                for (bool vk : {false, true}) {
                    auto one = [&](int ns, int start, int tail) {
                        const GridTiles t = grid_ops()->tiles(N, ns, start, tail, word, vk);
                        check(t.blocks() > 0 && grid_threads(t) <= (vk ? 512 : 1024) && t.ntx * t.vp >= N / 2 &&
                                  t.nty * t.vy >= N && t.ntz * t.vz >= N && t.blocks() <= std::max(N * N / 4, 65536),
                              "tiles", N, 100 * ns + 10 * start + tail);
                    };
                    for (auto &k : kinds) one(1, k[0], k[1]);
                    if (!vk)
                        for (int tail : {kGridPlain, kGridRestrict}) one(2, kGridFromZero, tail);
                    if (word == 8) {
                        one(1, kGridFromU, kGridNorm);
                        one(1, kGridProlong, kGridNorm);
                        one(0, kGridFromU, kGridResidual);
                    }
                }
    std::printf("grid_side_check: %s (%d cases, %d failures)\n", fails ? "FAILED" : "ok", cases, fails);
    return fails ? 1 : 0;
}
