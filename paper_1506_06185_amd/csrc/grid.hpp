// Structured-grid path of the cube: descriptors and launchers.
//
// The Kuhn tetrahedra tile the N^3 grid and the operator couples a node to
// its 6 axis neighbours (k = 1: one stencil everywhere; per-element k: a
// weight per edge), so a context on the cube keeps u and b of every level as
// one grid, x fastest, and all its global cycles, a recovery's intact side
// included, run there (faulty tetrahedra recover in slot space): node (x, y, z) at
// x + P (y + N z), 0 <= x, y < N, 0 <= z <= N, with the Dirichlet nodes stored
// as zeros.  The row pitch P exceeds N, and row y = N of a plane is row y = 0
// of the next one, so every neighbour of an interior node is a plain offset
// and a row's node pairs (2p, 2p + 1) are aligned.
#pragma once

#include <hip/hip_runtime.h>

namespace hhgr {

struct VolDesc;

// row pitch: 128 bytes (FP64) beyond the power of two that N often is, so
// that a column of rows does not fall on one memory channel
inline int grid_pitch(int N) { return N + 16; }
inline long long grid_plane(int N) { return (long long)grid_pitch(N) * N; }
// one plane of zeros above, and two rows beyond it
inline long long grid_len(int N) { return grid_plane(N) * (N + 1) + 2 * grid_pitch(N); }

constexpr int kGridFromU = 0, kGridFromZero = 1, kGridProlong = 2;
constexpr int kGridPlain = 0, kGridRestrict = 1, kGridNorm = 2, kGridResidual = 3;

// Tiles of one marching launch: a workgroup owns vp pairs x vy rows x vz
// planes and loads tp pairs x ty rows (its own and the halo that the launch's
// passes need).
struct GridTiles {
    int vp = 0, vy = 0, vz = 0;
    int tp = 0, ty = 0;
    int ntx = 0, nty = 0, ntz = 0;
    int blocks() const { return ntx * nty * ntz; }
};

// ns red-black SOR sweeps of one level in one launch, u -> v (different
// buffers): from u, from zero (u is not read) or from u + P ec (linear
// interpolation of the coarse grid ec).  tail kGridRestrict also writes
// bc = P^T (b - A v) at the interior coarse nodes, kGridNorm leaves
// per-workgroup sums of (b - A v)^2 in partial.  frz (optional): one byte per
// node of the grid; nonzero nodes keep their values (take no correction) and
// do not count.
// w (optional): per-element k, the weight of the edge from each node along
// +x, then (w + wstride) +y, then +z; else k = 1.  Each of the three arrays
// holds the nodes of even x + y + z, then (wstride / 2 on) the odd ones, node
// (x, y, z) at (x >> 1) + (P / 2) (y + N z).
// code (optional, k = 1 with elements left out): weights as above, in bytes
// that count the elements of the edge: weight = code h / 6, 6 where none is
// left out.
// Built: ns = 1 from u (any tail), from zero (plain, restrict) and
// interpolating (plain, norm); ns = 2 from zero with k = 1 (plain, restrict);
// norms in FP64 only; code in FP64 with frz and without norms.
template <typename T>
struct GridSweep {
    int N = 0;
    double h = 0, omega = 1;
    const T *u = nullptr;
    T *v = nullptr;
    const T *b = nullptr;
    const T *ec = nullptr;
    T *bc = nullptr;
    const unsigned char *frz = nullptr;
    double *partial = nullptr;
    const T *w = nullptr;
    const unsigned char *code = nullptr;
    long long wstride = 0;
};

// r = b - A (u + e): e (optional) is added first and u + e written to v; r
// (optional) in its own type; per-workgroup sums of r^2 to partial (optional)
struct GridResidual {
    int N = 0;
    double h = 0;
    const double *u = nullptr, *b = nullptr;
    const float *e = nullptr;
    double *v = nullptr;
    double *r64 = nullptr;
    float *r32 = nullptr;
    const unsigned char *frz = nullptr;
    double *partial = nullptr;
    const double *w = nullptr;
    long long wstride = 0;
};

// node list of volume containers in slot space (see VolGeom) and where their
// nodes lie on the grid (tetinfo: subcube corner and axis order per tet)
struct GridClosures {
    const VolDesc *vd = nullptr;
    int nvol = 0;
    const unsigned *list = nullptr;
    int nlist = 0;
    const int2 *rowC = nullptr;
    const int *tetinfo = nullptr;
    int M = 0, N = 0;
};
// what a transfer from the grid does with the interior nodes of the closures
constexpr int kInteriorCopy = 0, kInteriorZero = 1, kInteriorKeep = 2;

// faulty tetrahedra (subcube corner, axis order), passed by value
struct GridTets {
    int n = 0;
    int info[8][6];
};

// closures of the local hierarchy on the finest level: container f (slots from
// f stride on) holds tetrahedron f of tets; rowC: first red and black slot of
// the rows of a container (M nodes per edge)
struct GridLocal {
    GridTets tets;
    long long stride = 0;
    const int2 *rowC = nullptr;
    int M = 0, N = 0;
};

// tiles of vp x vy x vz own pairs, rows and planes (rows and planes rounded up
// to even numbers) for ns sweeps, or for a residual with tail kGridResidual;
// the tiles chosen for a launch of that kind; and their workgroup size, at
// most 1024
GridTiles grid_tiles_of(int N, int ns, int tail, int vp, int vy, int vz);
int grid_threads(const GridTiles &t);

// The launchers.  The engine reaches them through this table, so that its
// host logic also links without device code (it then keeps the cube's
// vectors in slot space throughout).
struct GridOps {
    // vk: for launches with edge weights
    GridTiles (*tiles)(int N, int ns, int start, int tail, int word, bool vk);
    void (*sweep64)(hipStream_t, int ns, int start, int tail, const GridTiles &, const GridSweep<double> &);
    void (*sweep32)(hipStream_t, int ns, int start, int tail, const GridTiles &, const GridSweep<float> &);
    void (*residual)(hipStream_t, const GridTiles &, const GridResidual &);
    // r = b - A u, bc = P^T r and v = u + P ec in plain form (sweep counts of zero)
    void (*plain_residual64)(hipStream_t, int N, double h, const double *u, const double *b, const double *w,
                             long long wstride, double *r);
    void (*plain_residual32)(hipStream_t, int N, double h, const float *u, const float *b, const float *w,
                             long long wstride, float *r);
    // ... of an intact side whose frozen nodes do not hold their coarse
    // parents' zero: r = 0 and no correction there; weights w, or code
    void (*plain_residual_intact)(hipStream_t, int N, double h, const double *u, const double *b, const double *w,
                                  const unsigned char *code, long long wstride, const unsigned char *frz, double *r);
    void (*plain_prolong_intact)(hipStream_t, int N, const double *u, const double *ec, const unsigned char *frz, double *v);
    void (*plain_restrict64)(hipStream_t, int N, const double *r, double *bc);
    void (*plain_restrict32)(hipStream_t, int N, const float *r, float *bc);
    void (*plain_prolong64)(hipStream_t, int N, const double *u, const double *ec, double *v);
    void (*plain_prolong32)(hipStream_t, int N, const float *u, const float *ec, float *v);
    // coarsest level (N <= 12) by sine transforms: u = A^{-1} b; st holds the
    // [(N-1)^2] orthonormal sine transform matrix and the [N-1] values
    // 2 - 2 cos(pi q / N)
    void (*coarse64)(hipStream_t, int N, const double *st, const double *b, double *u);
    void (*coarse32)(hipStream_t, int N, const double *st, const float *b, float *u);
    // ... of another operator (rows val of 7 entries: itself, +x, -x, +y, -y,
    // +z, -z) by PCG preconditioned with those transforms; ord: unknown of
    // every interior node, x fastest (kernels.hip)
    void (*coarse_pcg64)(hipStream_t, int N, const int *ord, const double *val, const double *st, const double *b, double *u, double rtol, int maxit);
    void (*coarse_pcg32)(hipStream_t, int N, const int *ord, const double *val, const double *st, const float *b, float *u, double rtol, int maxit);
    // a whole cycle on a grid of N <= 16 cells, its coarsest level of Nc cells
    // included, in one workgroup (tail_fits): u = cycle from zero, or (norm
    // not null) from u, with the squared residual norm of the result to *norm
    bool (*tail_fits)(int N, int Nc);
    void (*tail64)(hipStream_t, int N, int Nc, int nu_pre, int nu_post, double h, double omega, const double *st,
                   const double *b, double *u, double *norm);
    void (*tail32)(hipStream_t, int N, int Nc, int nu_pre, int nu_post, double h, double omega, const double *st,
                   const float *b, float *u, double *norm);
    // vector order ((N-1)^3 interior nodes) <-> grid; per-workgroup sums of
    // squares to partial (optional); returns the number of workgroups
    int (*from_user)(hipStream_t, int N, const double *user, double *grid, double *partial);
    void (*to_user)(hipStream_t, int N, const double *grid, double *user);
    // grid = M f with f in vector order, sums of squares as above; and
    // y = M x from the grid to vector order
    int (*mass_load)(hipStream_t, int N, double h, const double *f, double *grid, double *partial);
    void (*mass_user)(hipStream_t, int N, double h, const double *grid, double *user);
    // edge weights of a level from its k per element (w, and rounded to w32 if
    // not null)
    void (*weights)(hipStream_t, int N, double h, const double *k, double *w, float *w32, long long wstride);
    // the same weights in slot space: from a node of the closures (list: every
    // node) along the tetrahedron's three axes, to w0, w1, w2 at the closures'
    // weight slots; and of a master's edges along +x, -x, +y, -y, +z, -z, to
    // [6][n] (weights of edges on the cube's boundary, which nothing reads: 0)
    void (*closure_weights)(hipStream_t, const GridClosures &, const double *w, long long wstride, double *w0, double *w1,
                            double *w2);
    void (*master_weights)(hipStream_t, int n, const int *xyz, int N, const double *w, long long wstride, double *wi);
    // weights of the edges from the nodes of the closures (list: every node)
    // over the elements whose macro tetrahedron is not flagged in faulty (null:
    // over all): w from the level's k per element, or code (w null)
    void (*intact_weights)(hipStream_t, const GridClosures &, int n_sub, double h, const double *k,
                           const unsigned char *faulty, double *w, unsigned char *code, long long wstride);
    // dJ/dk_T = -(h/6) sum over the path edges (a, b) of T of (lam_a - lam_b)
    // (u_a - u_b), element order
    void (*grad_k)(hipStream_t, int N, double h, const double *u, const double *lam, double *out);
    // grid -> closures: u (interior nodes: kInterior...) and the interior nodes
    // of b (optional); interior nodes of the closures -> grid
    void (*to_closures)(hipStream_t, const GridLocal &, int interior, const double *gu, double *u, const double *gb,
                        double *b);
    void (*from_closures)(hipStream_t, const GridLocal &, const double *vec, double *grid);
    // at the masters flagged in gamma: save = b, then b = A u with the masters'
    // weights wi [6][n] (+x, -x, +y, -y, +z, -z); and b = save
    void (*neumann)(hipStream_t, int n, const int *xyz, int N, const double *wi, const unsigned char *gamma, const double *u,
                    double *b, double *save);
    void (*neumann_end)(hipStream_t, int n, const int *xyz, int N, const unsigned char *gamma, const double *save, double *b);
    // grid = 0 strictly inside the tetrahedra; frz = 1 on their closures, or
    // strictly inside them and at the masters flagged in frozen, else 0
    void (*zero_tets)(hipStream_t, int N, int m, const GridTets &, double *grid);
    void (*freeze_tets)(hipStream_t, int N, int m, const GridTets &, unsigned char *frz);
    void (*freeze_inside)(hipStream_t, int N, int m, const GridTets &, int n, const int *xyz, const unsigned char *frozen,
                          unsigned char *frz);
};
const GridOps *grid_ops() __attribute__((weak));

template <typename T>
void launch_coarse_pcg_sine(hipStream_t s, int N, const int *ord, const double *val, const double *st, const T *b, T *u, double rtol, int maxit);

}  // namespace hhgr
