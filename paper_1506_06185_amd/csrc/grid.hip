// HIP kernels (gfx950) of the structured-grid path (grid.hpp).
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstdlib>
#include <type_traits>

#include "elements.hpp"
#include "grid.hpp"
#include "kernels.hpp"

namespace hhgr {

extern __shared__ __align__(16) unsigned char grid_lds[];

namespace {

template <typename T>
struct alignas(2 * sizeof(T)) Pair {
    T lo, hi;
};

__device__ __forceinline__ unsigned grid_xcd(unsigned f, unsigned total) {
    const unsigned per = total >> 3, rem = total & 7u, x = f & 7u, loc = f >> 3;
    return x < rem ? x * (per + 1) + loc : rem * (per + 1) + (x - rem) * per + loc;
}

// workgroups of the variants with edge weights: their registers allow 3
// wavefronts per SIMD
constexpr int kVkThreads = 512;
// edges of a launch: weight h everywhere, weights in the vectors' type, or
// element counts in bytes (GridSweep::code)
constexpr int kEdgeUniform = 0, kEdgeWeights = 1, kEdgeCodes = 2;

// halo of a launch of K = 2 ns colour passes: nodes below and above a tile
// along each axis
constexpr int halo_lo(int K, int tail) { return tail == kGridResidual ? 1 : tail == kGridRestrict ? K + 2 : tail == kGridNorm ? K + 1 : K; }
constexpr int halo_hi(int K, int tail) { return tail == kGridResidual ? 1 : tail == kGridPlain ? K : K + 1; }

// sum over the workgroup to partial[blockIdx.x], in a fixed order (the LDS is free)
__device__ __forceinline__ void block_partial(double sum, double *partial) {
    double *red = (double *)grid_lds;
    const int tid = (int)threadIdx.x;
    red[tid] = sum;
    for (int n = (int)blockDim.x; n > 1;) {
        const int hf = (n + 1) >> 1;
        __syncthreads();
        if (tid + hf < n) red[tid] += red[tid + hf];
        n = hf;
    }
    if (tid == 0) partial[blockIdx.x] = red[0];
}

// ---------------------------------------------------------------------------
// ns red-black sweeps in one launch
// ---------------------------------------------------------------------------
// A workgroup marches through the planes of its tile.  A thread owns a pair
// of columns (2p, 2p + 1) of row y: column A has x + y even (red on even
// planes), column B has x + y odd.  At step z the active column X (A on even
// z, B on odd z) runs pass k = 1 .. K (red, black, red, ...) at its node of
// plane z - k + 1: that node has pass k's colour on every such plane, and
//   - its own old value is the column's pass k - 2 result of step z - 2,
//   - its neighbours along z are the column's pass k - 1 results of this step
//     and of step z - 2,
//   - its neighbours in the plane are pass k - 1 results of step z - 1 of
//     columns of the other kind: the pair's other column (in registers) and
//     three of neighbouring threads (in LDS).
// So every pass of a step reads what earlier steps published: one barrier per
// step, whatever the number of passes.  Passes at a tile's edge read nodes
// that the tile does not hold; the wrong values travel one node per pass and
// stay in the halo.
// VK (per-element k): a pass needs the 6 edge weights of its node, which it
// loads one step ahead; the residual of a red node reuses those of its red
// pass two steps before.  The weights are stored split by colour (grid.hpp),
// so the nodes of one pass read whole lines.  N = 128: 33, 63 and 47 us for a
// plain sweep, one with restriction, one with interpolation and norm (when the
// layout was chosen 37, 61 and 55, against 39, 71 and 64 in node order with
// every pass's weights loaded, and 43, 62 and 56 loading two steps ahead);
// bound by the instructions of the passes, of which the halo repeats as many
// again.  Bytes that count elements (k = 1, Dirichlet-Neumann) take 3 B per
// node in place of 24: 28, 60 and 32 us, at N = 256 184, 296 and 230 (edge
// weights 270, 391 and 361; one stencil with frozen nodes 99, 110 and 113).
template <typename T, int NS, int START, int TAIL, bool MASK, int VK>
__global__ void __launch_bounds__(VK ? kVkThreads : 1024) k_grid_sweep(GridSweep<T> g, GridTiles t, T h, T om, T omr) {
    constexpr int K = 2 * NS;
    constexpr bool RES = TAIL != kGridPlain;
    constexpr int NL = K + (RES ? 1 : 0);  // published results: pass 0 (the input) .. NL - 1
    constexpr int J0 = START == kGridFromZero ? 1 : 0;
    const int N = g.N, P = N + 16;
    const long long S = (long long)P * N;
    const unsigned f = grid_xcd(blockIdx.x, gridDim.x);
    const int ix = (int)(f % t.ntx), iy = (int)((f / t.ntx) % t.nty), iz = (int)(f / (t.ntx * t.nty));
    constexpr int HL = halo_lo(K, TAIL), HH = halo_hi(K, TAIL);
    // own ranges: pairs [P0, P1), rows [Y0, Y1), planes [Z0, Z1); loaded: + halo
    const int np = N / 2;
    const int P0 = ix * t.vp, P1 = min(np, P0 + t.vp);
    const int Y0 = iy * t.vy, Y1 = min(N, Y0 + t.vy);
    const int Z0 = iz * t.vz, Z1 = min(N, Z0 + t.vz);
    const int p0 = max(0, P0 - (HL + 1) / 2), p1 = min(np + 1, P1 + (HH + 1) / 2);
    const int y0 = max(0, Y0 - HL), y1 = min(N + 1, Y1 + HH);
    const int tid = (int)threadIdx.x;
    const int lr = tid / t.tp, lp = tid - lr * t.tp;
    const int p = p0 + lp, y = y0 + lr;
    const bool act = p < p1 && y < y1;
    const int yo = y & 1;
    // interior columns of A and B (x = 2p + yo and 2p + 1 - yo)
    const bool rowin = act && y >= 1 && y < N;
    bool in[2];
    in[0] = rowin && 2 * p + yo >= 1 && 2 * p + yo < N;
    in[1] = rowin && 2 * p + 1 - yo >= 1 && 2 * p + 1 - yo < N;
    const bool own = act && p >= P0 && p < P1 && y >= Y0 && y < Y1;
    // element offset of the pair in a plane (threads outside the tile read its first pair)
    const unsigned off = act ? (unsigned)(y * P + 2 * p) : (unsigned)(y0 * P + 2 * p0);

    const int rows = ((int)blockDim.x + t.tp - 1) / t.tp + 2;
    const int LS = rows * t.tp + 2;  // one published plane, a row of padding on each side
    T *const lds = (T *)grid_lds;
    const int li = (lr + 1) * t.tp + lp + 1;
    // neighbour of the other kind along x that is not the pair's own
    const int dxA = yo ? 1 : -1;
    // residual planes (ring of 3) for the restriction: [row][2 tp]
    const int RS = rows * 2 * t.tp + 2;
    T *const rs = lds + (NL - J0) * 2 * LS;
    const int ri = (lr + 1) * 2 * t.tp + 2 * lp + 1;

    // coarse grid of the interpolation and of the restriction
    const int Nc = N / 2, Pc = Nc + 16;
    const long long Sc = (long long)Pc * Nc;
    const int yc = act ? y : y0, pc = act ? p : p0;
    const unsigned cl = (unsigned)((yc >> 1) * Pc + pc), ch = (unsigned)(((yc + 1) >> 1) * Pc + pc);

    struct Load {
        Pair<T> u, b;
        T e0, e1, e2;
        unsigned short m, mu;
    };
    auto plane = [&](int z) { return min(max(z, 0), N); };
    // input of plane z and right-hand side of plane z - 1
    auto issue = [&](int z, Load &L) {
        const long long zu = plane(z), zb = plane(z - 1);
        if (START != kGridFromZero) L.u = *(const Pair<T> *)(g.u + zu * S + off);
        L.b = *(const Pair<T> *)(g.b + zb * S + off);
        if (START == kGridProlong) {
            const T *el = g.ec + (zu >> 1) * Sc, *eh = g.ec + ((zu + 1) >> 1) * Sc;
            L.e0 = el[cl];
            L.e1 = eh[ch];
            L.e2 = eh[ch + 1];
            if (MASK) L.mu = *(const unsigned short *)(g.frz + zu * S + off);
        }
        if (MASK) L.m = *(const unsigned short *)(g.frz + zb * S + off);
    };

    // published results of the two columns' last steps: pv[c][k], k = 0 .. K
    T pv[2][K + 1], uc[2], bh[2][NL + 1];
    unsigned fz[2] = {0u, 0u};  // frozen flags, bit k - 1: the node of pass k
#pragma unroll
    for (int c = 0; c < 2; c++) {
#pragma unroll
        for (int k = 0; k <= K; k++) pv[c][k] = T(0);
#pragma unroll
        for (int k = 0; k <= NL; k++) bh[c][k] = T(0);
        uc[c] = T(0);
    }
    double sum = 0.0;
    T acc = T(0);
    const int zs = (max(0, Z0 - HL) - 1) & ~1, ze = Z1 + (TAIL == kGridPlain ? K - 2 : TAIL == kGridNorm ? K - 1 : K);
    Load ld[2];
    issue(zs + 1, ld[1]);
    issue(zs + 2, ld[0]);
    const T hw = h / T(6);  // weight of one element at an edge (codes)
    // edge weights of a step's passes: along x to the neighbouring thread's
    // column and to the pair's other column, y - 1, y + 1, z - 1, z + 1
    using W = std::conditional_t<VK == kEdgeCodes, unsigned char, T>;
    using E = std::conditional_t<VK == kEdgeCodes, unsigned, T>;
    const W *gw = nullptr;
    if constexpr (VK == kEdgeCodes)
        gw = g.code;
    else
        gw = g.w;
    struct Edges {
        E x, o, ym, yp, zm, zp;
    };
    Edges ew[VK ? NL : 1] = {}, keep[2] = {};
    auto edges = [&](auto par, int z) {
        if constexpr (VK) {
            constexpr int X = decltype(par)::value;
            const int xl = X == 0 ? yo : 1 - yo;
            const bool right = (X == 0 ? dxA : -dxA) > 0;
            const unsigned PH = (unsigned)P >> 1;
            // (threads outside the tile and boundary nodes: any address of the grid)
            const unsigned o = (off >> 1) + (in[X] ? 0u : 1u + PH);
            const long long half = g.wstride >> 1;
#pragma unroll
            for (int k = 0; k < (NL > 2 ? 2 : NL); k++) {
                const long long zp = (min(max(z - k, 1), N - 1)) * (S >> 1);
                // the pass's own colour k & 1, and the other one
                const W *wo = gw + (k & 1 ? half : 0) + zp, *wn = gw + (k & 1 ? 0 : half) + zp;
                const E wr = wo[o], wl = wn[o + (unsigned)xl - 1u];
                ew[k].x = right ? wr : wl;
                ew[k].o = right ? wl : wr;
                ew[k].yp = wo[g.wstride + o];
                ew[k].ym = wn[g.wstride + o - PH];
                ew[k].zp = wo[2 * g.wstride + o];
                ew[k].zm = wn[2 * g.wstride + o - (S >> 1)];
            }
        }
    };
    edges(std::integral_constant<int, 0>(), zs);
    for (int q = tid; q < (NL - J0) * 2 * LS; q += (int)blockDim.x) lds[q] = T(0);
    __syncthreads();

    auto step = [&](auto par, int z) {
        constexpr int X = decltype(par)::value, Y = 1 - X;
        if (VK && NL > 2) ew[VK && NL > 2 ? 2 : 0] = keep[X];
        // input of plane z + 1 (both columns), right-hand side of plane z
        Load &L = ld[X ^ 1];
        T in0[2], b0[2];
        {
            T ul = START == kGridFromZero ? T(0) : L.u.lo, uh = START == kGridFromZero ? T(0) : L.u.hi;
            if (START == kGridProlong) {
                // a coarse node's own value (twice the half) at even (x, y, z)
                const T el = T(0.5) * (L.e0 + L.e1), eh = T(0.5) * (L.e0 + L.e2);
                ul += !MASK || !(L.mu & 0xffu) ? el : T(0);
                uh += !MASK || !(L.mu >> 8) ? eh : T(0);
            }
            in0[0] = yo ? uh : ul;
            in0[1] = yo ? ul : uh;
            b0[0] = yo ? L.b.hi : L.b.lo;
            b0[1] = yo ? L.b.lo : L.b.hi;
        }
        if (MASK) {
            const unsigned ml = (L.m & 0xffu) ? 1u : 0u, mh = (L.m >> 8) ? 1u : 0u;
            fz[0] = (fz[0] << 1) | (yo ? mh : ml);
            fz[1] = (fz[1] << 1) | (yo ? ml : mh);
        }
        issue(z + 3, L);
#pragma unroll
        for (int c = 0; c < 2; c++) {
#pragma unroll
            for (int k = NL; k > 0; k--) bh[c][k] = bh[c][k - 1];
            bh[c][0] = b0[c];
        }
        const int dx = X == 0 ? dxA : -dxA;
        // neighbours in the plane: results of step z - 1
        T nx[NL], ny[NL], nw[NL];
#pragma unroll
        for (int k = J0; k < NL; k++) {
            const T *l = lds + ((k - J0) * 2 + Y) * LS + li;
            nx[k] = l[dx];
            ny[k] = l[-t.tp];
            nw[k] = l[t.tp];
        }
        T res[K + 1];
        res[0] = in0[X];
        T rlast = T(0), rred = T(0);
#pragma unroll
        for (int k = 1; k <= NL; k++) {
            const int zp = z - k + 1;
            const bool up = in[X] && zp >= 1 && zp < N && (!MASK || !((fz[X] >> (k - 1)) & 1u));
            T ctr, rr;
            if (START == kGridFromZero && k == 1) {
                ctr = T(0);
                rr = bh[X][0];
            } else {
                ctr = k == 1 ? uc[X] : pv[X][k - 2];
                if constexpr (VK == kEdgeCodes) {
                    const Edges &e = ew[k - 1];
                    const T a = ((T(e.x) * nx[k - 1] + T(e.o) * pv[Y][k - 1]) + (T(e.ym) * ny[k - 1] + T(e.yp) * nw[k - 1])) +
                                (T(e.zp) * res[k - 1] + T(e.zm) * pv[X][k - 1]);
                    rr = bh[X][k - 1] - hw * (T(e.x + e.o + e.ym + e.yp + e.zm + e.zp) * ctr - a);
                } else if constexpr (VK) {
                    const Edges &e = ew[k - 1];
                    const T a = ((e.x * nx[k - 1] + e.o * pv[Y][k - 1]) + (e.ym * ny[k - 1] + e.yp * nw[k - 1])) +
                                (e.zp * res[k - 1] + e.zm * pv[X][k - 1]);
                    rr = bh[X][k - 1] - ((((e.x + e.o) + (e.ym + e.yp)) + (e.zm + e.zp)) * ctr - a);
                } else {
                    const T a = ((nx[k - 1] + pv[Y][k - 1]) + (ny[k - 1] + nw[k - 1])) + (res[k - 1] + pv[X][k - 1]);
                    rr = bh[X][k - 1] - h * (T(6) * ctr - a);
                }
            }
            if (k <= K) {
                T scale = om;
                if constexpr (VK == kEdgeCodes) {
                    const Edges &e = ew[k - 1];
                    scale = om / (hw * T(e.x + e.o + e.ym + e.yp + e.zm + e.zp));
                } else if constexpr (VK) {
                    const Edges &e = ew[k - 1];
                    scale = om / (((e.x + e.o) + (e.ym + e.yp)) + (e.zm + e.zp));
                }
                res[k] = up ? ctr + scale * rr : ctr;
                if (k == K) rlast = up ? omr * rr : T(0);
            } else {
                rred = up ? rr : T(0);
            }
        }
        if (VK) keep[X] = ew[0];
        edges(std::integral_constant<int, Y>(), z + 1);
        // the pair of plane z - K + 1 is final: X black now, Y red in step z - 1
        const int zo = z - K + 1;
        if (own && zo >= Z0 && zo < Z1) {
            const T x0 = X == 0 ? res[K] : pv[0][K - 1], x1 = X == 0 ? pv[1][K - 1] : res[K];
            Pair<T> o;
            o.lo = yo ? x1 : x0;
            o.hi = yo ? x0 : x1;
            *(Pair<T> *)(g.v + zo * S + off) = o;
        }
        if (TAIL == kGridNorm) {
            // residual of the black node of plane z - K + 1, of the red node of plane z - K
            if (own && zo >= Z0 && zo < Z1) sum += (double)rlast * (double)rlast;
            if (own && zo - 1 >= Z0 && zo - 1 < Z1) sum += (double)rred * (double)rred;
        }
        // publish; the input of plane z + 1 belongs to column X
#pragma unroll
        for (int k = J0; k < NL; k++) lds[((k - J0) * 2 + X) * LS + li] = res[k];
        if (TAIL == kGridRestrict) {
            const int zr = z - K;
            const int q0 = (zr + 3 * 1024) % 3, q1 = q0 == 2 ? 0 : q0 + 1, q2 = q1 == 2 ? 0 : q1 + 1;
            const int xl = X == 0 ? yo : 1 - yo;
            rs[q0 * RS + ri + xl] = rred;
            rs[q1 * RS + ri + xl] = rlast;
            // plane z - K - 1 is complete since the last barrier
            if (!yo) {
                const T *r = rs + q2 * RS + ri;
                const int zc = zr - 1, R2 = 2 * t.tp;
                const T c0 = r[0], xp = r[1], xm = r[-1], yp = r[R2], ym = r[-R2], pp = r[R2 + 1], mm = r[-R2 - 1];
                if (zc & 1) {
                    const T o = acc + T(0.5) * ((c0 + xp) + (yp + pp));
                    const int Zc = (zc - 1) >> 1;
                    if (own && p >= 1 && y >= 2 && Zc >= 1 && 2 * Zc >= Z0 && 2 * Zc < Z1)
                        g.bc[(long long)Zc * Sc + (unsigned)((y >> 1) * Pc + p)] = o;
                    acc = T(0.5) * ((c0 + xm) + (ym + mm));
                } else {
                    acc += c0 + T(0.5) * (((xp + xm) + (yp + ym)) + (pp + mm));
                }
            }
        }
#pragma unroll
        for (int k = 0; k <= K; k++) pv[X][k] = res[k];
        uc[Y] = in0[Y];
        __syncthreads();
    };
    for (int z = zs; z <= ze; z += 2) {
        step(std::integral_constant<int, 0>(), z);
        step(std::integral_constant<int, 1>(), z + 1);
    }
    if (TAIL == kGridNorm) block_partial(sum, g.partial);
}

// ---------------------------------------------------------------------------
// residual, with an FP32 correction added first
// ---------------------------------------------------------------------------
// The same march with no pass: step z publishes the pair of plane z + 1 and
// evaluates plane z from the plane published in step z - 1.
template <bool ADD, bool MASK, bool VK>
__global__ void __launch_bounds__(VK ? kVkThreads : 1024) k_grid_residual(GridResidual g, GridTiles t) {
    const int N = g.N, P = N + 16;
    const long long S = (long long)P * N;
    const unsigned f = grid_xcd(blockIdx.x, gridDim.x);
    const int ix = (int)(f % t.ntx), iy = (int)((f / t.ntx) % t.nty), iz = (int)(f / (t.ntx * t.nty));
    const int np = N / 2;
    const int P0 = ix * t.vp, P1 = min(np, P0 + t.vp), Y0 = iy * t.vy, Y1 = min(N, Y0 + t.vy);
    const int Z0 = iz * t.vz, Z1 = min(N, Z0 + t.vz);
    const int p0 = max(0, P0 - 1), p1 = min(np + 1, P1 + 1), y0 = max(0, Y0 - 1), y1 = min(N + 1, Y1 + 1);
    const int tid = (int)threadIdx.x, lr = tid / t.tp, lp = tid - lr * t.tp;
    const int p = p0 + lp, y = y0 + lr;
    const bool act = p < p1 && y < y1;
    const bool own = act && p >= P0 && p < P1 && y >= Y0 && y < Y1;
    const bool inlo = own && y >= 1 && p >= 1, inhi = own && y >= 1;
    const unsigned off = act ? (unsigned)(y * P + 2 * p) : (unsigned)(y0 * P + 2 * p0);
    const int rows = ((int)blockDim.x + t.tp - 1) / t.tp + 2;
    const int LS = rows * t.tp + 2, li = (lr + 1) * t.tp + lp + 1;
    Pair<double> *const lds = (Pair<double> *)grid_lds;
    const double h = g.h;
    struct Load {
        Pair<double> u, b;
        Pair<float> e;
    };
    // u (and e) of plane z, b of plane z - 1
    auto issue = [&](int z, Load &L) {
        const long long zu = min(max(z, 0), N), zb = min(max(z - 1, 0), N);
        L.u = *(const Pair<double> *)(g.u + zu * S + off);
        if (ADD) L.e = *(const Pair<float> *)(g.e + zu * S + off);
        L.b = *(const Pair<double> *)(g.b + zb * S + off);
    };
    Load ld[2];
    Pair<double> um = {0.0, 0.0}, uc = {0.0, 0.0};
    double sum = 0.0;
    const int zs = (max(0, Z0 - 1) - 1) & ~1, ze = Z1 - 1;
    issue(zs + 1, ld[1]);
    issue(zs + 2, ld[0]);
    auto step = [&](auto par, int z) {
        constexpr int X = decltype(par)::value;
        Load &L = ld[X ^ 1];
        Pair<double> up = L.u;
        if (ADD) {
            up.lo += (double)L.e.lo;
            up.hi += (double)L.e.hi;
        }
        const Pair<double> bb = L.b;
        issue(z + 3, L);
        lds[X * LS + li] = up;  // plane z + 1
        if (own && z >= Z0 && z < Z1) {
            const Pair<double> *l = lds + (X ^ 1) * LS + li;
            const Pair<double> ym = l[-t.tp], yp = l[t.tp];
            const double xm = l[-1].hi, xp = l[1].lo;
            const bool zin = z >= 1;
            bool a0 = inlo && zin, a1 = inhi && zin;
            if (MASK) {
                const unsigned short m = *(const unsigned short *)(g.frz + z * S + off);
                a0 = a0 && !(m & 0xffu);
                a1 = a1 && !(m >> 8);
            }
            double r0, r1;
            if constexpr (VK) {
                // colour-split weights: the pair's even node has the colour of y + z
                // (a boundary row or plane reads the weights of a node inside)
                const long long half = g.wstride >> 1, i = max(z, 1) * (S >> 1) + (off >> 1) + (y >= 1 ? 0 : P >> 1);
                const int cl = (y + z) & 1;
                const double *we = g.w + (cl ? half : 0) + i, *wo = g.w + (cl ? 0 : half) + i;
                const double *wye = we + g.wstride, *wyo = wo + g.wstride, *wze = wye + g.wstride, *wzo = wyo + g.wstride;
                const Pair<double> wx = {we[0], wo[0]}, wyp = {wye[0], wyo[0]}, wym = {wyo[-(P >> 1)], wye[-(P >> 1)]};
                const Pair<double> wzp = {wze[0], wzo[0]}, wzm = {wzo[-(S >> 1)], wze[-(S >> 1)]};
                const double wxm = wo[-1];
                const double d0 = ((wxm + wx.lo) + (wym.lo + wyp.lo)) + (wzm.lo + wzp.lo);
                const double d1 = ((wx.lo + wx.hi) + (wym.hi + wyp.hi)) + (wzm.hi + wzp.hi);
                r0 = bb.lo - (d0 * uc.lo - (((wxm * xm + wx.lo * uc.hi) + (wym.lo * ym.lo + wyp.lo * yp.lo)) +
                                            (wzm.lo * um.lo + wzp.lo * up.lo)));
                r1 = bb.hi - (d1 * uc.hi - (((wx.lo * uc.lo + wx.hi * xp) + (wym.hi * ym.hi + wyp.hi * yp.hi)) +
                                            (wzm.hi * um.hi + wzp.hi * up.hi)));
            } else {
                r0 = bb.lo - h * (6.0 * uc.lo - (((xm + uc.hi) + (ym.lo + yp.lo)) + (um.lo + up.lo)));
                r1 = bb.hi - h * (6.0 * uc.hi - (((uc.lo + xp) + (ym.hi + yp.hi)) + (um.hi + up.hi)));
            }
            Pair<double> r = {a0 ? r0 : 0.0, a1 ? r1 : 0.0};
            sum += r.lo * r.lo + r.hi * r.hi;
            if (ADD) *(Pair<double> *)(g.v + z * S + off) = uc;
            if (g.r64) *(Pair<double> *)(g.r64 + z * S + off) = r;
            if (g.r32) *(Pair<float> *)(g.r32 + z * S + off) = Pair<float>{(float)r.lo, (float)r.hi};
        }
        um = uc;
        uc = up;
        __syncthreads();
    };
    for (int z = zs; z <= ze; z += 2) {
        step(std::integral_constant<int, 0>(), z);
        step(std::integral_constant<int, 1>(), z + 1);
    }
    if (g.partial) block_partial(sum, g.partial);
}

// ---------------------------------------------------------------------------
// plain forms of the cycle's parts (sweep counts of zero): one node per thread
// ---------------------------------------------------------------------------
__device__ __forceinline__ bool grid_node(int N, int &x, int &y, int &z) {
    x = (int)(blockIdx.x * 64 + (threadIdx.x & 63)) + 1;
    y = (int)(blockIdx.y * 4 + (threadIdx.x >> 6)) + 1;
    z = (int)blockIdx.z + 1;
    return x < N && y < N;
}

// index of the weight of the edge from node (x, y, z) in its array
__device__ __forceinline__ long long grid_weight(int N, long long ws, int x, int y, int z) {
    return (((x + y + z) & 1) ? ws >> 1 : 0) + (x >> 1) + (long long)((N + 16) >> 1) * (y + (long long)N * z);
}

template <typename T>
__global__ void __launch_bounds__(256) k_grid_plain_residual(int N, T h, const T *u, const T *b, const T *w,
                                                             const unsigned char *code, const unsigned char *frz,
                                                             long long ws, T *r) {
    int x, y, z;
    if (!grid_node(N, x, y, z)) return;
    const int P = N + 16;
    const long long S = (long long)P * N, i = x + (long long)P * y + S * z;
    if (frz && frz[i]) {
        r[i] = T(0);
        return;
    }
    if (w || code) {
        auto at = [&](long long q) { return w ? w[q] : h / T(6) * T(code[q]); };
        const long long o = grid_weight(N, ws, x, y, z);
        const T a = at(grid_weight(N, ws, x - 1, y, z)), c = at(o), d = at(ws + grid_weight(N, ws, x, y - 1, z)), e = at(ws + o);
        const T f = at(2 * ws + grid_weight(N, ws, x, y, z - 1)), g = at(2 * ws + o);
        r[i] = b[i] - ((((a + c) + (d + e)) + (f + g)) * u[i] -
                       (((a * u[i - 1] + c * u[i + 1]) + (d * u[i - P] + e * u[i + P])) + (f * u[i - S] + g * u[i + S])));
        return;
    }
    r[i] = b[i] - h * (T(6) * u[i] - (((u[i - 1] + u[i + 1]) + (u[i - P] + u[i + P])) + (u[i - S] + u[i + S])));
}

// bc at coarse node (x, y, z) of the grid of N / 2 cells
template <typename T>
__global__ void __launch_bounds__(256) k_grid_plain_restrict(int N, const T *r, T *bc) {
    int x, y, z;
    if (!grid_node(N / 2, x, y, z)) return;
    const long long P = N + 16, S = P * N, i = 2 * (x + P * y + S * z);
    auto two = [&](long long d) { return r[i + d] + r[i - d]; };
    const T s = ((two(1) + two(P)) + (two(S) + two(1 + P))) + ((two(P + S) + two(1 + S)) + two(1 + P + S));
    const long long Pc = N / 2 + 16;
    bc[x + Pc * (y + (long long)(N / 2) * z)] = r[i] + T(0.5) * s;
}

template <typename T>
__global__ void __launch_bounds__(256) k_grid_plain_prolong(int N, const T *u, const T *ec, const unsigned char *frz,
                                                             T *v) {
    int x, y, z;
    if (!grid_node(N, x, y, z)) return;
    const long long P = N + 16, i = x + P * (y + (long long)N * z), Pc = N / 2 + 16, Nc = N / 2;
    const T e0 = ec[(x >> 1) + Pc * ((y >> 1) + Nc * (z >> 1))];
    const T e1 = ec[((x + 1) >> 1) + Pc * (((y + 1) >> 1) + Nc * ((z + 1) >> 1))];
    v[i] = frz && frz[i] ? u[i] : u[i] + T(0.5) * (e0 + e1);
}

// ---------------------------------------------------------------------------
// coarsest level: u = A^{-1} b by sine transforms along x, y and z
// ---------------------------------------------------------------------------
// One workgroup, everything in LDS: six products with the (N - 1)^2 sine
// matrix and a division by the eigenvalues.  Exact to rounding, whatever the
// right-hand side; the data (343 or 1331 unknowns) is far below one CU's
// LDS, so the time is the launch and six short barriers.
constexpr int kSineMax = 11;
__device__ __forceinline__ void sine_axis(int n, int stride, int q, int c, const double *st, const double *in, double *out) {
    // out at element q, coordinate c along the axis of that stride
    const double *a = in + q - c * stride;
    double s = 0.0;
    for (int j = 0; j < n; j++) s += st[c * n + j] * a[j * stride];
    out[q] = s;
}

template <typename T>
__global__ void __launch_bounds__(512) k_grid_coarse(int N, const double *st, const T *b, T *u) {
    double *const A = (double *)grid_lds, *const B = A + kSineMax * kSineMax * kSineMax;
    double *const S = B + kSineMax * kSineMax * kSineMax;
    const int n = N - 1, n2 = n * n, n3 = n2 * n, tid = (int)threadIdx.x, nt = (int)blockDim.x;
    const long long P = N + 16;
    for (int q = tid; q < n2 + n; q += nt) S[q] = st[q];
    for (int q = tid; q < n3; q += nt) A[q] = (double)b[(q % n + 1) + P * ((q / n) % n + 1 + (long long)N * (q / n2 + 1))];
    __syncthreads();
    for (int q = tid; q < n3; q += nt) sine_axis(n, 1, q, q % n, S, A, B);
    __syncthreads();
    for (int q = tid; q < n3; q += nt) sine_axis(n, n, q, (q / n) % n, S, B, A);
    __syncthreads();
    for (int q = tid; q < n3; q += nt) {
        sine_axis(n, n2, q, q / n2, S, A, B);
        B[q] *= (double)N / ((S[n2 + q % n] + S[n2 + (q / n) % n]) + S[n2 + q / n2]);
    }
    __syncthreads();
    for (int q = tid; q < n3; q += nt) sine_axis(n, 1, q, q % n, S, B, A);
    __syncthreads();
    for (int q = tid; q < n3; q += nt) sine_axis(n, n, q, (q / n) % n, S, A, B);
    __syncthreads();
    for (int q = tid; q < n3; q += nt) {
        sine_axis(n, n2, q, q / n2, S, B, A);
        u[(q % n + 1) + P * ((q / n) % n + 1 + (long long)N * (q / n2 + 1))] = (T)A[q];
    }
}

// ---------------------------------------------------------------------------
// the last levels (N <= 16) of a cycle in one workgroup
// ---------------------------------------------------------------------------
// At 15^3 nodes and fewer a launch costs more than its work (9 + 5 us for the
// two sweep launches of N = 16, 4 us for the coarsest level), so one
// workgroup runs every pass of these levels in LDS: u of a level lives there
// with its zero boundary, b and (while the level's residual takes its place)
// u in the registers of the threads that own the nodes.  A thread owns pairs
// of nodes (2p, 2p + 1), one of each colour; the LDS holds the colours apart,
// node (x, y, z) of colour c at c H + (x >> 1) + (N / 2 + 1) (y + (N + 1) z),
// so a pass reads and writes consecutive words.  16 us from zero at N = 16, bound
// by about 25 barriers and the latency between them (with the nodes in grid
// order in LDS, half of its banks idle, 17 us).
constexpr int kTailN = 16, kTailThreads = 1024;
constexpr __host__ __device__ int tail_half(int N) { return (N / 2 + 1) * (N + 1) * (N + 1); }
constexpr __host__ __device__ int tail_len(int N) { return 2 * tail_half(N); }

struct TailLds {
    double *A, *B, *S;  // sine transforms of the coarsest level
    double *red;
};

// index of node (x, y, z) in the colour-split layout of a level
__device__ __forceinline__ int tail_at(int N, int x, int y, int z) {
    return ((x + y + z) & 1) * tail_half(N) + (x >> 1) + (N / 2 + 1) * (y + (N + 1) * z);
}
// sum of the 6 neighbours of the pair's node o (0: 2p, 1: 2p + 1) of colour
// c; i: the pair's index, mate: the pair's other node
template <typename T>
__device__ __forceinline__ T tail_around(const T *lv, int N, int i, int c, int o, T mate) {
    const int PH = N / 2 + 1, SH = PH * (N + 1);
    const T *v = lv + (c ? 0 : tail_half(N)) + i;
    return ((mate + v[o ? 1 : -1]) + (v[-PH] + v[PH])) + (v[-SH] + v[SH]);
}

// NP: pairs per thread; lv: this level's u, then the coarser levels'; bl: the
// restricted right-hand side of the next coarser level, in grid order
template <typename T, int NP>
__device__ __forceinline__ void tail_level(int N, int Nc, const T (&b)[NP][2], T (&u)[NP][2], bool zero, T h, T om, int nu_pre,
                                           int nu_post, T *lv, T *bl, const TailLds &q) {
    const int tid = (int)threadIdx.x, nt = (int)blockDim.x;
    const int PH = N / 2 + 1, H = tail_half(N), np = N / 2, npairs = np * (N - 1) * (N - 1);
    const int safe = PH * (N + 2) + 1;  // an interior pair
    int idx[NP], par[NP];
    bool act[NP], lo[NP];
#pragma unroll
    for (int s = 0; s < NP; s++) {
        const int k = tid + s * nt;
        act[s] = k < npairs;
        const int p = k % np, y = (k / np) % (N - 1) + 1, z = k / (np * (N - 1)) + 1;
        idx[s] = act[s] ? p + PH * (y + (N + 1) * z) : safe;
        par[s] = (y + z) & 1;
        lo[s] = act[s] && p > 0;
    }
    for (int k = tid; k < tail_len(N); k += nt) lv[k] = T(0);
    __syncthreads();
    auto put = [&](const T(&v)[NP][2]) {
#pragma unroll
        for (int s = 0; s < NP; s++) {
            if (lo[s]) lv[par[s] * H + idx[s]] = v[s][0];
            if (act[s]) lv[(1 - par[s]) * H + idx[s]] = v[s][1];
        }
        __syncthreads();
    };
    auto sweep = [&]() {
        for (int c = 0; c < 2; c++) {
#pragma unroll
            for (int s = 0; s < NP; s++) {
                const int o = par[s] ^ c;  // the pair's node of colour c
                const bool on = o ? act[s] : lo[s];
                const int i = on ? idx[s] : safe;
                const T ctr = o ? u[s][1] : u[s][0], mate = o ? u[s][0] : u[s][1], bb = o ? b[s][1] : b[s][0];
                const T n = ctr + om * (bb - h * (T(6) * ctr - tail_around(lv, N, i, c, o, mate)));
                if (on) lv[c * H + i] = n;
                u[s][0] = on && !o ? n : u[s][0];
                u[s][1] = on && o ? n : u[s][1];
            }
            __syncthreads();
        }
    };
    if (zero) {
#pragma unroll
        for (int s = 0; s < NP; s++) u[s][0] = u[s][1] = T(0);
    } else {
        put(u);
    }
    for (int k = 0; k < nu_pre; k++) sweep();
    T r[NP][2];
#pragma unroll
    for (int s = 0; s < NP; s++)
#pragma unroll
        for (int o = 0; o < 2; o++) {
            const int i = (o ? act[s] : lo[s]) ? idx[s] : safe;
            r[s][o] = b[s][o] - h * (T(6) * u[s][o] - tail_around(lv, N, i, par[s] ^ o, o, u[s][1 - o]));
        }
    __syncthreads();
    put(r);
    // restriction to the coarser level
    const int M = N / 2, Pm = M + 2, Sm = Pm * (M + 1), nm = M - 1;
    T *const lc = lv + tail_len(N);
    for (int k = tid; k < nm * nm * nm; k += nt) {
        const int x = k % nm + 1, y = (k / nm) % nm + 1, z = k / (nm * nm) + 1;
        // fine node (2x, 2y, 2z), colour 0; an offset of odd sum is colour 1,
        // an odd step down in x is the pair before
        const T *e = lv + x + PH * (2 * y + 2 * (N + 1) * z), *o = e + H;
        const int Y = PH, Z = PH * (N + 1);
        const T s1 = ((o[0] + o[-1]) + (o[Y] + o[-Y])) + (o[Z] + o[-Z]);
        const T s2 = ((e[Y] + e[-1 - Y]) + (e[Y + Z] + e[-Y - Z])) + (e[Z] + e[-1 - Z]);
        const T v = e[0] + T(0.5) * ((s1 + s2) + (o[Y + Z] + o[-1 - Y - Z]));
        bl[x + Pm * y + Sm * z] = v;
    }
    __syncthreads();
    put(u);
    if (M == Nc) {
        for (int k = tid; k < tail_len(M); k += nt) lc[k] = T(0);
        const int n2 = nm * nm, n3 = n2 * nm;
        auto each = [&](auto f) {
            __syncthreads();
            for (int k = tid; k < n3; k += nt) f(k, k % nm, (k / nm) % nm, k / n2);
        };
        each([&](int k, int x, int y, int z) { q.A[k] = (double)bl[(x + 1) + Pm * (y + 1) + Sm * (z + 1)]; });
        each([&](int k, int x, int, int) { sine_axis(nm, 1, k, x, q.S, q.A, q.B); });
        each([&](int k, int, int y, int) { sine_axis(nm, nm, k, y, q.S, q.B, q.A); });
        each([&](int k, int x, int y, int z) {
            sine_axis(nm, n2, k, z, q.S, q.A, q.B);
            q.B[k] *= (double)M / ((q.S[n2 + x] + q.S[n2 + y]) + q.S[n2 + z]);
        });
        each([&](int k, int x, int, int) { sine_axis(nm, 1, k, x, q.S, q.B, q.A); });
        each([&](int k, int, int y, int) { sine_axis(nm, nm, k, y, q.S, q.A, q.B); });
        each([&](int k, int x, int y, int z) {
            sine_axis(nm, n2, k, z, q.S, q.B, q.A);
            lc[tail_at(M, x + 1, y + 1, z + 1)] = (T)q.A[k];
        });
        __syncthreads();
    } else if constexpr (NP > 1) {
        // one pair per thread below N = 16
        T bm[1][2], um[1][2];
        const int k = tid, mp = M / 2;
        const bool on = k < mp * nm * nm;
        const int i = on ? 2 * (k % mp) + Pm * ((k / mp) % nm + 1) + Sm * (k / (mp * nm) + 1) : 0;
        bm[0][0] = on && k % mp > 0 ? bl[i] : T(0);
        bm[0][1] = on ? bl[i + 1] : T(0);
        um[0][0] = um[0][1] = T(0);
        __syncthreads();
        tail_level<T, 1>(M, Nc, bm, um, true, T(2) * h, T(0.5) * om, nu_pre, nu_post, lc, bl, q);
    }
    // interpolation from lc
#pragma unroll
    for (int s = 0; s < NP; s++) {
        const int k = act[s] ? tid + s * nt : 0;
        const int x = 2 * (k % np), y = (k / np) % (N - 1) + 1, z = k / (np * (N - 1)) + 1;
        const T e0 = lc[tail_at(M, x >> 1, y >> 1, z >> 1)];
        const T e1 = lc[tail_at(M, x >> 1, (y + 1) >> 1, (z + 1) >> 1)], e2 = lc[tail_at(M, (x >> 1) + 1, (y + 1) >> 1, (z + 1) >> 1)];
        if (lo[s]) u[s][0] += T(0.5) * (e0 + e1);
        if (act[s]) u[s][1] += T(0.5) * (e0 + e2);
    }
    __syncthreads();
    put(u);
    for (int k = 0; k < nu_post; k++) sweep();
}

// FINEST: u is read and the squared residual norm of the result goes to norm;
// else the cycle starts from zero
template <typename T, int NP, bool FINEST>
__global__ void __launch_bounds__(kTailThreads) k_grid_tail(int N, int Nc, int nu_pre, int nu_post, T h, T om, const double *st,
                                                            const T *gb, T *gu, double *norm) {
    const int tid = (int)threadIdx.x, nt = (int)blockDim.x;
    const long long P = N + 16;
    TailLds q;
    q.A = (double *)grid_lds;
    q.B = q.A + 343;
    q.S = q.B + 343;
    q.red = q.S + 56;
    T *const bl = (T *)(q.red + kTailThreads), *const lv = bl + tail_len(kTailN / 2);
    const int nc = Nc - 1;
    for (int k = tid; k < nc * nc + nc; k += nt) q.S[k] = st[k];
    T b[NP][2], u[NP][2];
    const int np = N / 2, npairs = np * (N - 1) * (N - 1);
#pragma unroll
    for (int s = 0; s < NP; s++) {
        const int k = tid + s * nt;
        const bool on = k < npairs;
        const long long i = on ? 2 * (k % np) + P * ((k / np) % (N - 1) + 1 + (long long)N * (k / (np * (N - 1)) + 1)) : 0;
        // the boundary node x = 0 holds zeros
        const Pair<T> bb = *(const Pair<T> *)(gb + i);
        b[s][0] = on ? bb.lo : T(0);
        b[s][1] = on ? bb.hi : T(0);
        u[s][0] = u[s][1] = T(0);
        if (FINEST) {
            const Pair<T> uu = *(const Pair<T> *)(gu + i);
            u[s][0] = on ? uu.lo : T(0);
            u[s][1] = on ? uu.hi : T(0);
        }
    }
    tail_level<T, NP>(N, Nc, b, u, !FINEST, h, om, nu_pre, nu_post, lv, bl, q);
    double sum = 0.0;
#pragma unroll
    for (int s = 0; s < NP; s++) {
        const int k = tid + s * nt;
        if (k >= npairs) continue;
        const int p = k % np, y = (k / np) % (N - 1) + 1, z = k / (np * (N - 1)) + 1;
        Pair<T> o;
        o.lo = u[s][0];
        o.hi = u[s][1];
        *(Pair<T> *)(gu + 2 * p + P * (y + (long long)N * z)) = o;
        if (FINEST) {
            const int i = p + (N / 2 + 1) * (y + (N + 1) * z);
#pragma unroll
            for (int e = 0; e < 2; e++) {
                if (e == 0 && p == 0) continue;
                const double r = (double)(b[s][e] - h * (T(6) * u[s][e] - tail_around(lv, N, i, ((y + z) & 1) ^ e, e, u[s][1 - e])));
                sum += r * r;
            }
        }
    }
    if (FINEST) {
        q.red[tid] = sum;
        for (int n = nt; n > 1;) {
            const int hf = (n + 1) >> 1;
            __syncthreads();
            if (tid + hf < n) q.red[tid] += q.red[tid + hf];
            n = hf;
        }
        if (tid == 0) *norm = q.red[0];
    }
}

// ---------------------------------------------------------------------------
// vector order <-> grid: a wavefront per row
// ---------------------------------------------------------------------------
__global__ void __launch_bounds__(256) k_grid_from_user(int N, const double *user, double *grid, double *partial) {
    const int n = N - 1, w = (int)(threadIdx.x >> 6), lane = (int)(threadIdx.x & 63);
    const long long row = (long long)blockIdx.x * 4 + w;
    double sum = 0.0;
    if (row < (long long)n * n) {
        const int y = (int)(row % n), z = (int)(row / n);
        const double *s = user + row * n;
        double *d = grid + (long long)(N + 16) * (y + 1 + (long long)N * (z + 1)) + 1;
        for (int x = lane; x < n; x += 64) {
            const double v = s[x];
            d[x] = v;
            sum += v * v;
        }
    }
    if (partial) block_partial(sum, partial);
}

__global__ void __launch_bounds__(256) k_grid_to_user(int N, const double *grid, double *user) {
    const int n = N - 1, w = (int)(threadIdx.x >> 6), lane = (int)(threadIdx.x & 63);
    const long long row = (long long)blockIdx.x * 4 + w;
    if (row >= (long long)n * n) return;
    const int y = (int)(row % n), z = (int)(row / n);
    const double *s = grid + (long long)(N + 16) * (y + 1 + (long long)N * (z + 1)) + 1;
    double *d = user + row * n;
    for (int x = lane; x < n; x += 64) d[x] = s[x];
}

// ---------------------------------------------------------------------------
// y = M x with the unit cube's consistent P1 mass matrix: 0.4 h^3 on the
// diagonal, h^3/20 to the 6 axis neighbours and to +-(1,1,1), h^3/30 to
// +-(1,1,0), +-(0,1,1), +-(1,0,1)
// ---------------------------------------------------------------------------
// A workgroup marches through vz planes of a tile of 64 x 16 nodes (62 x 14
// of them its own), each thread with one column; a plane's 7 values around a
// node serve the node itself and the nodes above and below it, so a plane is
// read once and published once.  The sums over the neighbours are carried
// unweighted, so each weight multiplies once.  IG, OG: input, output on the
// grid instead of in vector order.
constexpr int kMassX = 64, kMassY = 16;
template <bool IG, bool OG>
__global__ void __launch_bounds__(1024) k_grid_mass(int N, int vz, double h3, const double *in, double *out, double *partial) {
    double *const lds = (double *)grid_lds;  // [2][(kMassY + 2) kMassX + 2]
    constexpr int LS = (kMassY + 2) * kMassX + 2;
    const int ntx = (N - 1 + kMassX - 3) / (kMassX - 2), nty = (N - 1 + kMassY - 3) / (kMassY - 2);
    const unsigned f = grid_xcd(blockIdx.x, gridDim.x);
    const int ix = (int)(f % ntx), iy = (int)((f / ntx) % nty), iz = (int)(f / (ntx * nty));
    const int lx = (int)(threadIdx.x & (kMassX - 1)), ly = (int)(threadIdx.x / kMassX);
    const int x = ix * (kMassX - 2) + lx, y = iy * (kMassY - 2) + ly;  // grid coordinates
    const int Z0 = 1 + iz * vz, Z1 = min(N, Z0 + vz);
    const bool in_xy = x >= 1 && x < N && y >= 1 && y < N;
    const bool own = in_xy && lx >= 1 && lx < kMassX - 1 && ly >= 1 && ly < kMassY - 1;
    const int n = N - 1;
    const long long SI = IG ? (long long)(N + 16) * N : (long long)n * n, SO = OG ? (long long)(N + 16) * N : (long long)n * n;
    const long long oi = !in_xy ? 0 : IG ? x + (long long)(N + 16) * y : (x - 1) + (long long)n * (y - 1);
    const long long oo = !in_xy ? 0 : OG ? x + (long long)(N + 16) * y : (x - 1) + (long long)n * (y - 1);
    const int li = (ly + 1) * kMassX + lx + 1;
    const double wc = 0.4 * h3, wax = h3 / 20.0, wfd = h3 / 30.0;
    auto load = [&](int z) -> double {
        const bool ok = in_xy && z >= 1 && z < N;
        const double v = in[(ok ? oi : 0) + (ok ? (long long)(IG ? z : z - 1) * SI : 0)];
        return ok ? v : 0.0;
    };
    // node of plane z - 1: its value v1 and the sums so far of its axis and body
    // diagonal neighbours (ax) and of its face diagonal ones (fd); of plane
    // z - 1 itself, what the node above takes: v1, x - 1 and y - 1 (fm), mm1
    double v1 = 0.0, ax = 0.0, fd = 0.0, fm = 0.0, mm1 = 0.0;
    double a0 = load(Z0 - 1), a1 = load(Z0), sum = 0.0;
    for (int z = Z0 - 1; z <= Z1; z++) {
        const double v = a0;
        a0 = a1;
        a1 = load(z + 2);
        double *l = lds + (z & 1) * LS + li;
        l[0] = v;
        __syncthreads();
        const double xp = l[1], xm = l[-1], yp = l[kMassX], ym = l[-kMassX], pp = l[kMassX + 1], mm = l[-kMassX - 1];
        if (own && z > Z0) {
            const double o = wc * v1 + (wax * (ax + (v + pp)) + wfd * (fd + (xp + yp)));
            out[oo + (long long)(OG ? z - 1 : z - 2) * SO] = o;
            sum += o * o;
        }
        ax = ((xp + xm) + (yp + ym)) + (v1 + mm1);
        fd = (pp + mm) + fm;
        fm = xm + ym;
        mm1 = mm;
        v1 = v;
    }
    if (partial) {
        __syncthreads();
        block_partial(sum, partial);
    }
}

// ---------------------------------------------------------------------------
// edge weights: (h/6) times the sum of k over the 6 elements whose axis path
// holds the edge; zero at edges with an end outside the interior's
// neighbourhood (never read)
// ---------------------------------------------------------------------------
template <int A, typename F>
__device__ __forceinline__ double edge_sum(int N, int x, int y, int z, F element) {
    constexpr int kP[6][3] = {{0, 1, 2}, {0, 2, 1}, {1, 0, 2}, {1, 2, 0}, {2, 0, 1}, {2, 1, 0}};
    double s = 0.0;
#pragma unroll
    for (int d = 0; d < 8; d++) {
        const int dl[3] = {d & 1, (d >> 1) & 1, (d >> 2) & 1};
        if (dl[A]) continue;
        const int ns = dl[0] + dl[1] + dl[2];
        const long long cell = (x - dl[0]) + (long long)N * ((y - dl[1]) + (long long)N * (z - dl[2]));
#pragma unroll
        for (int q = 0; q < 6; q++) {
            if (kP[q][ns] != A || (ns > 0 && !dl[kP[q][0]]) || (ns > 1 && !dl[kP[q][1]])) continue;
            s += element(cell, x - dl[0], y - dl[1], z - dl[2], kP[q], q);
        }
    }
    return s;
}
// the weights v of the edges from a node along x, y and z; element: value of
// an element of an edge (its cell's index and position, its axis order and
// number), summed in a fixed order
template <typename F>
__device__ __forceinline__ void node_edges(int N, int x, int y, int z, double (&v)[3], F element) {
    const bool xi = x >= 1 && x < N, yi = y >= 1 && y < N, zi = z >= 1 && z < N;
    v[0] = x < N && yi && zi ? edge_sum<0>(N, x, y, z, element) : 0.0;
    v[1] = y < N && xi && zi ? edge_sum<1>(N, x, y, z, element) : 0.0;
    v[2] = z < N && xi && yi ? edge_sum<2>(N, x, y, z, element) : 0.0;
}
__global__ void __launch_bounds__(256) k_grid_weights(int N, double h, const double *k, double *w, float *w32, long long ws) {
    const int x = (int)(blockIdx.x * 64 + (threadIdx.x & 63)), y = (int)(blockIdx.y * 4 + (threadIdx.x >> 6)), z = (int)blockIdx.z;
    if (x >= N || y >= N) return;
    const long long i = grid_weight(N, ws, x, y, z);
    double v[3];
    node_edges(N, x, y, z, v, [&](long long cell, int, int, int, const int *, int q) { return k[6 * cell + q]; });
#pragma unroll
    for (int a = 0; a < 3; a++) {
        const double e = v[a] * h / 6.0;
        w[a * ws + i] = e;
        if (w32) w32[a * ws + i] = (float)e;
    }
}

// dJ/dk of the 6 elements of a cell; the grid holds the Dirichlet zeros
__global__ void __launch_bounds__(256) k_grid_grad_k(int N, double h, const double *u, const double *lam, double *out) {
    const long long cell = blockIdx.x * 256LL + threadIdx.x;
    if (cell >= (long long)N * N * N) return;
    const int cx = (int)(cell % N), cy = (int)((cell / N) % N), cz = (int)(cell / ((long long)N * N));
    const long long P = N + 16, S = P * N, i = cx + P * cy + S * cz;
    double uc[8], lc[8];
#pragma unroll
    for (int d = 0; d < 8; d++) {
        const long long q = i + (d & 1) + ((d & 2) ? P : 0) + ((d & 4) ? S : 0);
        uc[d] = u[q];
        lc[d] = lam[q];
    }
    constexpr int kP[6][3] = {{0, 1, 2}, {0, 2, 1}, {1, 0, 2}, {1, 2, 0}, {2, 0, 1}, {2, 1, 0}};
#pragma unroll
    for (int q = 0; q < 6; q++) {
        int v = 0;
        double g = 0.0;
#pragma unroll
        for (int s = 0; s < 3; s++) {
            const int w = v | (1 << kP[q][s]);
            g += (lc[v] - lc[w]) * (uc[v] - uc[w]);
            v = w;
        }
        out[6 * cell + q] = -(h / 6.0) * g;
    }
}

// ---------------------------------------------------------------------------
// slot space <-> grid, and the nodes of single tetrahedra
// ---------------------------------------------------------------------------
// tetinfo: subcube corner V (3), first two axes a, b; closure node (i, j, k)
// at m V + i e_a + j (e_a + e_b) + k (1, 1, 1)
struct GNode {
    int x, y, z;
    long long w;  // weight slot
    int tet;
};
__device__ __forceinline__ bool closure_node(const GridClosures &c, GNode &o) {
    const unsigned per = ((unsigned)c.nlist + 255u) >> 8;
    const unsigned f = grid_xcd(blockIdx.x, gridDim.x);
    const int v = (int)(f / per), e = (int)((f % per) * 256 + threadIdx.x);
    if (e >= c.nlist) return false;
    const unsigned w = c.list[e];
    const int i = (int)(w & 1023u), j = (int)((w >> 10) & 1023u), k = (int)(w >> 20);
    const VolDesc d = c.vd[v];
    const int *ti = c.tetinfo + 6 * d.tet;
    const int m = c.M - 1;
    int X[3] = {m * ti[0] + k, m * ti[1] + k, m * ti[2] + k};
    const int a = ti[3], b = ti[4];
#pragma unroll
    for (int q = 0; q < 3; q++) X[q] += (q == a ? i + j : 0) + (q == b ? j : 0);
    o.x = X[0];
    o.y = X[1];
    o.z = X[2];
    o.tet = d.tet;
    const int2 r = c.rowC[k * c.M - ((k * (k - 1)) >> 1) + j];
    o.w = d.w + (((i + k) & 1) ? r.y : r.x) + (i >> 1);
    return true;
}

// Grid <-> closures of single tetrahedra.  Slots run along the tetrahedron's
// first axis a, the grid along x: where the two differ a wavefront takes
// patches of 8 nodes along x by 8 along a, so that both sides move 64-byte
// pieces (a node list in slot order reads one 8-byte word of every line).
// Loads and stores are marked as used once: lines that stay in the L2 of the
// XCD that converts them slow the local cycles, which go over these vectors
// from other XCDs (cycle of one tetrahedron at m = 128: 116 to 120 us after
// plain accesses, 110 to 114 after these, 108 with no conversion before).
// TO: grid -> u (interior nodes as told) and, if gb is given, the interior of b.
// A wavefront has four independent pieces in flight: of a row of the grid, or
// of a patch along a.
constexpr int kClosureSteps = 4, kClosurePatch = 8 * kClosureSteps;
__host__ __device__ constexpr int closure_waves(int M) {
    const int rows = M * M, patches = M * ((M + 7) / 8) * ((M + kClosurePatch - 1) / kClosurePatch);
    return rows > patches ? rows : patches;
}
// a value that is the same in every lane of a wavefront
#if __has_builtin(__builtin_amdgcn_readfirstlane)
__device__ __forceinline__ int wave_uniform(int v) { return __builtin_amdgcn_readfirstlane(v); }
#else
__device__ __forceinline__ int wave_uniform(int v) { return v; }
#endif
#if __has_builtin(__builtin_nontemporal_load)
__device__ __forceinline__ double load_once(const double *p) { return __builtin_nontemporal_load(p); }
__device__ __forceinline__ void store_once(double *p, double v) { __builtin_nontemporal_store(v, p); }
#else
__device__ __forceinline__ double load_once(const double *p) { return *p; }
__device__ __forceinline__ void store_once(double *p, double v) { *p = v; }
#endif
template <bool TO>
__global__ void __launch_bounds__(256) k_grid_closures(GridLocal c, int interior, const double *gu, double *u, const double *gb,
                                                       double *b, double *grid) {
    const int M = c.M, m = M - 1, waves = closure_waves(M), lane = (int)(threadIdx.x & 63);
    const int wv = wave_uniform((int)(blockIdx.x * 4 + (threadIdx.x >> 6))), t = wv / waves, w = wv - t * waves;
    if (t >= c.tets.n) return;
    const int V0 = c.tets.info[t][0], V1 = c.tets.info[t][1], V2 = c.tets.info[t][2], ax = c.tets.info[t][3], bx = c.tets.info[t][4];
    const int P = c.N + 16, S = P * c.N;  // (offsets within a subcube fit 32 bits)
    const int pa = ax == 0 ? 1 : ax == 1 ? P : S, pb = bx == 0 ? 1 : bx == 1 ? P : S, pc = ax + bx == 3 ? 1 : ax + bx == 2 ? P : S;
    // pieces: nodes (A, db, dc) along the axes a, b, c
    int a0, db, dc, rounds = 1;
    if (ax == 0) {  // a row along x
        if (w >= M * M) return;
        const int y = w % M, z = w / M;
        db = bx == 1 ? y : z;
        dc = bx == 1 ? z : y;
        if (db < dc) return;
        a0 = db + lane;
        rounds = (m - db) / (64 * kClosureSteps) + 1;
    } else {
        const int p8 = (M + 7) / 8, q = w / p8, pn = (M + kClosurePatch - 1) / kClosurePatch, r = q / pn;
        const int x0 = 8 * (w - q * p8), x = x0 + (lane & 7);
        a0 = kClosurePatch * (q - r * pn);
        // a patch that misses the closure (m >= A >= db >= dc >= 0)
        if (r >= M || (bx == 0 ? x0 + 7 < r || a0 + kClosurePatch <= x0 : x0 > r || a0 + kClosurePatch <= r)) return;
        db = bx == 0 ? x : r;
        dc = bx == 0 ? r : x;
        a0 += 2 * (lane >> 3);
    }
    const bool row = db >= dc && db <= m, face = db == dc || dc == 0;  // face: every node of the row is on the boundary
    const int *rc = (const int *)(c.rowC + (row ? dc * M - ((dc * (dc - 1)) >> 1) + db - dc : 0));
    const int red = rc[0], black = rc[1];  // first slots of the row's nodes
    const long long g0 = m * V0 + (long long)P * (m * V1) + (long long)S * (m * V2), s0 = (long long)t * c.stride;
    for (int q = 0; q < rounds; q++, a0 += 64 * kClosureSteps) {
        double uv[kClosureSteps], bv[kClosureSteps];
        bool in[kClosureSteps], inner[kClosureSteps];
        int s[kClosureSteps], g[kClosureSteps];
#pragma unroll
        for (int e = 0; e < kClosureSteps; e++) {
            // (a patch: nodes of one colour, consecutive slots, per step)
            const int A = a0 + (ax == 0 ? 64 * e : 16 * (e >> 1) + (e & 1)), i = A - db;
            in[e] = row && i >= 0 && A <= m;
            inner[e] = in[e] && !face && i > 0 && A < m;
            s[e] = (((i + dc) & 1) ? black : red) + (i >> 1);
            g[e] = A * pa + db * pb + dc * pc;
            uv[e] = bv[e] = 0.0;
            if (TO) {
                if (in[e] && (!inner[e] || interior == kInteriorCopy)) uv[e] = load_once(gu + g0 + g[e]);
                if (gb && inner[e]) bv[e] = load_once(gb + g0 + g[e]);
            } else if (inner[e]) {
                uv[e] = u[s0 + s[e]];
            }
        }
#pragma unroll
        for (int e = 0; e < kClosureSteps; e++) {
            if (TO) {
                if (in[e] && !(inner[e] && interior == kInteriorKeep)) store_once(u + s0 + s[e], uv[e]);
                if (gb && inner[e]) store_once(b + s0 + s[e], bv[e]);
            } else if (inner[e]) {
                store_once(grid + g0 + g[e], uv[e]);
            }
        }
    }
}

// per-element k: a node's three edges along its tetrahedron's axes, gathered
// from the grid's weights
__global__ void __launch_bounds__(256) k_grid_closure_weights(GridClosures c, const double *w, long long ws, double *w0, double *w1,
                                                              double *w2) {
    GNode o;
    if (!closure_node(c, o)) return;
    const bool in[3] = {o.x >= 1 && o.x < c.N, o.y >= 1 && o.y < c.N, o.z >= 1 && o.z < c.N};
    const bool has[3] = {o.x < c.N && in[1] && in[2], o.y < c.N && in[0] && in[2], o.z < c.N && in[0] && in[1]};
    const long long i = grid_weight(c.N, ws, min(o.x, c.N - 1), min(o.y, c.N - 1), min(o.z, c.N - 1));
    const double v[3] = {has[0] ? w[i] : 0.0, has[1] ? w[ws + i] : 0.0, has[2] ? w[2 * ws + i] : 0.0};
    const int *ti = c.tetinfo + 6 * o.tet;
    const int a = ti[3], b = ti[4], d = ti[5];
    w0[o.w] = a == 0 ? v[0] : a == 1 ? v[1] : v[2];
    w1[o.w] = b == 0 ? v[0] : b == 1 ? v[1] : v[2];
    w2[o.w] = d == 0 ? v[0] : d == 1 ? v[1] : v[2];
}
__global__ void __launch_bounds__(256) k_grid_master_weights(int n, const int *xyz, int N, const double *w, long long ws, double *wi) {
    const int t = (int)(blockIdx.x * 256 + threadIdx.x);
    if (t >= n) return;
    const int x = xyz[3 * t], y = xyz[3 * t + 1], z = xyz[3 * t + 2];  // an interior node
    const long long o = grid_weight(N, ws, x, y, z), m = n;
    wi[t] = w[o];
    wi[m + t] = w[grid_weight(N, ws, x - 1, y, z)];
    wi[2 * m + t] = w[ws + o];
    wi[3 * m + t] = w[ws + grid_weight(N, ws, x, y - 1, z)];
    wi[4 * m + t] = w[2 * ws + o];
    wi[5 * m + t] = w[2 * ws + grid_weight(N, ws, x, y, z - 1)];
}

// the intact side of a Dirichlet-Neumann recovery (eq. (5)): edge weights over
// the elements of intact tetrahedra; only edges in the closures of faulty ones
// lose any
__global__ void __launch_bounds__(256) k_grid_intact_weights(GridClosures c, int n_sub, double h, const double *k,
                                                             const unsigned char *faulty, double *w, unsigned char *code,
                                                             long long ws) {
    GNode o;
    if (!closure_node(c, o) || o.x >= c.N || o.y >= c.N || o.z >= c.N) return;
    const int m = c.M - 1;
    double v[3];
    node_edges(c.N, o.x, o.y, o.z, v, [&](long long cell, int cx, int cy, int cz, const int *p, int q) {
        const bool out = faulty && faulty[macro_tet_of(cx, cy, cz, p[0], p[1], p[2], m, n_sub)];
        return out ? 0.0 : w ? k[6 * cell + q] : 1.0;
    });
    const long long i = grid_weight(c.N, ws, o.x, o.y, o.z);
#pragma unroll
    for (int a = 0; a < 3; a++) {
        if (w)
            w[a * ws + i] = v[a] * h / 6.0;
        else
            code[a * ws + i] = (unsigned char)v[a];
    }
}
__global__ void __launch_bounds__(256) k_grid_neumann(int n, const int *xyz, int N, const double *wi, const unsigned char *gamma,
                                                      const double *u, double *b, double *save) {
    const int t = (int)(blockIdx.x * 256 + threadIdx.x);
    if (t >= n || !gamma[t]) return;
    const long long P = N + 16, S = P * N, m = n;
    const long long i = xyz[3 * t] + P * xyz[3 * t + 1] + S * xyz[3 * t + 2];
    const double uo = u[i];
    double s = 0.0;
    s += wi[t] * (uo - u[i + 1]);
    s += wi[m + t] * (uo - u[i - 1]);
    s += wi[2 * m + t] * (uo - u[i + P]);
    s += wi[3 * m + t] * (uo - u[i - P]);
    s += wi[4 * m + t] * (uo - u[i + S]);
    s += wi[5 * m + t] * (uo - u[i - S]);
    save[t] = b[i];
    b[i] = s;
}
__global__ void __launch_bounds__(256) k_grid_neumann_end(int n, const int *xyz, int N, const unsigned char *gamma, const double *save,
                                                          double *b) {
    const int t = (int)(blockIdx.x * 256 + threadIdx.x);
    if (t < n && gamma[t]) b[xyz[3 * t] + (long long)(N + 16) * (xyz[3 * t + 1] + (long long)N * xyz[3 * t + 2])] = save[t];
}
__global__ void __launch_bounds__(256) k_grid_freeze_masters(int n, const int *xyz, int N, const unsigned char *frozen,
                                                             unsigned char *frz) {
    const int t = (int)(blockIdx.x * 256 + threadIdx.x);
    if (t < n && frozen[t]) frz[xyz[3 * t] + (long long)(N + 16) * (xyz[3 * t + 1] + (long long)N * xyz[3 * t + 2])] = 1;
}

// nodes of the listed tetrahedra: strictly inside them (zeroed, or frozen) or
// their closures (frozen).  A wavefront per grid row of the tetrahedron's
// subcube walks the row's nodes of the tetrahedron, an interval along x.
constexpr int kTetsZero = 0, kTetsFreeze = 1, kTetsFreezeInside = 2;
template <int MODE>
__global__ void __launch_bounds__(256) k_grid_tets(int N, int m, GridTets t, double *grid, unsigned char *frz) {
    const int w = m + 1, per = (w * w + 3) / 4;
    const int q = (int)(blockIdx.x / per), row = (int)(blockIdx.x % per) * 4 + (int)(threadIdx.x >> 6);
    if (row >= w * w) return;
    const int dy = row % w, dz = row / w;
    int V[3] = {0, 0, 0}, a = 0, b = 0;
#pragma unroll
    for (int r = 0; r < 8; r++)
        if (r == q) {
            V[0] = t.info[r][0];
            V[1] = t.info[r][1];
            V[2] = t.info[r][2];
            a = t.info[r][3];
            b = t.info[r][4];
        }
    // d[a] >= d[b] >= d[c]; inside: all bounds strict by one
    constexpr int e = MODE == kTetsFreeze ? 0 : 1;
    const int c = 3 - a - b;
    const int db = b == 1 ? dy : dz, dc = c == 1 ? dy : dz, da = a == 1 ? dy : dz;
    int lo, hi;
    bool some;
    if (a == 0) {
        lo = db + e;
        hi = m - e;
        some = db >= dc + e && dc >= e;
    } else if (b == 0) {
        lo = dc + e;
        hi = da - e;
        some = da <= m - e && dc >= e;
    } else {
        lo = e;
        hi = db - e;
        some = da >= db + e && da <= m - e;
    }
    const int Y = m * V[1] + dy, Z = m * V[2] + dz, X0 = m * V[0];
    // the boundary nodes x = N and y = N have no place of their own
    if (!some || Y >= N) return;
    const long long i = X0 + (long long)(N + 16) * (Y + (long long)N * Z);
    for (int x = lo + (int)(threadIdx.x & 63); x <= hi; x += 64) {
        if (X0 + x >= N) break;
        if (MODE == kTetsZero)
            grid[i + x] = 0.0;
        else
            frz[i + x] = 1;
    }
}
__global__ void __launch_bounds__(256) k_grid_zero32(unsigned *p, long long n) {
    for (long long q = blockIdx.x * 256LL + threadIdx.x; q < n; q += 256LL * gridDim.x) p[q] = 0u;
}

size_t sweep_lds(const GridTiles &t, int ns, int start, int tail, int word) {
    const int threads = grid_threads(t);
    const size_t rows = (size_t)(threads + t.tp - 1) / t.tp + 2;
    if (tail == kGridResidual)
        return std::max(2 * (rows * t.tp + 2) * 2 * sizeof(double), threads * sizeof(double));
    const int K = 2 * ns, NL = K + (tail != kGridPlain) - (start == kGridFromZero);
    size_t n = (size_t)NL * 2 * (rows * t.tp + 2);
    if (tail == kGridRestrict) n += 3 * (rows * 2 * t.tp + 2);
    size_t by = n * word;
    if (tail == kGridNorm) by = std::max(by, (size_t)threads * sizeof(double));
    return by;
}

int cdiv(int a, int b) { return (a + b - 1) / b; }

}  // namespace

GridTiles grid_tiles_of(int N, int ns, int tail, int vp, int vy, int vz) {
    const int np = N / 2, hl = halo_lo(2 * ns, tail), hh = halo_hi(2 * ns, tail);
    GridTiles t;
    t.vp = std::min(vp, np);
    t.vy = std::min((vy + 1) & ~1, N);
    t.vz = std::min((vz + 1) & ~1, N);
    t.ntx = cdiv(np, t.vp);
    t.nty = cdiv(N, t.vy);
    t.ntz = cdiv(N, t.vz);
    // the halo ends at the boundary nodes x = 0 and x = N (pair np)
    for (int i = 0; i < t.ntx; i++) {
        const int a = std::max(0, i * t.vp - (hl + 1) / 2);
        const int b = std::min(np + 1, std::min(np, (i + 1) * t.vp) + (hh + 1) / 2);
        t.tp = std::max(t.tp, b - a);
    }
    for (int i = 0; i < t.nty; i++) {
        const int a = std::max(0, i * t.vy - hl), b = std::min(N + 1, std::min(N, (i + 1) * t.vy) + hh);
        t.ty = std::max(t.ty, b - a);
    }
    return t;
}

namespace {

template <typename T, int NS, int START, int TAIL>
void sweep_mask(hipStream_t s, const GridTiles &t, const GridSweep<T> &g) {
    const size_t lds = sweep_lds(t, NS, START, TAIL, (int)sizeof(T));
    const T h = (T)g.h, om = (T)(g.omega / (6.0 * g.h)), omr = (T)(1.0 - g.omega);
    const dim3 grid((unsigned)t.blocks()), block((unsigned)grid_threads(t));
    if constexpr (NS == 1) {
        if (g.w) {
            if (g.frz)
                hipLaunchKernelGGL((k_grid_sweep<T, 1, START, TAIL, true, kEdgeWeights>), grid, block, lds, s, g, t, h, (T)g.omega, omr);
            else
                hipLaunchKernelGGL((k_grid_sweep<T, 1, START, TAIL, false, kEdgeWeights>), grid, block, lds, s, g, t, h, (T)g.omega, omr);
            return;
        }
        if constexpr (sizeof(T) == 8 && TAIL != kGridNorm) {
            if (g.code) {
                hipLaunchKernelGGL((k_grid_sweep<T, 1, START, TAIL, true, kEdgeCodes>), grid, block, lds, s, g, t, h, (T)g.omega, omr);
                return;
            }
        }
    }
    if (g.frz)
        hipLaunchKernelGGL((k_grid_sweep<T, NS, START, TAIL, true, kEdgeUniform>), grid, block, lds, s, g, t, h, om, omr);
    else
        hipLaunchKernelGGL((k_grid_sweep<T, NS, START, TAIL, false, kEdgeUniform>), grid, block, lds, s, g, t, h, om, omr);
}

template <typename T>
void sweep_any(hipStream_t s, int ns, int start, int tail, const GridTiles &t, const GridSweep<T> &g) {
    const bool rt = tail == kGridRestrict;
    if (start == kGridFromZero && ns == 2)
        rt ? sweep_mask<T, 2, kGridFromZero, kGridRestrict>(s, t, g) : sweep_mask<T, 2, kGridFromZero, kGridPlain>(s, t, g);
    else if (start == kGridFromZero)
        rt ? sweep_mask<T, 1, kGridFromZero, kGridRestrict>(s, t, g) : sweep_mask<T, 1, kGridFromZero, kGridPlain>(s, t, g);
    else if constexpr (sizeof(T) == 8) {
        if (start == kGridProlong)
            tail == kGridNorm ? sweep_mask<T, 1, kGridProlong, kGridNorm>(s, t, g) : sweep_mask<T, 1, kGridProlong, kGridPlain>(s, t, g);
        else if (tail == kGridNorm)
            sweep_mask<T, 1, kGridFromU, kGridNorm>(s, t, g);
        else
            rt ? sweep_mask<T, 1, kGridFromU, kGridRestrict>(s, t, g) : sweep_mask<T, 1, kGridFromU, kGridPlain>(s, t, g);
    } else {
        if (start == kGridProlong)
            sweep_mask<T, 1, kGridProlong, kGridPlain>(s, t, g);
        else
            rt ? sweep_mask<T, 1, kGridFromU, kGridRestrict>(s, t, g) : sweep_mask<T, 1, kGridFromU, kGridPlain>(s, t, g);
    }
}

void residual_any(hipStream_t s, const GridTiles &t, const GridResidual &g) {
    const size_t lds = sweep_lds(t, 0, kGridFromU, kGridResidual, 8);
    const dim3 grid((unsigned)t.blocks()), block((unsigned)grid_threads(t));
    auto run = [&](auto kernel) { hipLaunchKernelGGL(kernel, grid, block, lds, s, g, t); };
    if (g.w) {
        if (g.e)
            g.frz ? run(k_grid_residual<true, true, true>) : run(k_grid_residual<true, false, true>);
        else
            g.frz ? run(k_grid_residual<false, true, true>) : run(k_grid_residual<false, false, true>);
    } else if (g.e) {
        g.frz ? run(k_grid_residual<true, true, false>) : run(k_grid_residual<true, false, false>);
    } else {
        g.frz ? run(k_grid_residual<false, true, false>) : run(k_grid_residual<false, false, false>);
    }
}

dim3 node_blocks(int N) { return dim3((unsigned)cdiv(N - 1, 64), (unsigned)cdiv(N - 1, 4), (unsigned)(N - 1)); }

template <typename T>
void plain_residual(hipStream_t s, int N, double h, const T *u, const T *b, const T *w, long long ws, T *r) {
    hipLaunchKernelGGL((k_grid_plain_residual<T>), node_blocks(N), dim3(256), 0, s, N, (T)h, u, b, w,
                       (const unsigned char *)nullptr, (const unsigned char *)nullptr, ws, r);
}
void plain_residual_intact(hipStream_t s, int N, double h, const double *u, const double *b, const double *w,
                           const unsigned char *code, long long ws, const unsigned char *frz, double *r) {
    hipLaunchKernelGGL((k_grid_plain_residual<double>), node_blocks(N), dim3(256), 0, s, N, h, u, b, w, code, frz, ws, r);
}
void weights(hipStream_t s, int N, double h, const double *k, double *w, float *w32, long long ws) {
    hipLaunchKernelGGL(k_grid_weights, dim3((unsigned)cdiv(N, 64), (unsigned)cdiv(N, 4), (unsigned)N), dim3(256), 0, s, N, h, k, w,
                       w32, ws);
}
template <typename T>
void plain_restrict(hipStream_t s, int N, const T *r, T *bc) {
    hipLaunchKernelGGL((k_grid_plain_restrict<T>), node_blocks(N / 2), dim3(256), 0, s, N, r, bc);
}
template <typename T>
void plain_prolong(hipStream_t s, int N, const T *u, const T *ec, T *v) {
    hipLaunchKernelGGL((k_grid_plain_prolong<T>), node_blocks(N), dim3(256), 0, s, N, u, ec, (const unsigned char *)nullptr, v);
}
void plain_prolong_intact(hipStream_t s, int N, const double *u, const double *ec, const unsigned char *frz, double *v) {
    hipLaunchKernelGGL((k_grid_plain_prolong<double>), node_blocks(N), dim3(256), 0, s, N, u, ec, frz, v);
}
template <typename T>
void coarse(hipStream_t s, int N, const double *st, const T *b, T *u) {
    const size_t lds = (2 * kSineMax * kSineMax * kSineMax + kSineMax * (kSineMax + 1)) * sizeof(double);
    hipLaunchKernelGGL((k_grid_coarse<T>), dim3(1), dim3(512), lds, s, N, st, b, u);
}
template <typename T, int NP, bool FINEST>
void tail_run(hipStream_t s, int N, int Nc, int nu_pre, int nu_post, double h, double omega, const double *st, const T *b, T *u,
              double *norm) {
    const size_t lds = (2 * 343 + 56 + kTailThreads) * sizeof(double) +
                       (tail_len(kTailN / 2) + tail_len(N) + tail_len(N / 2) + tail_len(N / 4)) * sizeof(T);
    hipLaunchKernelGGL((k_grid_tail<T, NP, FINEST>), dim3(1), dim3(kTailThreads), lds, s, N, Nc, nu_pre, nu_post, (T)h,
                       (T)(omega / (6.0 * h)), st, b, u, norm);
}
bool tail_fits(int N, int Nc) { return N <= kTailN && Nc <= 8 && N > Nc && (N / 2 == Nc || (N == kTailN && N / 4 == Nc)); }
template <typename T>
void tail_cycle(hipStream_t s, int N, int Nc, int nu_pre, int nu_post, double h, double omega, const double *st, const T *b, T *u,
                double *norm) {
    if (N > 8)
        norm ? tail_run<T, 2, true>(s, N, Nc, nu_pre, nu_post, h, omega, st, b, u, norm)
             : tail_run<T, 2, false>(s, N, Nc, nu_pre, nu_post, h, omega, st, b, u, norm);
    else
        norm ? tail_run<T, 1, true>(s, N, Nc, nu_pre, nu_post, h, omega, st, b, u, norm)
             : tail_run<T, 1, false>(s, N, Nc, nu_pre, nu_post, h, omega, st, b, u, norm);
}
int row_blocks(int N) { return (int)(((long long)(N - 1) * (N - 1) + 3) / 4); }
int from_user(hipStream_t s, int N, const double *user, double *grid, double *partial) {
    hipLaunchKernelGGL(k_grid_from_user, dim3((unsigned)row_blocks(N)), dim3(256), 256 * sizeof(double), s, N, user, grid,
                       partial);
    return row_blocks(N);
}
void to_user(hipStream_t s, int N, const double *grid, double *user) {
    hipLaunchKernelGGL(k_grid_to_user, dim3((unsigned)row_blocks(N)), dim3(256), 0, s, N, grid, user);
}
template <bool IG, bool OG>
int mass(hipStream_t s, int N, double h, const double *in, double *out, double *partial) {
    const int cols = cdiv(N - 1, kMassX - 2) * cdiv(N - 1, kMassY - 2);
    // planes per workgroup: rounds of 512 workgroups (two per CU) times the
    // steps of a march, which two planes of halo and the pipeline lengthen
    // (N = 32: 5.6 us with 4 planes, 18 with 32; N = 128: 13 with 8, 22 with 32)
    int vz = 32;
    double best = 1e300;
    for (int v = 32; v >= 4; v /= 2) {
        const double c = (double)cdiv(cols * cdiv(N - 1, v), 512) * (v + 3) * (v + 1) / v;
        if (c < best) {
            best = c;
            vz = v;
        }
    }
    const int nb = cols * cdiv(N - 1, vz);
    const size_t lds = 2 * ((kMassY + 2) * kMassX + 2) * sizeof(double);
    hipLaunchKernelGGL((k_grid_mass<IG, OG>), dim3((unsigned)nb), dim3(kMassX * kMassY), lds, s, N, vz, h * h * h, in,
                       out, partial);
    return nb;
}
int mass_load(hipStream_t s, int N, double h, const double *f, double *grid, double *partial) {
    return mass<false, true>(s, N, h, f, grid, partial);
}
void mass_user(hipStream_t s, int N, double h, const double *grid, double *user) {
    mass<true, false>(s, N, h, grid, user, nullptr);
}
unsigned closure_blocks(const GridClosures &c) { return (unsigned)(((c.nlist + 255) / 256) * c.nvol); }
dim3 closure_grid(const GridLocal &c) { return dim3((unsigned)((closure_waves(c.M) * c.tets.n + 3) / 4)); }
void to_closures(hipStream_t s, const GridLocal &c, int interior, const double *gu, double *u, const double *gb, double *b) {
    if (c.tets.n > 0)
        hipLaunchKernelGGL(k_grid_closures<true>, closure_grid(c), dim3(256), 0, s, c, interior, gu, u, gb, b, (double *)nullptr);
}
void from_closures(hipStream_t s, const GridLocal &c, const double *vec, double *grid) {
    if (c.tets.n > 0)
        hipLaunchKernelGGL(k_grid_closures<false>, closure_grid(c), dim3(256), 0, s, c, kInteriorCopy, (const double *)nullptr,
                           (double *)vec, (const double *)nullptr, (double *)nullptr, grid);
}
void closure_weights(hipStream_t s, const GridClosures &c, const double *w, long long ws, double *w0, double *w1, double *w2) {
    if (closure_blocks(c))
        hipLaunchKernelGGL(k_grid_closure_weights, dim3(closure_blocks(c)), dim3(256), 0, s, c, w, ws, w0, w1, w2);
}
void intact_weights(hipStream_t s, const GridClosures &c, int n_sub, double h, const double *k, const unsigned char *faulty, double *w,
                    unsigned char *code, long long ws) {
    if (closure_blocks(c))
        hipLaunchKernelGGL(k_grid_intact_weights, dim3(closure_blocks(c)), dim3(256), 0, s, c, n_sub, h, k, faulty, w, code, ws);
}
dim3 master_blocks(int n) { return dim3((unsigned)cdiv(n, 256)); }
void master_weights(hipStream_t s, int n, const int *xyz, int N, const double *w, long long ws, double *wi) {
    if (n > 0) hipLaunchKernelGGL(k_grid_master_weights, master_blocks(n), dim3(256), 0, s, n, xyz, N, w, ws, wi);
}
void neumann(hipStream_t s, int n, const int *xyz, int N, const double *wi, const unsigned char *gamma, const double *u, double *b,
             double *save) {
    if (n > 0) hipLaunchKernelGGL(k_grid_neumann, master_blocks(n), dim3(256), 0, s, n, xyz, N, wi, gamma, u, b, save);
}
void neumann_end(hipStream_t s, int n, const int *xyz, int N, const unsigned char *gamma, const double *save, double *b) {
    if (n > 0) hipLaunchKernelGGL(k_grid_neumann_end, master_blocks(n), dim3(256), 0, s, n, xyz, N, gamma, save, b);
}
void grad_k(hipStream_t s, int N, double h, const double *u, const double *lam, double *out) {
    hipLaunchKernelGGL(k_grid_grad_k, dim3((unsigned)(((long long)N * N * N + 255) / 256)), dim3(256), 0, s, N, h, u, lam, out);
}
template <int MODE>
void tets(hipStream_t s, int N, int m, const GridTets &t, double *grid, unsigned char *frz) {
    const unsigned per = (unsigned)(((m + 1) * (m + 1) + 3) / 4);
    if (t.n > 0) hipLaunchKernelGGL((k_grid_tets<MODE>), dim3(per * t.n), dim3(256), 0, s, N, m, t, grid, frz);
}
void zero_tets(hipStream_t s, int N, int m, const GridTets &t, double *grid) {
    tets<kTetsZero>(s, N, m, t, grid, nullptr);
}
void freeze_none(hipStream_t s, int N, unsigned char *frz) {
    hipLaunchKernelGGL(k_grid_zero32, dim3(1024), dim3(256), 0, s, (unsigned *)frz, (grid_len(N) + 3) / 4);
}
void freeze_tets(hipStream_t s, int N, int m, const GridTets &t, unsigned char *frz) {
    freeze_none(s, N, frz);
    tets<kTetsFreeze>(s, N, m, t, nullptr, frz);
}
void freeze_inside(hipStream_t s, int N, int m, const GridTets &t, int n, const int *xyz, const unsigned char *frozen,
                   unsigned char *frz) {
    freeze_none(s, N, frz);
    tets<kTetsFreezeInside>(s, N, m, t, nullptr, frz);
    if (n > 0) hipLaunchKernelGGL(k_grid_freeze_masters, master_blocks(n), dim3(256), 0, s, n, xyz, N, frozen, frz);
}

// Tile choice.  The time of a launch is modelled as the larger of two bounds
// plus a part of the smaller; the constants are a fit to 400 measured launches
// (N = 16 .. 512, every kind, FP64), whose fastest tiles the model misses by
// 1 % on average:
//   memory: what the tiles read, halo and partial lines at row ends included,
//     at 8.8 TB/s (halo reads hit in L2 in part) and the own nodes written at
//     4 TB/s; large grids need about 860 threads resident per CU for that;
//   latency: a step of the march costs 0.2 to 0.6 us (barrier, LDS reads, the
//     chain of passes), more with more threads on the CU, so small grids take
//     thin tiles on many CUs.  A residual with edge weights waits for them in
//     every step, 0.7 to 0.9 us (N = 64, 96, 128: 5.5, 11 and 21 us, against
//     9, 18 and 32 with the tiles of a plain residual's step).
// At N = 256 a plain sweep takes 91 us, at N = 512 680.
GridTiles tiles(int N, int ns, int start, int tail, int word, bool vk) {
    const int K = tail == kGridResidual ? 0 : 2 * ns, np = N / 2;
    const int hl = halo_lo(K, tail), hh = halo_hi(K, tail);
    const double wr = (double)N * N * N * word / 4.0e6;
    // registers: 128 at two sweeps or with a tail, fewer otherwise
    const int cap = vk ? 768 : ns >= 2 || tail == kGridRestrict || tail == kGridNorm ? 1024 : 1536;
    const int most = vk ? kVkThreads : 1024;
    // words read per pair: u and b (from zero: b), and three edge weights
    const double words = (start == kGridFromZero ? 2 : 4) + (vk ? 6 : 0);
    GridTiles best;
    double bc = 1e300;
    for (int ntx = 1, vp0 = 0; ntx <= np; ntx++) {
        const int vp = cdiv(np, ntx);
        if (vp == vp0) continue;
        vp0 = vp;
        if (vp < 4 && ntx > 1) break;
        for (int nty = 1, vy0 = 0; nty <= N / 2; nty++) {
            const int vy = (cdiv(N, nty) + 1) & ~1;
            if (vy == vy0) continue;
            vy0 = vy;
            GridTiles t = grid_tiles_of(N, ns, tail, vp, vy, N);
            const int th = grid_threads(t);
            if (th > most) continue;
            const size_t lds = sweep_lds(t, ns, start, tail, word);
            if (lds > (size_t)160 * 1024) continue;
            const int bpc = std::max(1, std::min({cap / th, (int)((size_t)160 * 1024 / lds), 8}));
            for (int ntz = 1, vz0 = 0; ntz <= N / 2; ntz++) {
                const int vz = (cdiv(N, ntz) + 1) & ~1;
                if (vz == vz0) continue;
                vz0 = vz;
                t.vz = vz;
                t.ntz = cdiv(N, vz);
                const int blocks = t.blocks(), rounds = cdiv(blocks, 256 * bpc), res = std::min(bpc, cdiv(blocks, 256));
                const double step = (K == 0 && vk ? 0.42 : 0.11) + 0.115 * K + (0.12 + 0.19 * K) * 1e-3 * th * res;
                const double lat = rounds * (vz + hl + K + 3) * step * (vk ? 1.6 : 1.0);
                double bw = wr + (double)blocks * (vz + hl + hh) * t.tp * t.ty * words * word * (1.0 + 60.0 / (2 * word * t.tp)) / 8.8e6;
                const double active = (double)blocks * th / (256.0 * rounds);  // threads resident per CU on average
                if (bw > 30.0) bw *= std::max(1.0, 860.0 / active);
                const double cost = std::max(lat, bw) + 0.18 * std::min(lat, bw);
                if (cost < bc) {
                    bc = cost;
                    best = t;
                }
            }
        }
    }
    return best;
}

const GridOps kOps = {tiles,
                      sweep_any<double>,
                      sweep_any<float>,
                      residual_any,
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
                      launch_coarse_pcg_sine<double>,
                      launch_coarse_pcg_sine<float>,
                      tail_fits,
                      tail_cycle<double>,
                      tail_cycle<float>,
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

}  // namespace

int grid_threads(const GridTiles &t) { return (t.tp * t.ty + 63) & ~63; }

const GridOps *grid_ops() { return &kOps; }

// b = M f, both in vector order
void launch_mass_grid(hipStream_t s, int N, double h, const double *f, double *b) {
    mass<false, false>(s, N, h, f, b, nullptr);
}

}  // namespace hhgr
