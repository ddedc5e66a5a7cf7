// Device helpers on the cube's elements that several kernel files share.
#pragma once

namespace hhgr {

__device__ __forceinline__ int perm_id(int a, int b) { return a == 0 ? (b == 1 ? 0 : 1) : a == 1 ? (b == 0 ? 2 : 3) : (b == 0 ? 4 : 5); }

// The fine element of cell (cx, cy, cz) with axis order p0, p1, p2, at a level
// with m segments per macro edge, lies in the macro tetrahedron of macro cell
// c / m whose axis order sorts the element's centroid offsets in that macro cell.
__device__ __forceinline__ int macro_tet_of(int cx, int cy, int cz, int p0, int p1, int p2, int m, int n_sub) {
    const int C0 = cx / m, C1 = cy / m, C2 = cz / m;
    // centroid offsets in quarter units: 3, 2, 1 along the element's axes p0, p1, p2
    const int D0 = 4 * (cx - m * C0) + (p0 == 0 ? 3 : p1 == 0 ? 2 : 1);
    const int D1 = 4 * (cy - m * C1) + (p0 == 1 ? 3 : p1 == 1 ? 2 : 1);
    const int D2 = 4 * (cz - m * C2) + (p0 == 2 ? 3 : p1 == 2 ? 2 : 1);
    const int a0 = D0 > D1 ? (D0 > D2 ? 0 : 2) : (D1 > D2 ? 1 : 2);
    const int a2 = D0 < D1 ? (D0 < D2 ? 0 : 2) : (D1 < D2 ? 1 : 2);
    const int a1 = 3 - a0 - a2;
    return 6 * (C0 + n_sub * (C1 + n_sub * C2)) + perm_id(a0, a1);
}

}  // namespace hhgr
