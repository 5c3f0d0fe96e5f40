// Velocity ghost rules and the exact median shared by the forward and the
// adjoint Navier-Stokes kernels.
#pragma once

#include "wl_device.h"
#include "wl_ns.h"

namespace wl {

// --------------------------------------------------------- velocity ghosts

// Value of velocity component c at (i, j, k), where at most one coordinate
// lies outside the grid (by up to two cells).  Ghost rules: periodic wrap;
// INFLOW ghosts = U; free-slip WALL: normal component odd about the wall
// face (boundary face 0), tangential components even; OUTFLOW (upper x): the
// boundary face is the plane uout, ghosts beyond it zero-gradient.
template <typename T, bool ALLPER>
__device__ __forceinline__ T vget(const VelField<T>& V, int c, int i, int j, int k) {
    const Grid& g = V.g;
    if (ALLPER) {
        i = i < 0 ? i + g.n0 : (i >= g.n0 ? i - g.n0 : i);
        j = j < 0 ? j + g.n1 : (j >= g.n1 ? j - g.n1 : j);
        if (g.ndim == 3) k = k < 0 ? k + g.n2 : (k >= g.n2 ? k - g.n2 : k);
        return V.u[c][cid(g, i, j, k)];
    }
    int q[3] = {i, j, k};
    const int n[3] = {g.n0, g.n1, g.n2};
    const int per[3] = {g.per0, g.per1, g.per2};
#pragma unroll
    for (int d = 0; d < 3; ++d)
        if (per[d]) q[d] = q[d] < 0 ? q[d] + n[d] : (q[d] >= n[d] ? q[d] - n[d] : q[d]);
#pragma unroll
    for (int d = 0; d < 3; ++d) {
        const int m = n[d], kk = q[d];
        if (kk >= 0 && kk < m) continue;
        // (the other coordinates are in range for every evaluation the kernels
        // make; clamping keeps any other request inside the array)
        auto at = [&](int idx) -> T {
            int r[3] = {q[0], q[1], q[2]};
            r[d] = idx;
#pragma unroll
            for (int e = 0; e < 3; ++e) r[e] = r[e] < 0 ? 0 : (r[e] >= n[e] ? n[e] - 1 : r[e]);
            return V.u[c][cid(g, r[0], r[1], r[2])];
        };
        if (kk < 0) {
            if (V.bclo[d] == WL_BC_INFLOW) return V.U[c];
            if (c == d) {
                const int mir = -kk;
                return -at(mir < m ? mir : 0);
            }
            const int mir = -1 - kk;
            return at(mir < m - 1 ? mir : m - 1);
        }
        if (c == d) {
            if (V.bchi[d] == WL_BC_OUTFLOW) {
                const int a = q[1] < 0 ? 0 : (q[1] >= g.n1 ? g.n1 - 1 : q[1]);
                const int b = q[2] < 0 ? 0 : (q[2] >= g.n2 ? g.n2 - 1 : q[2]);
                return V.uout[a + size_t(g.n1) * b];
            }
            if (kk == m) return T(0);
            return -at(m - 1 > 0 ? m - 1 : 0);
        }
        if (V.bchi[d] == WL_BC_OUTFLOW) return at(m - 1);
        if (kk == m) return at(m - 1);
        return at(m - 2 > 0 ? m - 2 : 0);
    }
    return V.u[c][cid(g, q[0], q[1], q[2])];
}

// vget without branches: one load from the address the rule picks, then a sign
// or a constant.  For the adjoint's gather, which makes 324 of these per cell
// and with the rule as branches waited for the load of each (64 x 32 x 32 in
// FP64: 314 -> 189 us with the loads of a face in flight together); the forward
// kernels make a tenth of that, where the selects cost more than the branches
// (momentum there 36 -> 49 us).
template <typename T, bool ALLPER>
__device__ __forceinline__ T vget_flat(const VelField<T>& V, int c, int i, int j, int k) {
    const Grid& g = V.g;
    if (ALLPER) return vget<T, true>(V, c, i, j, k);
    // the grid and boundary fields are uniform; through readfirstlane a choice
    // between two of them stays a choice between registers
    auto u_ = [](int v) { return __builtin_amdgcn_readfirstlane(v); };
    const int n0 = u_(g.n0), n1 = u_(g.n1), n2 = u_(g.n2);
    const bool p0 = u_(g.per0), p1 = u_(g.per1), p2 = u_(g.per2);
    if (p0) i = i < 0 ? i + n0 : (i >= n0 ? i - n0 : i);
    if (p1) j = j < 0 ? j + n1 : (j >= n1 ? j - n1 : j);
    if (p2) k = k < 0 ? k + n2 : (k >= n2 ? k - n2 : k);
    const bool o0 = unsigned(i) >= unsigned(n0), o1 = unsigned(j) >= unsigned(n1);
    const bool o2 = unsigned(k) >= unsigned(n2), out = o0 || o1 || o2;
    const int d = o0 ? 0 : (o1 ? 1 : 2);
    const int kk = o0 ? i : (o1 ? j : k), m = o0 ? n0 : (o1 ? n1 : n2);
    const bool in0 = u_(V.bclo[0]) == WL_BC_INFLOW, in1 = u_(V.bclo[1]) == WL_BC_INFLOW;
    const bool in2 = u_(V.bclo[2]) == WL_BC_INFLOW;
    const bool ex0 = u_(V.bchi[0]) == WL_BC_OUTFLOW, ex1 = u_(V.bchi[1]) == WL_BC_OUTFLOW;
    const bool ex2 = u_(V.bchi[2]) == WL_BC_OUTFLOW;
    const bool low = kk < 0, normal = c == d;
    const bool inflow = o0 ? in0 : (o1 ? in1 : in2), exits = o0 ? ex0 : (o1 ? ex1 : ex2);
    // the cell along d: mirrored below, the last one or the one before above
    const int mir = normal ? -kk : -1 - kk;
    int idx = mir < m ? mir : (normal ? 0 : m - 1);
    if (!low) idx = normal || exits || kk == m ? m - 1 : m - 2;
    idx = min(max(idx, 0), m - 1);
    const int x = o0 ? idx : i, yc = min(max(j, 0), n1 - 1), zc = min(max(k, 0), n2 - 1);
    const int y = out && d == 1 ? idx : yc, z = out && d == 2 ? idx : zc;
    const bool plane = out && !low && normal && exits;
    const T* base = plane ? V.uout : V.u[c];
    const size_t off = plane ? size_t(yc) + size_t(n1) * size_t(zc)
                             : size_t(x) + size_t(n0) * (size_t(y) + size_t(n1) * size_t(z));
    const T v = base[off];
    const bool above = out && !low && normal && !exits;  // wall: face 0, beyond it odd
    const T w = (out && low && normal && !inflow) || (above && kk != m) ? -v : v;
    return out && low && inflow ? V.U[c] : (above && kk == m ? T(0) : w);
}

// Whether the stencil of a flux through a lower d-face at (i, j, k) (two cells
// below, one above along d; the advecting pair one below along c) lies inside
// the grid for every active lane.
template <typename T>
__device__ __forceinline__ bool flux_inside(const VelField<T>& V, int c, int d, int i, int j, int k) {
    const Grid& g = V.g;
    const int li = max(d == 0 ? 2 : 0, c == 0 ? 1 : 0), lj = max(d == 1 ? 2 : 0, c == 1 ? 1 : 0);
    const int lk = max(d == 2 ? 2 : 0, c == 2 ? 1 : 0);
    const bool in = i >= li && i + (d == 0) < g.n0 && j >= lj && j + (d == 1) < g.n1 && k >= lk &&
                    k + (d == 2) < g.n2;
    return __all(in);
}

// Pressure-gradient update of one face: u - cl (p_here - p_lower) with
// cl = c dt L, one rounding (shared by the projection kernel and the
// momentum kernel that applies the predictor projection on the fly).
__device__ __forceinline__ float proj_face(float u, float cl, float ph, float pl) {
    return fmaf(-cl, ph - pl, u);
}
__device__ __forceinline__ double proj_face(double u, double cl, double ph, double pl) {
    return fma(-cl, ph - pl, u);
}

__device__ __forceinline__ float med3(float a, float b, float c) {
    return __builtin_amdgcn_fmed3f(a, b, c);
}
__device__ __forceinline__ double med3(double a, double b, double c) {
    return fmax(fmin(a, b), fmin(fmax(a, b), c));
}

}  // namespace wl
