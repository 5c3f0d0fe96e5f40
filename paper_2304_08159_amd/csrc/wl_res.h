// Multigrid levels resident in one workgroup (Sec. 2's GMG where the whole
// level fits one compute unit): iterates in registers and LDS, used by the
// V-cycle tail and by the batched solvers.  Every thread of the workgroup
// calls these together.
//
// A level is split into columns (all cells of one x, or x and y in 3D) along
// its last direction, the walk; with fewer columns than threads each column is
// cut into `parts` segments of `seg` cells, and a thread owns one segment.  Its
// iterate lives in registers, so the walk neighbours cost nothing, and only the
// lateral neighbours and the segment's two ends go through LDS.  What bounded
// the loops this replaces was latency: face coefficients and right-hand sides
// read from L2 cell by cell (500 to 800 cycles each), a division per cell and
// sweep.  Here each cell has a class, formed once: 0 where every face holds the
// level's constant (0 on walls), so the coefficients follow from the position;
// 1 where it is solid; 2 elsewhere.  Only lanes with cells of class 2 load
// coefficients, four rows at a time, and w / D comes from a table (class 0) or
// an array formed once (class 2).  Small levels keep coefficients and w / D in
// LDS instead.
//
// Measured per launch of the V-cycle tail: 64 x 32 down in FP64 21.3 -> 16.1 us,
// 16^3 down uniform in FP32 18.2 -> 14.8 us, 16^3 down past a sphere in FP64
// 35 -> 30 us (what is left: the coarsest solve, barriers, the launch).
//
// Two styles of arithmetic.  RS_TILED is that of k_smooth, k_resid_restrict
// (resid_row and its order of sums over the 2^d children) and k_prolong: the
// V-cycle tail's iterates are bitwise those of the per-level kernels.  RS_SEQ is
// that of wl_wg.h (w r / D, children summed one after another): the batched
// mixed-precision solves take it, and their iterates are bitwise those of their
// general path.  (The batched FP64 solves take RS_TILED, see res_solve64.)
#pragma once

#include <type_traits>

#include "wl_cg.h"
#include "wl_jacobi.h"

namespace wl {

constexpr int kResThreads = 1024;
constexpr int kResLevels = 8;
constexpr int kResChunk = 4;  // rows whose coefficients are loaded together
constexpr int kResChild = 2;  // coarse cells a thread sums (RS_SEQ in 3D)

template <typename T>
struct RLevel {
    int nx, ny, nw, N;          // lateral sides (ny = 1 in 2D), walk length, cells
    int px, py, pw;             // periodic
    int parts, seg;             // segments per column, cells per segment
    unsigned long long mx, mc;  // ceil(2^32 / d) for nx and the column count
    const T* Lx;                // face coefficients (global)
    const T* Ly;
    const T* Lw;
    T* wd;                      // w / D (RS_SEQ: D) of class-2 cells (global; levels not staged)
    T Lc, wD;                   // the constant coefficient; w / D of a uniform level
    int ox0, ox1, ob, ot;       // LDS offsets: iterate buffers, right-hand side, restriction sums
    int ol;                     // staged coefficients Lx, Ly (3D), Lw, w / D (D), or -1
    int ocw;                    // class words, one per thread (levels not staged)
};

// This thread's segment.
struct RGeo {
    int c0, k0, cnt;         // first cell, its walk index, cells (0: none)
    int oxm, oxp, oym, oyp;  // lateral neighbour offsets (self at a wall)
    int ilo, ihi;            // cells below the first and above the last (self at a wall)
    bool hxl, hxu, hyl, hyu, hwl, hwu;  // faces that exist (hwl / hwu: at the segment's ends)
};

template <typename T>
__device__ __forceinline__ RGeo res_geo(const RLevel<T>& L) {
    const int t = opaque(int(threadIdx.x));
    const int cols = L.nx * L.ny;
    const int part = int((unsigned long long)unsigned(t) * L.mc >> 32);
    RGeo q;
    if (part >= L.parts) {
        q = RGeo{};
        return q;
    }
    const int col = t - part * cols;
    const int j = int((unsigned long long)unsigned(col) * L.mx >> 32), i = col - j * L.nx;
    q.k0 = part * L.seg;
    q.cnt = min(L.seg, L.nw - q.k0);
    q.c0 = col + q.k0 * cols;
    q.hxl = i > 0 || L.px;
    q.hxu = i < L.nx - 1 || L.px;
    q.hyl = j > 0 || L.py;
    q.hyu = j < L.ny - 1 || L.py;
    q.oxm = i > 0 ? -1 : (L.px ? L.nx - 1 : 0);
    q.oxp = i < L.nx - 1 ? 1 : (L.px ? 1 - L.nx : 0);
    q.oym = (j > 0 ? -1 : (L.py ? L.ny - 1 : 0)) * L.nx;
    q.oyp = (j < L.ny - 1 ? 1 : (L.py ? 1 - L.ny : 0)) * L.nx;
    const int k1 = q.k0 + q.cnt, cl = q.c0 + (q.cnt - 1) * cols;
    q.hwl = q.k0 > 0 || L.pw;
    q.hwu = k1 < L.nw || L.pw;
    q.ilo = q.k0 > 0 ? q.c0 - cols : (L.pw ? q.c0 + (L.nw - 1) * cols : q.c0);
    q.ihi = k1 < L.nw ? cl + cols : (L.pw ? cl - (L.nw - 1) * cols : cl);
    return q;
}

// The six faces of a cell read from the arrays, 0 on walls; returns D.
template <typename T, bool D3>
__device__ __forceinline__ T res_faces(const RLevel<T>& L, const RGeo& q, int c, int k, T (&f)[6]) {
    const int cols = L.nx * L.ny;
    const bool up = k < L.nw - 1 || L.pw;
    const int cu = k < L.nw - 1 ? c + cols : (L.pw ? c - (L.nw - 1) * cols : c);
    f[0] = L.Lx[c];
    f[1] = q.hxu ? L.Lx[c + q.oxp] : T(0);
    f[2] = D3 ? L.Ly[c] : T(0);
    f[3] = D3 && q.hyu ? L.Ly[c + q.oyp] : T(0);
    f[4] = L.Lw[c];
    f[5] = up ? L.Lw[cu] : T(0);
    T D = T(0);
    D += f[0] + f[1];
    if (D3) D += f[2] + f[3];
    D += f[4] + f[5];
    return D;
}

enum { RS_TILED = 0, RS_SEQ = 1 };

// Class word of this thread's segment (2 bits per cell), and w / D (RS_SEQ: D)
// of its class-2 cells into L.wd.  seg <= 16.
template <typename T, bool D3, int STYLE>
__device__ __forceinline__ unsigned res_classify(const RLevel<T>& L, T omega) {
    const RGeo q = res_geo(L);
    const int cols = L.nx * L.ny;
    unsigned w = 0;
    for (int m = 0; m < q.cnt; ++m) {
        const int c = q.c0 + m * cols, k = q.k0 + m;
        T f[6];
        const T D = res_faces<T, D3>(L, q, c, k, f);
        const bool wl_ = k > 0 || L.pw, wu_ = k < L.nw - 1 || L.pw;
        const bool same = f[0] == (q.hxl ? L.Lc : T(0)) && f[1] == (q.hxu ? L.Lc : T(0)) &&
                          (!D3 || (f[2] == (q.hyl ? L.Lc : T(0)) && f[3] == (q.hyu ? L.Lc : T(0)))) &&
                          f[4] == (wl_ ? L.Lc : T(0)) && f[5] == (wu_ ? L.Lc : T(0));
        const unsigned cls = !(D > T(0)) ? 1u : same ? 0u : 2u;
        if (cls && L.wd) L.wd[c] = cls == 2 ? (STYLE == RS_SEQ ? D : omega / D) : T(0);
        w |= cls << (2 * m);
    }
    return w;
}

// Coefficients and w / D (RS_SEQ: D) of a staged level into LDS.
template <typename T, bool D3, int STYLE>
__device__ __forceinline__ void res_stage(const RLevel<T>& L, T omega, T* lds) {
    const RGeo q = res_geo(L);
    const int cols = L.nx * L.ny;
    T* s = lds + L.ol;
    for (int m = 0; m < q.cnt; ++m) {
        const int c = q.c0 + m * cols;
        T f[6];
        const T D = res_faces<T, D3>(L, q, c, q.k0 + m, f);
        s[c] = f[0];
        if (D3) s[L.N + c] = f[2];
        s[(D3 ? 2 : 1) * L.N + c] = f[4];
        s[(D3 ? 3 : 2) * L.N + c] = D > T(0) ? (STYLE == RS_SEQ ? D : omega / D) : T(0);
    }
}

enum { RK_ZERO = 0, RK_SWEEP = 1, RK_RESID = 2 };

// One level's segment in this thread: M >= seg cells.  UNIF: one coefficient
// everywhere, periodic.  STAGED: coefficients and w / D from LDS.
template <typename T, int M, bool D3, bool UNIF, bool STAGED, int STYLE>
struct ResLev {
    // (FP64: two rows, 28 registers of coefficients instead of 56)
    static constexpr int kRows = sizeof(T) == 8 ? 2 : kResChunk;
    static constexpr int CH = M < kRows ? M : kRows;
    static constexpr unsigned kBits = (1u << (2 * CH)) - 1u;  // class bits of a chunk
    const RLevel<T>& L;
    T* lds;
    RGeo q;
    int cols;
    unsigned cw;
    T x[M];
    T omega;
    // class 0: w / D (RS_SEQ: 1 / D and D) inside, at the segment's first and last cell
    T wdm, wdl, wdh, Dm, Dl, Dh;

    __device__ __forceinline__ ResLev(const RLevel<T>& L_, T omega_, T* lds_, const unsigned* cws)
        : L(L_), lds(lds_), q(res_geo(L_)), cols(L_.nx * L_.ny), cw(0), omega(omega_) {
#pragma unroll
        for (int m = 0; m < M; ++m) x[m] = T(0);
        if (!UNIF && !STAGED) {
            cw = cws[L.ocw + int(threadIdx.x)];
            const T Lc = L.Lc;
            T D = T(0);
            D += (q.hxl ? Lc : T(0)) + (q.hxu ? Lc : T(0));
            if (D3) D += (q.hyl ? Lc : T(0)) + (q.hyu ? Lc : T(0));
            Dm = D + (Lc + Lc);
            Dl = q.hwl ? Dm : D + Lc;
            Dh = q.hwu ? Dm : D + Lc;
            const T num = STYLE == RS_SEQ ? T(1) : omega;
            wdm = num / Dm;
            wdl = q.hwl ? wdm : num / Dl;
            wdh = q.hwu ? wdm : num / Dh;
        }
    }

    // A pass over the segment from the iterate in x and Xin (this level's
    // published iterate): the damped-Jacobi update of x (RK_ZERO: from zero),
    // or the residual handed to fn(m, r) (RK_RESID); with norm, returns the
    // sum of the squared residuals.  bfn(m, c): right-hand side of the cell.
    //
    // Class 0 needs no face coefficient at all: at a wall the neighbour is the
    // cell itself, so the difference that face multiplies is zero, and Lc is a
    // power of two (1 on the fine level, doubled per level in 3D), so A x =
    // Lc s, s the sum of the second differences, has the bits of the general
    // form.  The other classes are computed apart, by the lanes that have them.
    template <int KIND, bool NORM, typename Bf, typename Fn>
    __device__ __forceinline__ double pass(const T* Xin, Bf&& bfn, Fn&& fn) {
        double sum = 0.0;
        if (q.cnt == 0) return sum;
        const int c0 = opaque(q.c0);
        T lo = T(0), hi = T(0);
        if (KIND != RK_ZERO) {
            lo = Xin[q.ilo];
            hi = Xin[q.ihi];
        }
        T prev = lo;
        T b[CH], bn[CH];
#pragma unroll
        for (int r = 0; r < CH; ++r) bn[r] = bfn(r, c0 + (r < q.cnt ? r * cols : 0));
#pragma unroll
        for (int mb = 0; mb < M; mb += CH) {
            if (mb >= q.cnt) continue;  // rows this segment does not have
            T ld[CH][7];
            // right-hand sides a chunk ahead (they may come from L2)
#pragma unroll
            for (int r = 0; r < CH; ++r) {
                b[r] = bn[r];
                const int m = mb + CH + r;
                if (m < M) bn[r] = bfn(m, c0 + (m < q.cnt ? m * cols : 0));
            }
            const bool odd_cells = !UNIF && (STAGED || ((cw >> (2 * mb)) & kBits));
            if (odd_cells) {
                const T* s = STAGED ? lds + L.ol : nullptr;
                const T* gx = STAGED ? s : L.Lx;
                const T* gy = STAGED ? s + L.N : L.Ly;
                const T* gw = STAGED ? s + (D3 ? 2 : 1) * L.N : L.Lw;
                const T* gd = STAGED ? gw + L.N : L.wd;
#pragma unroll
                for (int r = 0; r < CH; ++r) {
                    const int m = mb + r;
                    const int c = c0 + (CH > 2 && m >= q.cnt ? 0 : m * cols);
                    const bool last = (m & 1) && m + 1 >= q.cnt;
                    if (KIND != RK_ZERO) {
                        ld[r][0] = gx[c];
                        ld[r][1] = q.hxu ? gx[c + q.oxp] : T(0);
                        if (D3) {
                            ld[r][2] = gy[c];
                            ld[r][3] = q.hyu ? gy[c + q.oyp] : T(0);
                        }
                        ld[r][4] = gw[c];
                        ld[r][5] = !last || q.hwu ? gw[last ? q.ihi : c + cols] : T(0);
                    }
                    if (KIND != RK_RESID) ld[r][6] = gd[c];
                }
            }
#pragma unroll
            for (int r = 0; r < CH; ++r) {
                const int m = mb + r;
                const bool on = CH <= 2 || m < q.cnt, last = (m & 1) && m + 1 >= q.cnt;
                const int c = c0 + (on ? m * cols : 0);
                const T xI = KIND == RK_ZERO ? T(0) : x[m];
                T xxl = T(0), xxu = T(0), xyl = T(0), xyu = T(0), xwl = T(0), xwu = T(0);
                if (KIND != RK_ZERO) {
                    xxl = Xin[c + q.oxm];
                    xxu = Xin[c + q.oxp];
                    if (D3) {
                        xyl = Xin[c + q.oym];
                        xyu = Xin[c + q.oyp];
                    }
                    xwl = prev;
                    xwu = m + 1 < M && !last ? x[m + 1 < M ? m + 1 : m] : hi;
                }
                // directions in the order x, y, z (2D: x, then the walk y)
                const T yl = D3 ? xyl : xwl, yu = D3 ? xyu : xwu;
                const T zl = D3 ? xwl : T(0), zu = D3 ? xwu : T(0);
                T rr = b[r], xn = T(0);
                if (UNIF && KIND == RK_RESID) {
                    const T Lz = D3 ? L.Lc : T(0);
                    rr = resid_row(b[r], xI, xxl, xxu, yl, yu, zl, zu, L.Lc, L.Lc, L.Lc, L.Lc, Lz,
                                   Lz, D3);
                } else if (UNIF) {
                    if (KIND != RK_ZERO)
                        rr = b[r] - jacobi_ax_uniform(xI, xxl, xxu, yl, yu, zl, zu, L.Lc, D3);
                    xn = jacobi_new_scaled(xI, rr, true, L.wD);
                } else if (!STAGED) {
                    if (KIND != RK_ZERO) {
                        T sd = (xxu - xI) - (xI - xxl);
                        sd += (yu - xI) - (xI - yl);
                        if (D3) sd += (zu - xI) - (xI - zl);
                        rr = fma(-L.Lc, sd, b[r]);
                    }
                    const T wd = last ? wdh : m == 0 ? wdl : wdm;
                    if (STYLE == RS_SEQ)
                        xn = xI - div_by(omega * rr, last ? Dh : m == 0 ? Dl : Dm, wd);
                    else
                        xn = fma(-wd, rr, xI);
                }
                if (odd_cells && (STAGED || ((cw >> (2 * m)) & 3u))) {
                    const T(&f)[7] = ld[r];
                    const T fy0 = D3 ? f[2] : f[4], fy1 = D3 ? f[3] : f[5];
                    const T fz0 = D3 ? f[4] : T(0), fz1 = D3 ? f[5] : T(0);
                    // (resid_row: the compiler would share the product of the
                    // face between two rows and round the other differently)
                    if (KIND != RK_ZERO)
                        rr = resid_row(b[r], xI, xxl, xxu, yl, yu, zl, zu, f[0], f[1], fy0, fy1,
                                       fz0, fz1, D3);
                    else
                        rr = b[r];
                    if (STYLE == RS_SEQ)
                        xn = f[6] > T(0) ? xI - omega * rr / f[6] : T(0);
                    else
                        xn = jacobi_new_scaled(xI, rr, f[6] > T(0), f[6]);
                }
                if (NORM && on) sum = fma(double(rr), double(rr), sum);
                if (KIND == RK_RESID)
                    fn(m, on ? rr : T(0));
                else
                    x[m] = xn;
                prev = xI;
            }
        }
        return sum;
    }

    __device__ __forceinline__ void put(T* X) const {
        const int c0 = opaque(q.c0);
#pragma unroll
        for (int m = 0; m < M; ++m)
            if (m < q.cnt) X[c0 + m * cols] = x[m];
    }
    __device__ __forceinline__ void get(const T* X) {
        const int c0 = opaque(q.c0);
#pragma unroll
        for (int m = 0; m < M; ++m)
            if (m < q.cnt) x[m] = X[c0 + m * cols];
    }
    // what a solve keeps of the level between its phases
    __device__ __forceinline__ void save(T (&v)[M]) const {
#pragma unroll
        for (int m = 0; m < M; ++m) v[m] = x[m];
    }
    __device__ __forceinline__ void load(const T (&v)[M]) {
#pragma unroll
        for (int m = 0; m < M; ++m) x[m] = v[m];
    }
    // publish x into X; `same`: X is the buffer the last pass read
    __device__ __forceinline__ void publish(T* X, bool same) const {
        if (same) __syncthreads();
        put(X);
        __syncthreads();
    }

    // The residual of x (published in Xin) summed over the children of each
    // coarse cell into Bc.  RS_TILED: the walk pair first in 3D and the x pair
    // first in 2D, as k_resid_restrict sums them; RS_SEQ: one after another, x
    // fastest.  The x pair are lanes 2q and 2q + 1.  tmp: a quarter of the
    // level (RS_TILED in 3D), the level (RS_SEQ in 3D).  overlap: Bc or tmp
    // lie in memory the pass reads, or in each other.
    template <typename Bf>
    __device__ __forceinline__ void restrict_to(const T* Xin, Bf&& bfn, T* Bc, T* tmp, bool overlap) {
        if (D3 && STYLE == RS_SEQ) {
            T v[M];
#pragma unroll
            for (int m = 0; m < M; ++m) v[m] = T(0);
            pass<RK_RESID, false>(Xin, bfn, [&](int m, T r) { v[m] = r; });
            if (overlap) __syncthreads();
            const int c0 = opaque(q.c0);
#pragma unroll
            for (int m = 0; m < M; ++m)
                if (m < q.cnt) tmp[c0 + m * cols] = v[m];
            __syncthreads();
            // up to kResChild coarse cells a thread (the host's plan sees to it)
            const int hx = L.nx / 2, per = hx * (L.ny / 2), nc = L.N / 8;
            T sum[kResChild];
#pragma unroll
            for (int u = 0; u < kResChild; ++u) {
                const int c = int(threadIdx.x) + u * int(blockDim.x);
                sum[u] = T(0);
                if (c >= nc) continue;
                const int kk = c / per, rem = c - kk * per, jj = rem / hx, ii = rem - jj * hx;
                const T* f = tmp + 2 * ii + L.nx * (2 * jj) + cols * (2 * kk);
                sum[u] = f[0];
                sum[u] += f[1];
                sum[u] += f[L.nx];
                sum[u] += f[L.nx + 1];
                sum[u] += f[cols];
                sum[u] += f[cols + 1];
                sum[u] += f[cols + L.nx];
                sum[u] += f[cols + L.nx + 1];
            }
            if (overlap) __syncthreads();
#pragma unroll
            for (int u = 0; u < kResChild; ++u) {
                const int c = int(threadIdx.x) + u * int(blockDim.x);
                if (c < nc) Bc[c] = sum[u];
            }
            __syncthreads();
            return;
        }
        T h[M / 2];
#pragma unroll
        for (int m = 0; m < M / 2; ++m) h[m] = T(0);
        pass<RK_RESID, false>(Xin, bfn, [&](int m, T r) {
            if (D3) {
                h[m / 2] = (m & 1) ? h[m / 2] + r : r;
            } else if (STYLE == RS_SEQ) {  // right on even lanes, the ones that store
                const T o = lane_swap(r);
                h[m / 2] = (m & 1) ? (h[m / 2] + r) + o : r + o;
            } else {
                const T s = r + lane_swap(r);
                h[m / 2] = (m & 1) ? h[m / 2] + s : s;
            }
        });
        if (D3) {
#pragma unroll
            for (int m = 0; m < M / 2; ++m) h[m] = h[m] + lane_swap(h[m]);
        }
        if (overlap) __syncthreads();
        const int col = opaque(q.c0 - q.k0 * cols);  // i + nx j
        const int j = int((unsigned long long)unsigned(col) * L.mx >> 32), i = col - j * L.nx;
        T* out = D3 ? tmp : Bc;
        const int hx = L.nx / 2;
        if (q.cnt && !(i & 1)) {
            const int base = i / 2 + hx * j, step = hx * L.ny;
#pragma unroll
            for (int m = 0; m < M / 2; ++m)
                if (2 * m < q.cnt) out[base + step * (q.k0 / 2 + m)] = h[m];
        }
        __syncthreads();
        if (D3) {
            // y pairs
            const int hy = L.ny / 2, nc = L.N / 8, per = hx * hy;
            for (int c = int(threadIdx.x); c < nc; c += int(blockDim.x)) {
                const int kk = c / per, rem = c - kk * per, jj = rem / hx, ii = rem - jj * hx;
                const T* s = tmp + ii + hx * (2 * jj + L.ny * kk);
                Bc[c] = s[0] + s[hx];
            }
            __syncthreads();
        }
    }

    // x += P xc (xc: the coarse level's iterate in LDS).
    __device__ __forceinline__ void prolong(const RLevel<T>& C, const T* xc) {
        if (q.cnt == 0) return;
        const int col = opaque(q.c0 - q.k0 * cols);
        const int j = int((unsigned long long)unsigned(col) * L.mx >> 32), i = col - j * L.nx;
        int ip, iq, jp = 0, jq = 0;
        prolong_pair(i, C.nx, L.px, ip, iq);
        if (D3) prolong_pair(j, C.ny, L.py, jp, jq);
        const int cpl = C.nx * C.ny;
        auto plane = [&](int K) -> T {
            const T* r = xc + cpl * K;
            const T a = lerp34(r[ip + C.nx * jp], r[iq + C.nx * jp]);
            if (!D3) return a;
            const T b = lerp34(r[ip + C.nx * jq], r[iq + C.nx * jq]);
            return lerp34(a, b);
        };
        const int K0 = q.k0 / 2;
        T pm = plane(K0 > 0 ? K0 - 1 : (L.pw ? C.nw - 1 : 0)), pc = plane(K0);
#pragma unroll
        for (int m = 0; m < M; m += 2) {
            if (m >= q.cnt) break;
            const int K = K0 + m / 2;
            const T pp = plane(K < C.nw - 1 ? K + 1 : (L.pw ? 0 : K));
            x[m] = x[m] + lerp34(pc, pm);
            x[m + 1] = x[m + 1] + lerp34(pc, pp);
            pm = pc;
            pc = pp;
        }
    }

    // a / d for rd = 1 / d correctly rounded: the quotient's residual corrects
    // it to the correctly rounded one (Markstein, 1990)
    static __device__ __forceinline__ T div_by(T a, T d, T rd) {
        const T qt = a * rd;
        return fma(fma(-qt, d, a), rd, qt);
    }
    static __device__ __forceinline__ T lane_swap(T v) {  // the neighbouring lane's (t ^ 1)
        if (sizeof(T) == 8) return T(dpp_f64<0xB1>(double(v)));
        return T(__int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(float(v)), 0xB1, 0xf,
                                                            0xf, false)));
    }
};

// Lower levels of a V-cycle: right-hand side in LDS (L.ob), pre-smoothed
// iterate left in L.ox1 and the restricted residual in the next level's ob.
template <typename T, int M, bool D3, bool UNIF, bool STAGED, int STYLE>
__device__ __forceinline__ void res_down_m(const RLevel<T>& L, const RLevel<T>& C, T omega, T* lds,
                                           const unsigned* cws) {
    ResLev<T, M, D3, UNIF, STAGED, STYLE> S(L, omega, lds, cws);
    const T* B = lds + L.ob;
    auto bf = [&](int, int c) { return B[c]; };
    auto nop = [](int, T) {};
    S.template pass<RK_ZERO, false>(nullptr, bf, nop);
    S.publish(lds + L.ox0, false);
    S.template pass<RK_SWEEP, false>(lds + L.ox0, bf, nop);
    S.publish(lds + L.ox1, false);
    S.restrict_to(lds + L.ox1, bf, lds + C.ob, lds + L.ox0, false);
}

// ... and on the way up: the coarse correction (the next level's ox0) added,
// two sweeps, the result in ox0 (or in global memory, gout).
template <typename T, int M, bool D3, bool UNIF, bool STAGED, int STYLE>
__device__ __forceinline__ void res_up_m(const RLevel<T>& L, const RLevel<T>& C, T omega, T* lds,
                                         const unsigned* cws, T* gout) {
    ResLev<T, M, D3, UNIF, STAGED, STYLE> S(L, omega, lds, cws);
    const T* B = lds + L.ob;
    auto bf = [&](int, int c) { return B[c]; };
    auto nop = [](int, T) {};
    S.get(lds + L.ox1);
    S.prolong(C, lds + C.ox0);
    S.publish(lds + L.ox0, false);
    S.template pass<RK_SWEEP, false>(lds + L.ox0, bf, nop);
    S.publish(lds + L.ox1, false);
    S.template pass<RK_SWEEP, false>(lds + L.ox1, bf, nop);
    if (gout)
        S.put(gout);
    else
        S.publish(lds + L.ox0, false);
}

// MAXM: the longest segment of the caller's levels, 4 or 8.
template <typename T, bool D3, bool UNIF, int MAXM, int STYLE>
__device__ __forceinline__ void res_down(const RLevel<T>& L, const RLevel<T>& C, T omega, T* lds,
                         const unsigned* cws) {
    if (UNIF) {
        if (L.seg <= 2)
            res_down_m<T, 2, D3, UNIF, false, STYLE>(L, C, omega, lds, cws);
        else if (MAXM == 4 || L.seg <= 4)
            res_down_m<T, 4, D3, UNIF, false, STYLE>(L, C, omega, lds, cws);
        else
            res_down_m<T, 8, D3, UNIF, false, STYLE>(L, C, omega, lds, cws);
    } else if (L.ol >= 0) {
        if (L.seg <= 2)
            res_down_m<T, 2, D3, UNIF, true, STYLE>(L, C, omega, lds, cws);
        else
            res_down_m<T, 4, D3, UNIF, true, STYLE>(L, C, omega, lds, cws);
    } else if (MAXM == 4 || L.seg <= 4) {
        res_down_m<T, 4, D3, UNIF, false, STYLE>(L, C, omega, lds, cws);
    } else {
        res_down_m<T, 8, D3, UNIF, false, STYLE>(L, C, omega, lds, cws);
    }
}

template <typename T, bool D3, bool UNIF, int MAXM, int STYLE>
__device__ __forceinline__ void res_up(const RLevel<T>& L, const RLevel<T>& C, T omega, T* lds,
                       const unsigned* cws, T* gout = nullptr) {
    if (UNIF) {
        if (L.seg <= 2)
            res_up_m<T, 2, D3, UNIF, false, STYLE>(L, C, omega, lds, cws, gout);
        else if (MAXM == 4 || L.seg <= 4)
            res_up_m<T, 4, D3, UNIF, false, STYLE>(L, C, omega, lds, cws, gout);
        else
            res_up_m<T, 8, D3, UNIF, false, STYLE>(L, C, omega, lds, cws, gout);
    } else if (L.ol >= 0) {
        if (L.seg <= 2)
            res_up_m<T, 2, D3, UNIF, true, STYLE>(L, C, omega, lds, cws, gout);
        else
            res_up_m<T, 4, D3, UNIF, true, STYLE>(L, C, omega, lds, cws, gout);
    } else if (MAXM == 4 || L.seg <= 4) {
        res_up_m<T, 4, D3, UNIF, false, STYLE>(L, C, omega, lds, cws, gout);
    } else {
        res_up_m<T, 8, D3, UNIF, false, STYLE>(L, C, omega, lds, cws, gout);
    }
}

// ------------------------------------------------------------- host planning
// Geometry of one level for a workgroup of `threads`; false when it has more
// columns than threads or segments longer than maxseg.  Every level but the
// coarsest has even sides, and even segments keep the walk pairs of a
// restriction in one thread.
template <typename T>
inline bool res_plan_level(const Grid& g, const T* const Lc[3], T constant, T wD, int threads,
                           int maxseg, bool coarsest, RLevel<T>& L) {
    L = RLevel<T>{};
    const bool d3 = g.ndim == 3;
    L.nx = g.n0;
    L.ny = d3 ? g.n1 : 1;
    L.nw = d3 ? g.n2 : g.n1;
    L.N = int(cells(g));
    L.px = g.per0;
    L.py = d3 ? g.per1 : 0;
    L.pw = d3 ? g.per2 : g.per1;
    L.Lx = Lc[0];
    L.Ly = d3 ? Lc[1] : nullptr;
    L.Lw = d3 ? Lc[2] : Lc[1];
    L.Lc = constant;
    L.wD = wD;
    L.ol = -1;
    L.ot = 0;
    const int cols = L.nx * L.ny;
    if (coarsest) {  // solved, not smoothed
        L.parts = 1;
        L.seg = L.nw;
        return true;
    }
    if (cols > threads || (L.nw & 1) || (L.nx & 1) || (d3 && (L.ny & 1))) return false;
    const int parts = threads / cols;
    L.seg = (L.nw + parts - 1) / parts;
    L.seg += L.seg & 1;
    L.parts = (L.nw + L.seg - 1) / L.seg;
    const unsigned long long two32 = 1ull << 32;
    L.mx = (two32 + unsigned(L.nx) - 1) / unsigned(L.nx);
    L.mc = (two32 + unsigned(cols) - 1) / unsigned(cols);
    return L.seg <= maxseg && cols * L.parts <= threads;
}

// LDS layout of the lower levels lev[first .. n) from element offset `off` on
// (X0, X1 and B each; the coarsest only B and X0), then, while it ends before
// `limit`, staged coefficients from the coarsest smoothed level upwards in
// [stage, limit).  Levels that are not staged get class words.  Returns the
// first free element of the iterate region.
template <typename T>
inline int res_layout(RLevel<T>* lev, int first, int n, int off) {
    for (int l = first; l < n; ++l) {
        RLevel<T>& L = lev[l];
        L.ox0 = off;
        off += L.N;
        if (l < n - 1) {
            L.ox1 = off;
            off += L.N;
        }
        L.ob = off;
        off += L.N;
    }
    return off;
}

template <typename T>
inline int res_stage_layout(RLevel<T>* lev, int first, int n, int stage, int limit, bool d3) {
    for (int l = n - 2; l >= first; --l) {
        RLevel<T>& L = lev[l];
        const int need = (d3 ? 4 : 3) * L.N;
        if (L.seg > 4 || stage + need > limit) break;
        L.ol = stage;
        stage += need;
    }
    return stage;
}

}  // namespace wl
