// Coarsest-level solves shared by the multigrid kernels, the V-cycle tail and
// the batched one-workgroup solvers.
#pragma once

#include "wl_device.h"

namespace wl {

// Iterative solve of the coarsest level: conjugate gradients on M = -A (SPD on
// the active set, D > 0), the right-hand side restricted to the active cells
// and made mean-free there; FP64, minimum-norm (mean-free) result, stopped at
// ||r|| <= tol ||r0||.  No preconditioner: the pressure of cells a body nearly
// closes is set by how far the iteration resolves their weak modes, so a
// diagonal one changes an FP32 pressure there (by a tenth of its norm past a
// thin torus) and is no faster.
//
// Latency bounds it (128 cells are two wavefronts' work), so the iteration is
// arranged with one reduction (Chronopoulos and Gear, 1989): with w = M r the
// sums r r and r w are formed together, and p and M p follow by recurrence.
// Each thread holds its cells' stencils in registers; r of the neighbours goes
// through LDS.  Levels of at most kCgWaveMax cells take one
// wave (no barrier at all); larger ones the first nw = ceil(N / 128) waves of
// the workgroup, two cells per thread (t and t + 64 nw), two barriers an
// iteration.  Every rounding is spelled out (contraction off, fused
// multiply-adds written as such), so the standalone kernels, the V-cycle tail
// and the batched solvers, which all call it, agree bit for bit.  Measured per
// solve: 693 uniform cells, FP32 level, 45 -> 23 us (one cell a thread and two
// shuffled sums an iteration before); past a sphere, 385 cells, FP64, 100 us as
// a launch of its own -> about 62 us inside the V-cycle tail; the batched
// solver's 4 x 4 levels, which took a whole workgroup's barriers, 1.08x
// (128^2 Poisson batch) and 1.22x (64^2 Navier-Stokes batch) on the whole call.
constexpr int kCgWaveMax = 128;
constexpr int kCgGroupWaves = kCoarseMax / 128;
struct CgLds {
    double u[kCoarseMax];
    double red[2][2 * kCgGroupWaves];
};

__device__ __forceinline__ void wave_lds_sync() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_s_waitcnt(0xc07f);  // lgkmcnt(0): this wave's LDS traffic done
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// Data-parallel move of a double across the lanes of a row (CTRL: a DPP
// control, every lane valid).
template <int CTRL>
__device__ __forceinline__ double dpp_f64(double v) {
    const long long u = __double_as_longlong(v);
    const int lo = __builtin_amdgcn_update_dpp(0, int(u), CTRL, 0xf, 0xf, false);
    const int hi = __builtin_amdgcn_update_dpp(0, int(u >> 32), CTRL, 0xf, 0xf, false);
    return __longlong_as_double((static_cast<long long>(hi) << 32) |
                                static_cast<long long>(static_cast<unsigned>(lo)));
}

__device__ __forceinline__ double readlane_f64(double v, int lane) {
    const long long u = __double_as_longlong(v);
    const int lo = __builtin_amdgcn_readlane(int(u), lane);
    const int hi = __builtin_amdgcn_readlane(int(u >> 32), lane);
    return __longlong_as_double((static_cast<long long>(hi) << 32) |
                                static_cast<long long>(static_cast<unsigned>(lo)));
}

// Sum over the 64 lanes of a full wave, the same value in every lane: lane
// pairs, quads, half rows and rows by data-parallel moves (each add takes
// two equal partial sums in either order, so every lane of a row ends with
// the same bits), then the four row sums in row order.
__device__ __forceinline__ double wave_sum_f64(double v) {
#pragma clang fp contract(off)
    v = v + dpp_f64<0xB1>(v);   // quad_perm [1, 0, 3, 2]
    v = v + dpp_f64<0x4E>(v);   // quad_perm [2, 3, 0, 1]
    v = v + dpp_f64<0x141>(v);  // row_half_mirror
    v = v + dpp_f64<0x140>(v);  // row_mirror
    return (readlane_f64(v, 0) + readlane_f64(v, 16)) + (readlane_f64(v, 32) + readlane_f64(v, 48));
}

// WAVE: called by the first wave alone; else by every thread of the workgroup
// (at least 64 nw), the waves beyond nw only meeting the barriers.
// Returns whether the residual reached the tolerance with a finite iterate (a
// residual that is no number ends the loop as a small one does, but only a step
// that was not finite can make it so; tested after the loop, since a second
// comparison in it made a solve of 693 cells 24.0 instead of 23.0 us).
template <typename T, int PER, bool WAVE>
__device__ __forceinline__ bool coarse_cg(const Grid& g, const T* L0, const T* L1, const T* L2,
                                          T Lc, int uniform, const T* b, T* xout, double tol,
                                          int maxit, CgLds& S) {
#pragma clang fp contract(off)
    const int N = int(cells(g));
    const int t = opaque(int(threadIdx.x));
    const int stride = WAVE ? 64 : 64 * ((N + 64 * PER - 1) / (64 * PER));
    const bool worker = WAVE || t < stride;
    double* su = S.u;
    if (!WAVE && t < 2 * 2 * kCgGroupWaves) (&S.red[0][0])[t] = 0.0;
    double D[PER], cf[PER][6], x[PER], r[PER], p[PER], q[PER], w[PER], bt[PER];
    int nb[PER][6];
    bool act[PER], own[PER];
#pragma unroll
    for (int m = 0; m < PER; ++m) {
        const int c = t + stride * m;
        own[m] = worker && c < N;
        D[m] = 0.0;
        bt[m] = 0.0;
#pragma unroll
        for (int f = 0; f < 6; ++f) {
            cf[m][f] = 0.0;
            nb[m][f] = own[m] ? c : 0;
        }
        if (own[m]) {
            const int i = c % g.n0, j = (c / g.n0) % g.n1, k = c / (g.n0 * g.n1);
            const int n[3] = {g.n0, g.n1, g.n2}, per[3] = {g.per0, g.per1, g.per2};
            const int co[3] = {i, j, k}, st[3] = {1, g.n0, g.n0 * g.n1};
            const T* Ld[3] = {L0, L1, L2};
#pragma unroll
            for (int d = 0; d < 3; ++d) {
                if (d >= g.ndim) break;
                const int lo = nb_lo(co[d], n[d], per[d]), up = nb_up(co[d], n[d], per[d]);
                nb[m][2 * d] = c + (lo - co[d]) * st[d];
                nb[m][2 * d + 1] = c + (up - co[d]) * st[d];
                const double Ll = uniform ? double(Lc) : double(Ld[d][c]);
                const double Lu = (co[d] < n[d] - 1 || per[d])
                                      ? (uniform ? double(Lc) : double(Ld[d][nb[m][2 * d + 1]]))
                                      : 0.0;
                cf[m][2 * d] = Ll;
                cf[m][2 * d + 1] = Lu;
                D[m] = D[m] + (Ll + Lu);
            }
            bt[m] = double(b[c]);
        }
        act[m] = D[m] > 0.0;
    }
    if (!WAVE) __syncthreads();  // the cleared sums
    int buf = 0;
    // two sums over the working threads, the same in every thread; the
    // group's buffers alternate, so one is written again only after the
    // barrier that follows its last read
    auto sums = [&](double& a, double& c) {
        if (worker) {
            a = wave_sum_f64(a);
            c = wave_sum_f64(c);
        }
        if (WAVE) return;
        if (worker && (t & 63) == 0) {
            S.red[buf][t >> 6] = a;
            S.red[buf][kCgGroupWaves + (t >> 6)] = c;
        }
        __syncthreads();
        // every wave reads each value once (lane l the value l mod 16) and
        // sums the two halves of its rows by data-parallel moves
        double v = S.red[buf][t & (2 * kCgGroupWaves - 1)];
        v = v + dpp_f64<0xB1>(v);   // quad_perm [1, 0, 3, 2]
        v = v + dpp_f64<0x4E>(v);   // quad_perm [2, 3, 0, 1]
        v = v + dpp_f64<0x141>(v);  // row_half_mirror
        a = readlane_f64(v, 0);
        c = readlane_f64(v, kCgGroupWaves);
        buf ^= 1;
    };
    static_assert(kCgGroupWaves == 8, "the sums take half a row per value");
    auto publish = [&]() {  // the LDS writes before it are seen by all working threads
        if (WAVE)
            wave_lds_sync();
        else
            __syncthreads();
    };
    double sumb = 0.0, cnt = 0.0;
#pragma unroll
    for (int m = 0; m < PER; ++m) {
        sumb = sumb + (act[m] ? bt[m] : 0.0);
        cnt = cnt + (act[m] ? 1.0 : 0.0);
    }
    sums(sumb, cnt);
    const double mean = cnt > 0.0 ? sumb / cnt : 0.0;
    // solve M x = B with B = -(b - mean) on active cells
#pragma unroll
    for (int m = 0; m < PER; ++m) {
        x[m] = 0.0;
        r[m] = act[m] ? -(bt[m] - mean) : 0.0;
        p[m] = 0.0;
        q[m] = 0.0;
        if (own[m]) su[t + stride * m] = r[m];
    }
    publish();
    double goal = 0.0, inv_rr0 = 0.0, pq = 0.0;
    bool done = false;
    for (int it = 0; it <= maxit; ++it) {
        double rr = 0.0, rw = 0.0;
#pragma unroll
        for (int m = 0; m < PER; ++m) {
            double v = 0.0;
            if (act[m]) {
                v = D[m] * r[m];
#pragma unroll
                for (int f = 0; f < 6; ++f) v = fma(-cf[m][f], su[nb[m][f]], v);
            }
            w[m] = v;
            rr = fma(r[m], r[m], rr);
            rw = fma(r[m], v, rw);
        }
        sums(rr, rw);
        // converged (or zero from the start), not a number, or out of iterations
        done = !(rr > goal);
        if (done || it == maxit) break;
        if (it == 0) goal = tol * tol * rr;
        const double beta = rr * inv_rr0;            // 0 at first
        pq = fma(-beta * beta, pq, rw);              // p M p = r w - beta^2 (p M p before)
        if (!(pq > 0.0)) break;
        const double alpha = rr / pq;
        inv_rr0 = 1.0 / rr;
        if (WAVE) wave_lds_sync();  // every lane has read su (the group: the sums' barrier)
#pragma unroll
        for (int m = 0; m < PER; ++m) {
            p[m] = fma(beta, p[m], r[m]);
            q[m] = fma(beta, q[m], w[m]);
            x[m] = fma(alpha, p[m], x[m]);
            r[m] = fma(-alpha, q[m], r[m]);
            if (own[m]) su[t + stride * m] = r[m];
        }
        publish();
    }
    // mean-free result on the active cells
    double xs = 0.0, zero = 0.0;
#pragma unroll
    for (int m = 0; m < PER; ++m) xs = xs + (act[m] ? x[m] : 0.0);
    sums(xs, zero);
    const double xm = cnt > 0.0 ? xs / cnt : 0.0;
#pragma unroll
    for (int m = 0; m < PER; ++m)
        if (own[m]) xout[t + stride * m] = act[m] ? T(x[m] - xm) : T(0);
    return done && isfinite(xs);
}

// The iterative coarsest solve of a workgroup of at least 512 threads (every
// thread calls it): levels of at most kCgWaveMax cells by the first wave,
// larger ones by the group.  No barrier at the end.
template <typename T>
__device__ __forceinline__ void coarse_cg_wg(const Grid& g, const T* L0, const T* L1, const T* L2,
                                              T Lc, int uniform, const T* b, T* xout, double tol,
                                              int maxit, CgLds& S) {
    const int N = int(cells(g));
    if (N > kCgWaveMax)
        coarse_cg<T, 2, false>(g, L0, L1, L2, Lc, uniform, b, xout, tol, maxit, S);
    else if (threadIdx.x >= 64)
        return;
    else if (N <= 64)
        coarse_cg<T, 1, true>(g, L0, L1, L2, Lc, uniform, b, xout, tol, maxit, S);
    else
        coarse_cg<T, 2, true>(g, L0, L1, L2, Lc, uniform, b, xout, tol, maxit, S);
}

}  // namespace wl
