// Whole pressure solves of one workgroup with the fine level resident too
// (wl_res.h): the batched solvers' path for requests whose fine iterate fits
// the LDS of a compute unit.  FP64 V-cycles, or FP32 V-cycles under an FP64
// defect correction.  The general path (wl_wg.h: every level in global memory)
// serves larger requests; on 128^2 FP64 requests it moved 5 MB per V-cycle and
// workgroup through L2 (330 us per V-cycle, 256 requests in 3.6 ms; resident:
// 92 us, 1.0 ms).  What bounds it now is instruction issue on the fine level
// (9 us per sweep of 128^2 in FP64) and, below it, barriers and LDS round trips
// of a few waves (30 of the 92 us).
#pragma once

#include "wl_res.h"
#include "wl_wgsolve.h"

namespace wl {

constexpr int kResRows = 16;           // longest segment of a fine level
constexpr int kResGlobal = 4;          // levels with class words
constexpr int kResBytes = 135 * 1024;  // LDS of the iterates and staged coefficients

// A resident solve's plan: lev[0] is the fine level; its iterate shares the
// LDS of all coarser ones, which are idle while it is smoothed (and the other
// way round: its iterate stays in registers meanwhile).
struct ResPlan64 {
    RLevel<double> lev[kResLevels];
    Grid gc;  // the coarsest level
    int n;
};
struct ResPlan32 {
    RLevel<double> fine;  // FP64 x, coefficients
    RLevel<float> lev[kResLevels];
    Grid gc;
    int n;
};

struct ResLds {
    double raw[kResBytes / 8];
    unsigned cws[kResGlobal * kResThreads];
};

// Coarse coefficients: half the sum of the covered fine faces.
template <typename T, bool D3>
__device__ inline void res_coarsen(const RLevel<T>& F, const RLevel<T>& C) {
    const int cf = F.nx * F.ny, cc = C.nx * C.ny;
    T* Cx = const_cast<T*>(C.Lx);
    T* Cy = const_cast<T*>(C.Ly);
    T* Cw = const_cast<T*>(C.Lw);
    for (int c = int(threadIdx.x); c < C.N; c += int(blockDim.x)) {
        const int k = c / cc, col = c - k * cc, j = col / C.nx, i = col - j * C.nx;
        const int f = 2 * i + F.nx * (D3 ? 2 * j : 0) + cf * 2 * k;
        if (D3) {
            Cx[c] = T(0.5) * (((F.Lx[f] + F.Lx[f + F.nx]) + F.Lx[f + cf]) + F.Lx[f + cf + F.nx]);
            Cy[c] = T(0.5) * (((F.Ly[f] + F.Ly[f + 1]) + F.Ly[f + cf]) + F.Ly[f + cf + 1]);
            Cw[c] = T(0.5) * (((F.Lw[f] + F.Lw[f + 1]) + F.Lw[f + F.nx]) + F.Lw[f + F.nx + 1]);
        } else {
            Cx[c] = T(0.5) * (F.Lx[f] + F.Lx[f + cf]);
            Cw[c] = T(0.5) * (F.Lw[f] + F.Lw[f + 1]);
        }
    }
    __syncthreads();
}

// Coefficients of every coarse level, class words, staged coefficients.
template <typename T, bool D3, int STYLE>
__device__ __forceinline__ void res_setup(const RLevel<T>* lev, int n, T omega, T* lds,
                                          unsigned* cws) {
    for (int l = 1; l < n; ++l) res_coarsen<T, D3>(lev[l - 1], lev[l]);
    for (int l = 0; l < n - 1; ++l) {
        const RLevel<T>& L = lev[l];
        if (L.ol >= 0)
            res_stage<T, D3, STYLE>(L, omega, lds);
        else
            cws[L.ocw + int(threadIdx.x)] = res_classify<T, D3, STYLE>(L, omega);
    }
    __syncthreads();
}

// The levels below the fine one: right-hand side in lev[1].ob, the corrected
// iterate left in lev[1].ox0.  Ends with a barrier.
template <typename T, bool D3, int STYLE>
__device__ __forceinline__ void res_below(const RLevel<T>* lev, int n, const Grid& gc, T omega,
                                          double tol, T* lds, unsigned* cws, CgLds& cg) {
    for (int l = 1; l < n - 1; ++l)
        res_down<T, D3, false, 4, STYLE>(lev[l], lev[l + 1], omega, lds, cws);
    {
        const RLevel<T>& C = lev[n - 1];
        coarse_cg_wg<T>(gc, C.Lx, D3 ? C.Ly : C.Lw, D3 ? C.Lw : nullptr, C.Lc, 0, lds + C.ob,
                        lds + C.ox0, tol, C.N + 64, cg);
    }
    __syncthreads();
    for (int l = n - 2; l >= 1; --l)
        res_up<T, D3, false, 4, STYLE>(lev[l], lev[l + 1], omega, lds, cws);
}

// b_in projected onto the active cells (mean-free there) into b: returns
// ||b||^2.  The sums run in the order of wg_project_rhs; cws: the level's class
// words.
__device__ __forceinline__ double res_project(const RLevel<double>& L, const unsigned* cws,
                                              const double* b_in, double* b, double* red) {
    const int cols = L.nx * L.ny, t0 = opaque(int(threadIdx.x));
    auto active = [&](int c) {
        const int k = int((unsigned long long)unsigned(c) * L.mc >> 32), part = k / L.seg;
        return ((cws[L.ocw + c - (k - part) * cols] >> (2 * (k - part * L.seg))) & 3u) != 1u;
    };
    double sb = 0.0, cnt = 0.0;
    for (int c = t0; c < L.N; c += int(blockDim.x))
        if (active(c)) {
            sb += b_in[c];
            cnt += 1.0;
        }
    sb = wg_sum(sb, red);
    cnt = wg_sum(cnt, red);
    const double mean = cnt > 0.0 ? sb / cnt : 0.0;
    double b2 = 0.0;
    for (int c = t0; c < L.N; c += int(blockDim.x)) {
        const double v = active(c) ? b_in[c] - mean : 0.0;
        b[c] = v;
        b2 += v * v;
    }
    return wg_sum(b2, red);
}

// FP64 V-cycles on A x = b_in until ||r|| <= tol ||b||; x and b (scratch) in
// global memory.  As solve_one's general path, with the norm taken by the first
// pre-smoothing sweep of the next V-cycle, and in the RS_TILED style: one fused
// multiply-add where RS_SEQ divides, the children summed pair by pair.  The
// solutions differ from the general path's by rounding: 2e-18 (128^2) to 2e-15
// (90 x 44) of their norm over seven sizes in 2D and 3D, after the same V-cycles.
template <bool D3>
__device__ __forceinline__ void res_solve64(const ResPlan64& P, double omega, const double* b_in,
                                            double* xg, double* b, double tol, int max_vcycles,
                                            WgLds& S, ResLds& R, int* status, int* vcycles,
                                            double* rel) {
    constexpr int M = kResRows;
    double* lds = R.raw;
    const int n = P.n;
    res_setup<double, D3, RS_TILED>(P.lev, n, omega, lds, R.cws);
    const RLevel<double>& F = P.lev[0];
    using Lev = ResLev<double, M, D3, false, false, RS_TILED>;
    const double b2 = res_project(F, R.cws, b_in, b, S.red);
    *status = WL_OK;
    *vcycles = 0;
    *rel = 0.0;
    if (b2 == 0.0) {
        for (int c = int(threadIdx.x); c < F.N; c += int(blockDim.x)) xg[c] = 0.0;
        __syncthreads();
        return;
    }
    double* X = lds + F.ox0;
    auto bf = [&](int, int c) { return b[c]; };
    auto nop = [](int, double) {};
    double x[M];  // what stays in registers below the fine level
    {
        Lev U(F, omega, lds, R.cws);
        U.get(xg);
        U.publish(X, false);
        U.save(x);
    }
    int k = 0, st = WL_OK;
    double r2;
    for (;;) {
        {
            Lev U(F, omega, lds, R.cws);
            U.load(x);
            r2 = wg_sum(U.template pass<RK_SWEEP, true>(X, bf, nop), S.red);
            if (r2 <= tol * tol * b2 || k >= max_vcycles || !isfinite(r2)) break;
            U.publish(X, false);  // the sums' barrier followed the pass
            U.template pass<RK_SWEEP, false>(X, bf, nop);
            U.publish(X, true);
            U.restrict_to(X, bf, lds + P.lev[1].ob, lds + F.ot, true);
            U.save(x);
        }
        res_below<double, D3, RS_TILED>(P.lev, n, P.gc, omega, 1e-10, lds, R.cws, S.cg);
        Lev U(F, omega, lds, R.cws);
        U.load(x);
        U.prolong(P.lev[1], lds + P.lev[1].ox0);
        U.publish(X, true);
        U.template pass<RK_SWEEP, false>(X, bf, nop);
        U.publish(X, true);
        U.template pass<RK_SWEEP, false>(X, bf, nop);
        U.publish(X, true);
        U.save(x);
        ++k;
    }
    if (!isfinite(r2))
        st = WL_ERR_NONFINITE;
    else if (!(r2 <= tol * tol * b2))
        st = WL_ERR_NOT_CONVERGED;
    // the measured iterate is the published one
    for (int c = int(threadIdx.x); c < F.N; c += int(blockDim.x)) xg[c] = X[c];
    __syncthreads();
    *status = st;
    *vcycles = k;
    *rel = sqrt(r2 / b2);
}

// FP32 V-cycles (kWgMixedInner per outer iteration, from zero) under the FP64
// defect correction x += e, until ||r||^2 <= tol2 (see wg_solve_mixed); b is
// projected already, the classes of P.fine and P.lev set up.
template <bool D3>
__device__ __forceinline__ int res_solve_mixed(const ResPlan32& P, float omega, double* xg,
                                               const double* b, double tol2, int max_vcycles,
                                               WgLds& S, ResLds& R, int* vcycles, double* r2_out) {
    constexpr int M = kResRows;
    float* lds = reinterpret_cast<float*>(R.raw);
    const int n = P.n;
    int k = 0, status = WL_OK;
    double r2 = 0.0;
    for (;;) {
        float e[M];
        {
            ResLev<double, M, D3, false, false, RS_SEQ> U(P.fine, 1.0, R.raw, R.cws);
            double* X = R.raw;
            U.get(xg);
            U.publish(X, false);
            auto bf = [&](int, int c) { return b[c]; };
            r2 = wg_sum(U.template pass<RK_RESID, true>(X, bf, [&](int m, double r) { e[m] = float(r); }),
                        S.red);
        }
        if (!isfinite(r2)) {
            status = WL_ERR_NONFINITE;
            break;
        }
        if (r2 <= tol2 || k >= max_vcycles) break;
        const int mm = min(kWgMixedInner, max_vcycles - k);
        const RLevel<float>& F = P.lev[0];
        using Lev = ResLev<float, M, D3, false, false, RS_SEQ>;
        float* X = lds + F.ox0;
        auto bf = [&](int m, int) { return e[m]; };
        auto nop = [](int, float) {};
        float x[M];
#pragma unroll
        for (int m = 0; m < M; ++m) x[m] = 0.0f;
        for (int v = 0; v < mm; ++v) {
            {
                Lev U(F, omega, lds, R.cws);
                U.load(x);
                if (v == 0)
                    U.template pass<RK_ZERO, false>(nullptr, bf, nop);
                else
                    U.template pass<RK_SWEEP, false>(X, bf, nop);
                U.publish(X, true);
                U.template pass<RK_SWEEP, false>(X, bf, nop);
                U.publish(X, true);
                U.restrict_to(X, bf, lds + P.lev[1].ob, lds + F.ot, true);
                U.save(x);
            }
            res_below<float, D3, RS_SEQ>(P.lev, n, P.gc, omega, 1e-6, lds, R.cws, S.cg);
            Lev U(F, omega, lds, R.cws);
            U.load(x);
            U.prolong(P.lev[1], lds + P.lev[1].ox0);
            U.publish(X, true);
            U.template pass<RK_SWEEP, false>(X, bf, nop);
            U.publish(X, true);
            U.template pass<RK_SWEEP, false>(X, bf, nop);
            U.publish(X, true);
            U.save(x);
        }
        {
            const RGeo q = res_geo(F);
#pragma unroll
            for (int m = 0; m < M; ++m)
                if (m < q.cnt) xg[q.c0 + m * F.nx * F.ny] += double(x[m]);
        }
        __syncthreads();
        k += mm;
    }
    if (status == WL_OK && !(r2 <= tol2)) status = WL_ERR_NOT_CONVERGED;
    __syncthreads();
    *vcycles = k;
    *r2_out = r2;
    return status;
}

// ------------------------------------------------------------- host planning
// LDS layout of a resident hierarchy whose fine level keeps one buffer that
// overlaps the coarser levels; false when it does not fit.  reserve: bytes the
// overlapped region must have at least; ncls: class-word slots used so far.
template <typename T>
inline bool res_plan_lds(RLevel<T>* lev, int n, bool d3, size_t reserve, int& ncls) {
    const int limit = int(kResBytes / sizeof(T));
    int used = res_layout(lev, 1, n, 0);
    lev[0].ox0 = lev[0].ox1 = 0;
    // FP64 (RS_TILED): the fine level's restriction sums; FP32 (RS_SEQ): its
    // residual takes its iterate's place (see restrict_to)
    if (d3 && sizeof(T) == 8) {
        lev[0].ot = used;
        used += lev[0].N / 4;
    }
    used = used > lev[0].N ? used : lev[0].N;
    const int res = int((reserve + sizeof(T) - 1) / sizeof(T));
    used = used > res ? used : res;
    if (used > limit) return false;
    res_stage_layout(lev, 1, n, used, limit, d3);
    for (int l = 0; l < n - 1; ++l) {
        if (lev[l].ol >= 0) continue;
        if (ncls == kResGlobal) return false;
        lev[l].ocw = ncls++ * kResThreads;
    }
    return true;
}

}  // namespace wl
