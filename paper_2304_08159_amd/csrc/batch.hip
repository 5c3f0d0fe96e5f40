// Batched Poisson solves for many small problems: a persistent kernel per kind
// of request (a fine level resident in one workgroup, in 2D or 3D and FP64 or
// mixed precision; larger ones) whose workgroups take requests from a device
// work queue (an atomic head index over the kind's requests) until it is empty,
// the kinds side by side; a request is solved entirely by
// the workgroup that took it, with the same method as wl_poisson_solve
// (Sec. 2's project!: matrix-free GMG, damped Jacobi, sum restriction,
// cell-centred linear prolongation, coarse coefficients = 1/2 the covered fine
// faces, minimum-norm coarsest solve) in FP64, or in FP32 V-cycles with an
// FP64 defect correction around them (per request).  Every reduction is a
// fixed-order workgroup sum, so a request's result does not depend on which
// workgroup solved it or on the rest of the batch.
#include <algorithm>
#include <cmath>
#include <cstring>
#include <mutex>
#include <string>
#include <vector>

#include "wl_fork.h"
#include "wl_internal.h"
#include "wl_ressolve.h"
#include "wl_wg.h"
#include "wl_wgsolve.h"

namespace wl {
namespace {

constexpr int kBatchThreads = 1024;
constexpr size_t kBatchMaxCells = 262144;  // per request (e.g. 512^2, 64^3)

using BatchLevel = WgLevel<double>;  // uniform = 0, Lc = 1 (coefficients from the request)

struct BatchReq {
    int nlev;
    double tol, omega;
    int max_vcycles;
    int mixed;                            // FP32 inner V-cycles, FP64 outer
    int kind;                             // general path (0) or which resident one
    const double* b_in;
    double* x;                            // resident path: solution, projected right-hand side
    double* b;
    union {
        struct {
            BatchLevel lev[kMaxLevels];        // mixed: only the fine level (FP64 x, b, L)
            WgLevel<float> lev32[kMaxLevels];  // mixed: the FP32 hierarchy
        };
        ResPlan64 p64;
        ResPlan32 p32;
    };
};
// the request table is part of the footprint: the resident plans must not grow it
static_assert(sizeof(ResPlan64) <= sizeof(BatchLevel) * kMaxLevels + sizeof(WgLevel<float>) * kMaxLevels &&
                  sizeof(ResPlan32) <= sizeof(BatchLevel) * kMaxLevels + sizeof(WgLevel<float>) * kMaxLevels,
              "resident plan larger than the general one");

struct BatchRes {
    int status, vcycles;
    double rel;
};

__device__ void solve_one(const BatchReq& q, BatchRes& res, WgLds& S) {
    const BatchLevel& F = q.lev[0];
    const int nlev = q.nlev;
    const double w = q.omega;
    double* red = S.red;
    double* x = F.x[0];
    double* x1 = F.x[1];
    const int N = int(cells(F.g));
    for (int l = 1; l < nlev; ++l) wg_coarsen<double>(q.lev[l - 1], q.lev[l]);
    // right-hand side projected onto the active cells, mean-free there
    const XAccess<double, XM_ZERO> Z{nullptr};
    const Coeffs<double> C = wg_coeffs(F);
    double sb = 0.0, cnt = 0.0;
    for (int c = threadIdx.x; c < N; c += blockDim.x) {
        int i, j, k;
        wg_coords(F.g, c, i, j, k);
        double xI, Ax, D;
        apply_row<double, XM_ZERO, false>(F.g, Z, C, i, j, k, xI, Ax, D);
        if (D > 0.0) {
            sb += q.b_in[c];
            cnt += 1.0;
        }
    }
    sb = wg_sum(sb, red);
    cnt = wg_sum(cnt, red);
    const double mean = cnt > 0.0 ? sb / cnt : 0.0;
    double b2 = 0.0;
    for (int c = threadIdx.x; c < N; c += blockDim.x) {
        int i, j, k;
        wg_coords(F.g, c, i, j, k);
        double xI, Ax, D;
        apply_row<double, XM_ZERO, false>(F.g, Z, C, i, j, k, xI, Ax, D);
        const double bv = D > 0.0 ? q.b_in[c] - mean : 0.0;
        F.b[c] = bv;
        b2 += bv * bv;
    }
    __syncthreads();
    b2 = wg_sum(b2, red);
    if (b2 == 0.0) {
        for (int c = threadIdx.x; c < N; c += blockDim.x) x[c] = 0.0;
        __syncthreads();
        if (threadIdx.x == 0) res = BatchRes{WL_OK, 0, 0.0};
        __syncthreads();
        return;
    }
    const double tol2 = q.tol * q.tol * b2;
    // first sweep of the first V-cycle, with the norm of the initial residual
    double r2 = wg_sweep<double, XM_PLAIN>(F, XAccess<double, XM_PLAIN>{x}, F.b, w,
                                           x1, true, red);
    int k = 0;
    int status = WL_OK;
    while (!(r2 <= tol2) && k < q.max_vcycles) {
        if (!isfinite(r2)) {
            status = WL_ERR_NONFINITE;
            break;
        }
        if (nlev == 1) {
            coarse_cg_wg<double>(F.g, F.L[0], F.L[1], F.L[2], F.Lc, 0, F.b, x, 1e-10, N + 64, S.cg);
            __syncthreads();
        } else {
            wg_sweep<double, XM_PLAIN>(F, XAccess<double, XM_PLAIN>{x1}, F.b, w, x, false, red);
            wg_restrict<double>(F, x, F.b, q.lev[1]);
            wg_vcycle_tail<double>(&q.lev[1], nlev - 1, w, 1e-10, S);
            const BatchLevel& C1 = q.lev[1];
            wg_prolong<double>(F, C1, C1.x[1], x);
            wg_sweep<double, XM_PLAIN>(F, XAccess<double, XM_PLAIN>{x}, F.b, w, x1, false, red);
            wg_sweep<double, XM_PLAIN>(F, XAccess<double, XM_PLAIN>{x1}, F.b, w, x, false, red);
        }
        ++k;
        r2 = wg_sweep<double, XM_PLAIN>(F, XAccess<double, XM_PLAIN>{x}, F.b, w, x1,
                                        true, red);
    }
    if (status == WL_OK && !isfinite(r2)) status = WL_ERR_NONFINITE;
    if (status == WL_OK && !(r2 <= tol2)) status = WL_ERR_NOT_CONVERGED;
    if (threadIdx.x == 0) res = BatchRes{status, k, sqrt(r2 / b2)};
    __syncthreads();
}

// Mixed precision (see wg_solve_mixed): the FP32 coefficients of every level
// from the request's FP64 ones, the projected right-hand side, then the
// defect-correction loop.
__device__ void solve_one_mixed(const BatchReq& q, BatchRes& res, WgLds& S) {
    const BatchLevel& F = q.lev[0];
    wg_coeffs32(F, q.lev32, q.nlev);
    const double b2 = wg_project_rhs(F, q.b_in, S.red);
    if (b2 == 0.0) {
        const int N = int(cells(F.g));
        for (int c = threadIdx.x; c < N; c += blockDim.x) F.x[0][c] = 0.0;
        __syncthreads();
        if (threadIdx.x == 0) res = BatchRes{WL_OK, 0, 0.0};
        __syncthreads();
        return;
    }
    double r2 = 0.0;
    int k = 0;
    const int st = wg_solve_mixed(F, q.lev32, q.nlev, float(q.omega), q.tol * q.tol * b2, 0.0,
                                  q.max_vcycles, S, &k, &r2);
    if (threadIdx.x == 0) res = BatchRes{st, k, sqrt(r2 / b2)};
    __syncthreads();
}

// A request on the resident path (wl_ressolve.h).
template <bool D3, bool MIXED>
__device__ __forceinline__ void solve_resident(const BatchReq& q, BatchRes& res, WgLds& S,
                                               ResLds& R) {
    int st = WL_OK, k = 0;
    double rel = 0.0;
    if (MIXED) {
        const ResPlan32& P = q.p32;
        const RLevel<double>& F = P.fine;
        // FP32 coefficients of the fine level, the classes of both
        for (int c = int(threadIdx.x); c < F.N; c += int(blockDim.x)) {
            const_cast<float*>(P.lev[0].Lx)[c] = float(F.Lx[c]);
            if (D3) const_cast<float*>(P.lev[0].Ly)[c] = float(F.Ly[c]);
            const_cast<float*>(P.lev[0].Lw)[c] = float(F.Lw[c]);
        }
        R.cws[F.ocw + int(threadIdx.x)] = res_classify<double, D3, RS_SEQ>(F, 1.0);
        __syncthreads();
        res_setup<float, D3, RS_SEQ>(P.lev, P.n, float(q.omega), reinterpret_cast<float*>(R.raw), R.cws);
        const double b2 = res_project(F, R.cws, q.b_in, q.b, S.red);
        if (b2 == 0.0) {
            for (int c = int(threadIdx.x); c < F.N; c += int(blockDim.x)) q.x[c] = 0.0;
            __syncthreads();
        } else {
            double r2 = 0.0;
            st = res_solve_mixed<D3>(P, float(q.omega), q.x, q.b, q.tol * q.tol * b2,
                                     q.max_vcycles, S, R, &k, &r2);
            rel = sqrt(r2 / b2);
        }
    } else {
        res_solve64<D3>(q.p64, q.omega, q.b_in, q.x, q.b, q.tol, q.max_vcycles, S, R, &st, &k, &rel);
    }
    if (threadIdx.x == 0) res = BatchRes{st, k, rel};
    __syncthreads();
}

// Persistent kernels: each workgroup takes the next request from the queue
// until none is left (every workgroup reaches the exit).  One kernel per kind
// of request: at 1024 threads a wave has 128 registers, and each resident kind
// by itself spills 19 (2D FP64), 12 (2D mixed), 72 (3D FP64) and 20 (3D mixed) of
// them, all kinds inlined into one kernel 686; as functions that one kernel calls,
// the 2D requests took 1.09 instead of 0.82 ms (128^2, FP64), their descriptors
// and coefficients then read through generic pointers.
__global__ __launch_bounds__(kBatchThreads) void k_poisson_batch(const BatchReq* __restrict__ reqs,
                                                                 int count, unsigned* head,
                                                                 BatchRes* __restrict__ res) {
    __shared__ WgLds S;
    __shared__ int take;
    for (;;) {
        if (threadIdx.x == 0) take = int(atomicAdd(head, 1u));
        __syncthreads();
        const int r = take;
        __syncthreads();
        if (r >= count) return;
        if (reqs[r].mixed)
            solve_one_mixed(reqs[r], res[r], S);
        else
            solve_one(reqs[r], res[r], S);
    }
}

template <bool D3, bool MIXED>
__global__ __launch_bounds__(kBatchThreads) void k_poisson_resident(
    const BatchReq* __restrict__ reqs, int count, unsigned* head, BatchRes* __restrict__ res) {
    __shared__ WgLds S;
    __shared__ ResLds R;
    __shared__ int take;
    for (;;) {
        if (threadIdx.x == 0) take = int(atomicAdd(head, 1u));
        __syncthreads();
        const int r = take;
        __syncthreads();
        if (r >= count) return;
        solve_resident<D3, MIXED>(reqs[r], res[r], S, R);
    }
}

// Kinds of request, each served by a kernel of its own.
enum { kGeneral = 0, kRes2 = 1, kRes2Mixed = 2, kRes3 = 3, kRes3Mixed = 4, kKinds = 5 };

// The resident plan of a request whose general one is in q (its scratch
// arrays serve both: the sweep buffers, which the resident path does not need,
// hold w / D).  Taken when the fine level splits into segments of at most 16
// cells (up to 16,384 cells) and the levels fit the LDS; 256 requests of 128^2 in
// FP64 then take 2.17 instead of 4.31 ms, 200 of 192 x 64 in FP32 with FP64
// correction 1.6 instead of 4.1 ms.  Larger fine levels do not fit the LDS and
// keep the general path.
void plan_resident(BatchReq& q) {
    const int nlev = q.nlev;
    if (nlev < 2 || nlev > kResLevels) return;
    const BatchLevel& F = q.lev[0];
    const bool d3 = F.g.ndim == 3;
    auto level = [&](auto& out, const auto& L, double Lc, bool last) {
        using V = std::remove_const_t<std::remove_pointer_t<decltype(out.Lx)>>;
        const V* Lp[3] = {L.L[0], L.L[1], L.L[2]};
        return res_plan_level<V>(L.g, Lp, V(Lc), V(0), kBatchThreads, kResRows, last, out);
    };
    int ncls = 0;
    double* x = F.x[0];
    double* b = F.b;
    double Lc = 1.0;
    if (q.mixed) {
        ResPlan32 P{};
        P.n = nlev;
        P.gc = q.lev32[nlev - 1].g;
        if (!level(P.fine, F, 1.0, false)) return;
        P.fine.ocw = kResThreads * ncls++;
        for (int l = 0; l < nlev; ++l, Lc *= d3 ? 2.0 : 1.0) {
            if (!level(P.lev[l], q.lev32[l], Lc, l == nlev - 1)) return;
            P.lev[l].wd = q.lev32[l].x[0];
        }
        if (!res_plan_lds(P.lev, nlev, d3, size_t(P.fine.N) * sizeof(double), ncls)) return;
        for (int l = 1; l < nlev - 1; ++l)
            if (P.lev[l].seg > 4) return;
        q.kind = d3 ? kRes3Mixed : kRes2Mixed;
        q.p32 = P;
    } else {
        ResPlan64 P{};
        P.n = nlev;
        P.gc = q.lev[nlev - 1].g;
        for (int l = 0; l < nlev; ++l, Lc *= d3 ? 2.0 : 1.0) {
            if (!level(P.lev[l], q.lev[l], Lc, l == nlev - 1)) return;
            P.lev[l].wd = l == 0 ? q.lev[0].x[1] : q.lev[l].x[0];
        }
        if (!res_plan_lds(P.lev, nlev, d3, 0, ncls)) return;
        for (int l = 1; l < nlev - 1; ++l)
            if (P.lev[l].seg > 4) return;
        q.kind = d3 ? kRes3 : kRes2;
        q.p64 = P;
    }
    q.x = x;
    q.b = b;
}

// Checks one request and fills its descriptor, carving its level arrays.
wl_status plan_one(const wl_batch_request& in, Carver& c, BatchReq& q) {
    const int ndim = in.ndim;
    if (ndim != 2 && ndim != 3) return set_error("batch request: ndim must be 2 or 3"), WL_ERR_INVALID_ARG;
    if (ndim == 2 && in.n[2] != 1) {
        set_error("batch request: 2D problems need n[2] == 1");
        return WL_ERR_INVALID_ARG;
    }
    for (int d = 0; d < ndim; ++d)
        if (in.n[d] < 2) {
            set_error("batch request: every direction needs at least 2 cells");
            return WL_ERR_INVALID_ARG;
        }
    const size_t N = size_t(in.n[0]) * in.n[1] * in.n[2];
    if (N > kBatchMaxCells) {
        set_error("batch request larger than 262144 cells (use wl_poisson_solve)");
        return WL_ERR_INVALID_ARG;
    }
    if (!(in.tol >= 0.0) || in.max_vcycles < 0) {
        set_error("batch request: tol must be >= 0 and max_vcycles >= 0");
        return WL_ERR_INVALID_ARG;
    }
    const int nlev = auto_levels(ndim, in.n, 0);
    int m[3] = {in.n[0], in.n[1], in.n[2]};
    for (int l = 1; l < nlev; ++l)
        for (int d = 0; d < ndim; ++d) m[d] /= 2;
    if (size_t(m[0]) * m[1] * m[2] > size_t(kCoarseMax)) {
        set_error("batch request: coarsest multigrid level exceeds 1024 cells");
        return WL_ERR_INVALID_ARG;
    }
    if (in.mixed != 0 && in.mixed != 1) {
        set_error("batch request: mixed must be 0 or 1");
        return WL_ERR_INVALID_ARG;
    }
    q = BatchReq{};
    q.nlev = nlev;
    q.tol = in.tol;
    q.omega = 2.0 * ndim / (2.0 * ndim + 1.0);
    q.max_vcycles = in.max_vcycles;
    q.mixed = in.mixed;
    q.b_in = static_cast<const double*>(in.b);
    int n[3] = {in.n[0], in.n[1], in.n[2]};
    if (in.mixed) {
        // FP64 fine level (x, projected b, the request's coefficients) and an
        // FP32 hierarchy (e, sweep buffer, right-hand side, coefficients)
        BatchLevel& F = q.lev[0];
        F.g = Grid{n[0], n[1], n[2], in.periodic[0] != 0, in.periodic[1] != 0,
                   ndim == 3 && in.periodic[2] != 0, ndim};
        F.Lc = 1.0;
        F.uniform = 0;
        const size_t N0 = size_t(n[0]) * n[1] * n[2];
        F.x[0] = static_cast<double*>(in.x);
        F.x[1] = nullptr;
        F.b = c.take<double>(N0);
        const double* co = static_cast<const double*>(in.coeffs);
        for (int d = 0; d < 3; ++d) F.L[d] = d < ndim ? const_cast<double*>(co + d * N0) : nullptr;
        for (int l = 0; l < nlev; ++l) {
            WgLevel<float>& L = q.lev32[l];
            L.g = Grid{n[0], n[1], n[2], F.g.per0, F.g.per1, F.g.per2, ndim};
            L.Lc = 1.0f;
            L.uniform = 0;
            const size_t Nl = size_t(n[0]) * n[1] * n[2];
            L.x[0] = c.take<float>(Nl);
            L.x[1] = c.take<float>(Nl);
            L.b = c.take<float>(Nl);
            for (int d = 0; d < 3; ++d) L.L[d] = d < ndim ? c.take<float>(Nl) : nullptr;
            for (int d = 0; d < ndim; ++d) n[d] /= 2;
        }
        plan_resident(q);
        return WL_OK;
    }
    for (int l = 0; l < nlev; ++l) {
        BatchLevel& L = q.lev[l];
        L.g = Grid{n[0], n[1], n[2], in.periodic[0] != 0, in.periodic[1] != 0,
                   ndim == 3 && in.periodic[2] != 0, ndim};
        L.Lc = 1.0;
        L.uniform = 0;
        const size_t Nl = size_t(n[0]) * n[1] * n[2];
        if (l == 0) {
            L.x[0] = static_cast<double*>(in.x);
            L.x[1] = c.take<double>(Nl);
            L.b = c.take<double>(Nl);
            const double* co = static_cast<const double*>(in.coeffs);
            for (int d = 0; d < 3; ++d) L.L[d] = d < ndim ? const_cast<double*>(co + d * Nl) : nullptr;
        } else {
            L.x[0] = c.take<double>(Nl);
            L.x[1] = c.take<double>(Nl);
            L.b = c.take<double>(Nl);
            for (int d = 0; d < 3; ++d) L.L[d] = d < ndim ? c.take<double>(Nl) : nullptr;
        }
        for (int d = 0; d < ndim; ++d) n[d] /= 2;
    }
    plan_resident(q);
    return WL_OK;
}

struct BatchLayout {
    BatchReq* dev_reqs = nullptr;
    BatchRes* dev_res = nullptr;
    unsigned* dev_head = nullptr;
};

// Checks every request and carves the batch's device arrays from c; with
// table non-null, also fills the count request descriptors there, request r
// at place[r]; without, place (when given) receives their kinds.
wl_status plan(const wl_batch_request* reqs, int count, Carver& c, BatchLayout& lay,
               BatchReq* table, int* place = nullptr) {
    if (count < 0) return set_error("count must be >= 0"), WL_ERR_INVALID_ARG;
    if (count > 0 && !reqs) return set_error("reqs is NULL"), WL_ERR_INVALID_ARG;
    lay.dev_reqs = c.take<BatchReq>(size_t(count > 0 ? count : 1));
    lay.dev_res = c.take<BatchRes>(size_t(count > 0 ? count : 1));
    lay.dev_head = c.take<unsigned>(kKinds);  // within the 256 bytes one took
    for (int r = 0; r < count; ++r) {
        BatchReq q;
        const wl_status st = plan_one(reqs[r], c, q);
        if (st != WL_OK) {
            set_error("request " + std::to_string(r) + ": " + last_error_text());
            return st;
        }
        if (table)
            table[place[r]] = q;
        else if (place)
            place[r] = q.kind;
    }
    return WL_OK;
}

// ------------------------------------------------ no-allocation variant
// Device scratch of wl_poisson_batch_solve_noalloc: the request table, the
// results, the queue head and every request's level arrays, carved exactly as
// from a caller workspace.  One copy per GPU, held until the process ends.
constexpr size_t kNoAllocScratchBytes = size_t(32) << 20;
static __device__ __align__(256) char scratch[kNoAllocScratchBytes];

// Device address of this GPU's copy of `scratch`, looked up once per device
// with that device current (the host-side name of the array is not a device
// address and must never be handed to a kernel or a copy).
constexpr int kMaxDevices = 64;
constexpr int kNoAllocMaxRequests = 256;
std::mutex g_noalloc_host_mu;
BatchReq g_noalloc_table[kNoAllocMaxRequests];
BatchRes g_noalloc_res[kNoAllocMaxRequests];
int g_noalloc_place[kNoAllocMaxRequests];
SideStreams g_noalloc_side[kMaxDevices];  // made by a GPU's first call with several kinds, kept
std::mutex g_scratch_mu;
void* g_scratch_ptr[kMaxDevices] = {};

wl_status scratch_for_current_device(void** out, int* device) {
    int dev = 0;
    WL_CHECK_HIP(hipGetDevice(&dev));
    if (dev < 0 || dev >= kMaxDevices) {
        set_error("device index beyond the no-allocation scratch table");
        return WL_ERR_INVALID_ARG;
    }
    std::lock_guard<std::mutex> lock(g_scratch_mu);
    if (!g_scratch_ptr[dev]) {
        void* ptr = nullptr;
        WL_CHECK_HIP(hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch)));
        if (!ptr || reinterpret_cast<uintptr_t>(ptr) % 256) {
            set_error("scratch symbol address is null or misaligned");
            return WL_ERR_HIP;
        }
        g_scratch_ptr[dev] = ptr;
    }
    *out = g_scratch_ptr[dev];
    *device = dev;
    return WL_OK;
}

int compute_units() {
    static const int n = [] {
        int dev = 0, v = 0;
        if (hipGetDevice(&dev) != hipSuccess) return 256;
        if (hipDeviceGetAttribute(&v, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess)
            return 256;
        return v > 0 ? v : 256;
    }();
    return n;
}

// Plans the batch into workspace (>= its footprint, 256-byte aligned),
// uploads the request table (host staging: table, count entries) and zero
// queue heads, runs the persistent kernels and copies the results back through
// res (count entries; synchronises).
//
// The kinds run side by side, each on a stream: a request keeps one compute
// unit busy whatever its kind, so the batch takes as long as its longest
// requests and not as all kinds one after another (two requests of each of the
// five kinds 7.09 -> 3.30 ms, the longest kind by itself 2.76; 16 of each 7.80 ->
// 4.04).  A stream costs some 35 us to make and release, so a batch of one kind
// makes none; with one request of 16^2 cells in either precision the two come
// out even (0.44 ms).  side: where the streams are kept (null: made and released
// here).
wl_status batch_run(const wl_batch_request* reqs, int count, void* workspace, size_t ws_bytes,
                    void* hip_stream, wl_batch_result* results, BatchReq* table, BatchRes* res,
                    int* place, SideStreams* side) {
    if (reinterpret_cast<uintptr_t>(workspace) % 256)
        return set_error("workspace must be 256-byte aligned"), WL_ERR_INVALID_ARG;
    for (int r = 0; r < count && reqs; ++r)
        if (!reqs[r].coeffs || !reqs[r].x || !reqs[r].b) {
            set_error("request " + std::to_string(r) + ": coeffs / x / b is NULL");
            return WL_ERR_INVALID_ARG;
        }
    Carver need;
    BatchLayout dry;
    WL_TRY(plan(reqs, count, need, dry, nullptr, place));
    if (ws_bytes < need.off) {
        set_error("workspace smaller than wl_poisson_batch_footprint");
        return WL_ERR_OUT_OF_MEMORY;
    }
    Carver c;
    c.base = static_cast<char*>(workspace);
    BatchLayout lay;
    // the requests of each kind together, in the caller's order
    int n[kKinds] = {}, start[kKinds], at[kKinds];
    for (int r = 0; r < count; ++r) ++n[place[r]];
    for (int k = 0, sum = 0; k < kKinds; sum += n[k++]) start[k] = at[k] = sum;
    for (int r = 0; r < count; ++r) place[r] = at[place[r]]++;
    WL_TRY(plan(reqs, count, c, lay, table, place));
    hipStream_t s = reinterpret_cast<hipStream_t>(hip_stream);
    // request table and zero queue heads (the no-allocation scratch keeps
    // the last call's contents, so the heads are cleared on every call)
    const unsigned zero[kKinds] = {};
    WL_CHECK_HIP(hipMemcpyAsync(lay.dev_reqs, table, sizeof(BatchReq) * size_t(count),
                                hipMemcpyHostToDevice, s));
    WL_CHECK_HIP(hipMemcpyAsync(lay.dev_head, zero, sizeof(zero), hipMemcpyHostToDevice, s));
    const int kinds = int(std::count_if(n, n + kKinds, [](int c) { return c > 0; }));
    struct Own : SideStreams {  // released once the fork below has ended
        ~Own() { release(); }
    } own;
    SideStreams& streams = side ? *side : own;
    streams.make(kinds - 1);
    Fork fork(streams, s);
    if (kinds > 1) WL_TRY(fork.open());
    for (int k = 0; k < kKinds; ++k) {
        if (n[k] == 0) continue;
        const int grid = std::min(n[k], compute_units());
        const BatchReq* q = lay.dev_reqs + start[k];
        BatchRes* out = lay.dev_res + start[k];
        unsigned* head = lay.dev_head + k;
        hipStream_t ks;
        WL_TRY(fork.next(&ks));
        switch (k) {
            case kRes2: k_poisson_resident<false, false><<<grid, kBatchThreads, 0, ks>>>(q, n[k], head, out); break;
            case kRes2Mixed: k_poisson_resident<false, true><<<grid, kBatchThreads, 0, ks>>>(q, n[k], head, out); break;
            case kRes3: k_poisson_resident<true, false><<<grid, kBatchThreads, 0, ks>>>(q, n[k], head, out); break;
            case kRes3Mixed: k_poisson_resident<true, true><<<grid, kBatchThreads, 0, ks>>>(q, n[k], head, out); break;
            default: k_poisson_batch<<<grid, kBatchThreads, 0, ks>>>(q, n[k], head, out); break;
        }
        WL_CHECK_HIP(hipGetLastError());
    }
    WL_TRY(fork.join());
    WL_CHECK_HIP(hipMemcpyAsync(res, lay.dev_res, sizeof(BatchRes) * size_t(count),
                                hipMemcpyDeviceToHost, s));
    WL_CHECK_HIP(hipStreamSynchronize(s));
    wl_status worst = WL_OK;
    for (int r = 0; r < count; ++r) {
        const BatchRes& o = res[place[r]];
        results[r].status = o.status;
        results[r].vcycles = o.vcycles;
        results[r].rel_resid = o.rel;
        if (o.status != WL_OK && worst == WL_OK) worst = wl_status(o.status);
    }
    if (worst == WL_ERR_NOT_CONVERGED) set_error("some batch requests reached max_vcycles");
    if (worst == WL_ERR_NONFINITE) set_error("non-finite residual in a batch request");
    return worst;
}

}  // namespace
}  // namespace wl

using namespace wl;

extern "C" {

wl_status wl_poisson_batch_footprint(const wl_batch_request* reqs, int count, size_t* bytes) {
    clear_error();
    if (!bytes) return set_error("bytes is NULL"), WL_ERR_INVALID_ARG;
    Carver c;
    BatchLayout lay;
    WL_TRY(plan(reqs, count, c, lay, nullptr));
    *bytes = c.off;
    return WL_OK;
}

wl_status wl_poisson_batch_solve(const wl_batch_request* reqs, int count, void* workspace,
                                 size_t ws_bytes, void* hip_stream, wl_batch_result* results) {
    clear_error();
    if (count == 0) return WL_OK;
    if (!workspace || !results) return set_error("workspace / results is NULL"), WL_ERR_INVALID_ARG;
    if (count < 0) return set_error("count must be >= 0"), WL_ERR_INVALID_ARG;
    if (!reqs) return set_error("reqs is NULL"), WL_ERR_INVALID_ARG;
    std::vector<BatchReq> table(static_cast<size_t>(count));
    std::vector<BatchRes> res(static_cast<size_t>(count));
    std::vector<int> place(static_cast<size_t>(count));
    return batch_run(reqs, count, workspace, ws_bytes, hip_stream, results, table.data(),
                     res.data(), place.data(), nullptr);
}

wl_status wl_poisson_batch_solve_noalloc(const wl_batch_request* reqs, int count,
                                         void* hip_stream, wl_batch_result* results) {
    clear_error();
    if (count == 0) return WL_OK;
    if (!results) return set_error("results is NULL"), WL_ERR_INVALID_ARG;
    if (count < 0 || count > kNoAllocMaxRequests) {
        set_error("the no-allocation entry point takes 0 to " +
                  std::to_string(kNoAllocMaxRequests) + " requests per call");
        return WL_ERR_INVALID_ARG;
    }
    Carver need;
    BatchLayout dry;
    WL_TRY(plan(reqs, count, need, dry, nullptr));
    if (need.off > kNoAllocScratchBytes) {
        set_error("batch needs " + std::to_string(need.off) + " bytes of scratch; the "
                  "no-allocation entry point holds " + std::to_string(kNoAllocScratchBytes) +
                  " (use wl_poisson_batch_solve with a workspace)");
        return WL_ERR_INVALID_ARG;
    }
    void* ws = nullptr;
    int dev = 0;
    WL_TRY(scratch_for_current_device(&ws, &dev));
    // fixed host staging (no heap); one call at a time in this process
    std::lock_guard<std::mutex> lock(g_noalloc_host_mu);
    return batch_run(reqs, count, ws, kNoAllocScratchBytes, hip_stream, results, g_noalloc_table,
                     g_noalloc_res, g_noalloc_place, &g_noalloc_side[dev]);
}

}  // extern "C"
