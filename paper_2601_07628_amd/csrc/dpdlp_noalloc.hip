// KKT evaluation that allocates nothing (dpdlp_kkt_noalloc in dpdlp.h), for
// callers that cannot call hipMalloc: code under HIP graph capture, tight
// serving loops.  It evaluates the relative KKT error of App. B.4 of an LP
// (or a diagonal QP, Sec. 6) given in CSR and CSC directly from the caller's
// device arrays, with per-column primal steps tau * col_scale_j^2 (the
// solver's scaled-space step mapped to the original space, so the result is
// the solver's own termination measure, the one dpdlp_kkt reports).
//
// Its only device memory beyond the inputs and outputs is the per-workgroup
// partial sums, kept in the file-scope array `scratch` below.  Every
// workgroup writes all of its slots on every call before the final kernel
// reads them, so nothing needs clearing; calls that overlap on one GPU share
// the array and race.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <cstdint>
#include <mutex>

#include "dpdlp_internal.h"
#include "dpdlp_kernels.h"

namespace {

constexpr int kNaThreads = 256;                 // threads per workgroup
constexpr int kNaLanesLog2 = 3, kNaLanes = 1 << kNaLanesLog2;      // lanes per row / column
constexpr int kNaLong = 8 * kNaLanes;           // entries from which a wave takes a segment
constexpr int kNaSegs = kNaThreads / kNaLanes;  // rows or columns per workgroup and round
constexpr int kNaMaxCount = 16777216;           // rows or columns of a call
constexpr int kNaRowQ = 3;                      // row-pass partial quantities
constexpr int kNaColQ = 4;                      // column-pass partial quantities
// Workgroups per pass at most: one round each up to 131072 rows or columns (a
// round is a chain of three memory round trips; eight rounds per workgroup
// and one pass after the other took 44 us for a 1M-nonzero LP, now 23), more
// rounds beyond, so that the final workgroup adds at most 4 partials per
// thread and quantity.
constexpr int kNaMaxBlocks = 4096;
constexpr int kNaFinish = 1024;                 // threads of the final workgroup
constexpr int kNaMaxDevices = 64;

}  // namespace

// Partial sums of both passes: [kNaRowQ][kNaMaxBlocks] then [kNaColQ][kNaMaxBlocks]
// (0.23 MB per GPU, held until the process ends).
static __device__ __align__(256) double scratch[(kNaRowQ + kNaColQ) * kNaMaxBlocks];

namespace {

std::mutex g_na_mu;
double *g_na_ptr[kNaMaxDevices] = {};

// Device address of `scratch` on the current device, looked up once per
// device (each GPU holds its own copy of the array at its own address).
int scratch_address(double **out)
{
    int dev = -1;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) {
        dpdlp::set_error(std::string("hipGetDevice: ") + hipGetErrorString(e));
        return DPDLP_E_HIP;
    }
    if (dev < 0 || dev >= kNaMaxDevices) {
        dpdlp::set_error("dpdlp_kkt_noalloc: device ordinal beyond 63");
        return DPDLP_E_NOT_SUPPORTED;
    }
    std::lock_guard<std::mutex> lk(g_na_mu);
    if (!g_na_ptr[dev]) {
        void *p = nullptr;
        e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
        if (e != hipSuccess || !p) {
            dpdlp::set_error(std::string("hipGetSymbolAddress(scratch): ") + hipGetErrorString(e));
            return DPDLP_E_HIP;
        }
        g_na_ptr[dev] = static_cast<double *>(p);
    }
    *out = g_na_ptr[dev];
    return DPDLP_OK;
}

__device__ __forceinline__ double clampd(double v, double lo, double hi)
{
    return v < lo ? lo : (v > hi ? hi : v);
}

// Fixed-order workgroup sum of NQ values; thread 0 writes part[q * nb + block].
template <int NQ>
__device__ void block_partials(double (&acc)[NQ], double *part, int nb, int block)
{
    __shared__ double s[NQ][kNaThreads / 64];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
#pragma unroll
    for (int q = 0; q < NQ; ++q) {
        const double v = dpdlp::group_reduce<dpdlp::SumOp>(acc[q], 6);
        if (lane == 0) s[q][wave] = v;
    }
    __syncthreads();
    if (threadIdx.x == 0) {
#pragma unroll
        for (int q = 0; q < NQ; ++q) {
            double v = s[q][0];
            for (int w = 1; w < kNaThreads / 64; ++w) v += s[q][w];
            part[(size_t)q * nb + block] = v;
        }
    }
}

// sum of a_p v[idx_p] over p = b + lane, b + lane + L, ... < e, in that order;
// up to four entries' loads go out before the first gather, and the gathers
// before the first product.
template <int L>
__device__ __forceinline__ double strided_dot(const double *__restrict__ val,
                                              const int32_t *__restrict__ idx,
                                              const double *__restrict__ v, int b, int e, int lane)
{
    double s = 0.0;
    for (dpdlp::Walk w(b, e, lane); w.has(); w.step(4 * L)) {
        const int32_t *wi = idx + w.p;
        const double *wa = val + w.p;
        double a[4] = {0.0, 0.0, 0.0, 0.0}, x[4] = {0.0, 0.0, 0.0, 0.0};
        int k[4] = {0, 0, 0, 0};
#pragma unroll
        for (int u = 0; u < 4; ++u)
            if (w.has(u * L)) { k[u] = wi[u * L]; a[u] = wa[u * L]; }
#pragma unroll
        for (int u = 0; u < 4; ++u)
            if (w.has(u * L)) x[u] = v[k[u]];
#pragma unroll
        for (int u = 0; u < 4; ++u)
            if (w.has(u * L)) s += a[u] * x[u];
    }
    return s;
}

// The product of one row or column per kNaLanes lanes, valid in the first of
// them.  Segments of more than kNaLong entries are taken by the whole wave,
// one after another: at 8 lanes a segment of 5000 would be 157 trips of two
// memory latencies, at 64 lanes it is 20 (a skewed LP of 300k columns took
// 328 us, now 77; of 30k columns 85, now 14).  4 or 16 lanes per segment
// instead of 8 measured within 10% on both kinds, 16 never faster.
__device__ __forceinline__ double segment_dot(const double *__restrict__ val,
                                              const int32_t *__restrict__ idx,
                                              const double *__restrict__ v, int b, int e)
{
    const int lane = threadIdx.x & 63, l = lane & (kNaLanes - 1);
    const bool wide = e - b > kNaLong;
    double s = dpdlp::group_reduce<dpdlp::SumOp>(
        wide ? 0.0 : strided_dot<kNaLanes>(val, idx, v, b, e, l), kNaLanesLog2);
    for (unsigned long long todo = __ballot(wide && l == 0); todo; todo &= todo - 1) {
        const int src = __ffsll((long long)todo) - 1;
        const int wb = __shfl(b, src, 64), we = __shfl(e, src, 64);
        const double t = dpdlp::group_reduce<dpdlp::SumOp>(strided_dot<64>(val, idx, v, wb, we, lane), 6);
        if (lane == src) s = t;
    }
    return s;
}

struct NaArgs {
    int m, n, nbr, nbc;
    const int32_t *rp, *ci, *cp, *ri;
    const double *val, *vt, *x, *y, *c, *clo, *chi, *vlo, *vhi, *dc, *q;
    double tau;
    double *rpart, *cpart;
};

// Row pass (workgroups 0 .. nbr - 1): per row i, (A x)_i by 8 lanes in fixed
// strided order, then
//   0 sum ((A x)_i - proj_[lo_i, hi_i]((A x)_i))^2
//   1 sum (lo_i y_i^+ - hi_i y_i^-)          (= -p(-y; lo, hi))
//   2 sum of the squared finite bounds        (||[lo, hi]||^2)
__device__ void na_rows(const NaArgs &a, int block)
{
    double acc[kNaRowQ] = {0.0, 0.0, 0.0};
    const int lane = threadIdx.x & (kNaLanes - 1);
    for (int i0 = block * kNaSegs; i0 < a.m; i0 += a.nbr * kNaSegs) {
        const int i = i0 + threadIdx.x / kNaLanes;
        const bool in = i < a.m;
        double l = 0.0, h = 0.0, yi = 0.0;
        if (in && lane == 0) { l = a.clo[i]; h = a.chi[i]; yi = a.y[i]; }
        const double s = segment_dot(a.val, a.ci, a.x, in ? a.rp[i] : 0, in ? a.rp[i + 1] : 0);
        if (in && lane == 0) {
            const double res = s - clampd(s, l, h);
            acc[0] += res * res;
            if (yi > 0.0) acc[1] += l * yi;
            else if (yi < 0.0) acc[1] += h * yi;
            if (std::isfinite(l)) acc[2] += l * l;
            if (std::isfinite(h)) acc[2] += h * h;
        }
    }
    block_partials<kNaRowQ>(acc, a.rpart, a.nbr, block);
}

// Column pass (the other workgroups): per column j, g = c_j + q_j x_j - (A^T y)_j,
// the projected step u = x_j - tau_j g with tau_j = tau * dc_j^2 and
// s = (clamp(u) - u) / tau_j:
//   0 sum (g - s)^2   1 sum c_j x_j + q_j x_j^2 / 2   2 sum s_j x_j - q_j x_j^2 / 2
//   3 sum c_j^2
__device__ void na_cols(const NaArgs &a, int block)
{
    double acc[kNaColQ] = {0.0, 0.0, 0.0, 0.0};
    const int lane = threadIdx.x & (kNaLanes - 1);
    for (int j0 = block * kNaSegs; j0 < a.n; j0 += a.nbc * kNaSegs) {
        const int j = j0 + threadIdx.x / kNaLanes;
        const bool in = j < a.n;
        double xj = 0.0, cj = 0.0, qj = 0.0, tj = a.tau, lo = 0.0, hi = 0.0;
        if (in && lane == 0) {
            xj = a.x[j]; cj = a.c[j]; lo = a.vlo[j]; hi = a.vhi[j];
            if (a.q) qj = a.q[j];
            if (a.dc) tj = a.tau * a.dc[j] * a.dc[j];
        }
        const double s = segment_dot(a.vt, a.ri, a.y, in ? a.cp[j] : 0, in ? a.cp[j + 1] : 0);
        if (in && lane == 0) {
            const double qx = a.q ? qj * xj : 0.0;
            const double g = cj + qx - s;
            const double u = xj - tj * g;
            const double sj = (clampd(u, lo, hi) - u) / tj;
            const double d = g - sj;
            acc[0] += d * d;
            const double half_xqx = 0.5 * qx * xj;
            acc[1] += cj * xj + half_xqx;
            acc[2] += sj * xj - half_xqx;
            acc[3] += cj * cj;
        }
    }
    block_partials<kNaColQ>(acc, a.cpart, a.nbc, block);
}

// Both passes in one launch: they do not depend on each other.
__global__ __launch_bounds__(kNaThreads) void k_na_passes(NaArgs a)
{
    if ((int)blockIdx.x < a.nbr) na_rows(a, blockIdx.x);
    else na_cols(a, blockIdx.x - a.nbr);
}

// One workgroup: the partials of each quantity summed in a fixed order, then
// r_primal, r_dual, r_gap, primal and dual objective into out5 (App. B.4).
__global__ __launch_bounds__(kNaFinish) void k_na_finish(const double *rpart, int nbr,
                                                        const double *cpart, int nbc,
                                                        double *out5)
{
    constexpr int Q = kNaRowQ + kNaColQ;
    __shared__ double s[Q][kNaFinish / 64];
    double a[Q];
    for (int q = 0; q < Q; ++q) a[q] = 0.0;
    for (int i = threadIdx.x; i < nbr; i += kNaFinish)
        for (int q = 0; q < kNaRowQ; ++q) a[q] += rpart[(size_t)q * nbr + i];
    for (int i = threadIdx.x; i < nbc; i += kNaFinish)
        for (int q = 0; q < kNaColQ; ++q) a[kNaRowQ + q] += cpart[(size_t)q * nbc + i];
#pragma unroll
    for (int q = 0; q < Q; ++q) {
        const double v = dpdlp::group_reduce<dpdlp::SumOp>(a[q], 6);
        if ((threadIdx.x & 63) == 0) s[q][threadIdx.x >> 6] = v;
    }
    __syncthreads();
    if (threadIdx.x != 0) return;
    double t[Q];
    for (int q = 0; q < Q; ++q) {
        t[q] = s[q][0];
        for (int w = 1; w < kNaFinish / 64; ++w) t[q] += s[q][w];
    }
    const double pres = t[0], py = t[1], bn2 = t[2];
    const double dres = t[3], cx = t[4], sx = t[5], cn2 = t[6];
    const double dobj = py + sx;
    out5[0] = sqrt(pres) / (1.0 + sqrt(bn2));
    out5[1] = sqrt(dres) / (1.0 + sqrt(cn2));
    out5[2] = fabs(cx - dobj) / (1.0 + fmax(fabs(cx), fabs(dobj)));
    out5[3] = cx;
    out5[4] = dobj;
}

}  // namespace

extern "C" int dpdlp_kkt_noalloc(const dpdlp_csr_lp *lp, const int32_t *col_ptr,
                                 const int32_t *row_idx, const double *val_csc,
                                 const double *col_scale, const double *q, const double *x,
                                 const double *y, double tau, double *out5, void *stream)
{
    if (!lp || !col_ptr || !row_idx || !val_csc || !x || !y || !out5 || !lp->row_ptr ||
        !lp->col_idx || !lp->val || !lp->c || !lp->con_lo || !lp->con_hi || !lp->var_lo ||
        !lp->var_hi) {
        dpdlp::set_error("dpdlp_kkt_noalloc: NULL argument");
        return DPDLP_E_INVALID_ARG;
    }
    if (lp->mem_kind != DPDLP_MEM_DEVICE) {
        dpdlp::set_error("dpdlp_kkt_noalloc: every array must be device memory (mem_kind = DPDLP_MEM_DEVICE)");
        return DPDLP_E_INVALID_ARG;
    }
    if (lp->m < 1 || lp->n < 1 || lp->m > kNaMaxCount || lp->n > kNaMaxCount) {
        dpdlp::set_error("dpdlp_kkt_noalloc: m and n must lie in [1, 16777216]");
        return DPDLP_E_INVALID_ARG;
    }
    if (!(tau > 0.0) || !std::isfinite(tau)) {
        dpdlp::set_error("dpdlp_kkt_noalloc: tau must be positive and finite");
        return DPDLP_E_INVALID_ARG;
    }
    double *sc = nullptr;
    const int rc = scratch_address(&sc);
    if (rc != DPDLP_OK) return rc;
    hipStream_t s = (hipStream_t)stream;
    NaArgs a{};
    a.m = lp->m; a.n = lp->n;
    a.nbr = std::min((lp->m + kNaSegs - 1) / kNaSegs, kNaMaxBlocks);
    a.nbc = std::min((lp->n + kNaSegs - 1) / kNaSegs, kNaMaxBlocks);
    a.rp = lp->row_ptr; a.ci = lp->col_idx; a.val = lp->val;
    a.cp = col_ptr; a.ri = row_idx; a.vt = val_csc;
    a.x = x; a.y = y; a.c = lp->c; a.clo = lp->con_lo; a.chi = lp->con_hi;
    a.vlo = lp->var_lo; a.vhi = lp->var_hi; a.dc = col_scale; a.q = q;
    a.tau = tau;
    a.rpart = sc; a.cpart = sc + (size_t)kNaRowQ * kNaMaxBlocks;
    hipLaunchKernelGGL(k_na_passes, dim3(a.nbr + a.nbc), dim3(kNaThreads), 0, s, a);
    hipLaunchKernelGGL(k_na_finish, dim3(1), dim3(kNaFinish), 0, s, a.rpart, a.nbr, a.cpart, a.nbc,
                       out5);
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) {
        dpdlp::set_error(std::string("dpdlp_kkt_noalloc launch: ") + hipGetErrorString(e));
        return DPDLP_E_HIP;
    }
    return DPDLP_OK;
}
