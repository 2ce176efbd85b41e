// Device kernels of the single-GPU restarted reflected-Halpern PDHG solver,
// written for gfx950 (MI355X): wave64, 256-thread workgroups, LDS-staged
// nonzero tiles, deterministic reductions (no floating-point atomics).
//
// The tile framework: a matrix in CSR (segments = rows) or CSC (segments =
// columns) is cut on the host into tiles of at most kTileNnzMax nonzeros
// (nonzero-aware partitioning, Sec. 4.3 of the D-PDLP paper, applied to
// workgroups).  One workgroup owns one tile:
//   1. it streams the tile's (index, value) pairs once with coalesced loads
//      (non-temporal where the data exceed the Infinity Cache), gathers the
//      vector entry, and stages the products in LDS;
//   2. groups of lanes reduce one segment each from LDS in the order of a
//      2^W-strided sum and a butterfly (W per tile from the mean segment
//      length; the lanes per tile from a model of its waves' time), with lane
//      permutations of the vector ALU;
//   3. one thread per segment applies the fused epilogue (projection,
//      reflection, Halpern, or a residual contribution) with coalesced
//      vector loads and stores.
// Where the gathers of a tile hit the same cache lines out of order (rows of
// a transportation LP, whose columns are strided), the host may store each
// tile's nonzeros sorted by gathered index, so that one wave's lanes load
// neighbouring entries together; pos then gives every nonzero's position in
// the tile's segment order, where its product is stored in LDS, so the
// segment sums are unchanged.
// A segment longer than a tile is split into pieces.  Few of them may stay in
// one workgroup, one after another (merge_short_splits); otherwise each
// piece's workgroup publishes its part and the pieces are added in piece order
// by the sliced step's combine, or by a small follow-up kernel.  The summation
// order is fixed by the tiling alone, so results are bitwise reproducible run
// to run.
//
// The XCD-sliced form (the paper's 2-D partition, Sec. 3.1 / App. D, across
// the 8 XCDs): the gathered dimension is cut into S slices, slice s runs on
// XCD s % 8 so its share of the gathered vector stays in that XCD's L2;
// PartialOp writes one sum per (segment, slice) pair that has nonzeros, and
// k_combine adds a segment's slice sums in slice order before the epilogue.
#pragma once
#include <hip/hip_runtime.h>

#include <cmath>
#include <cstdint>
#include <type_traits>

#include "dpdlp_internal.h"

namespace dpdlp {

template <typename T>
__device__ __forceinline__ T clampv(T v, T lo, T hi)
{
    return v < lo ? lo : (v > hi ? hi : v);
}

// Loads and stores of what a pass touches once.  NT: past the caches
// (non-temporal), for passes whose data would only push the gathered vectors
// out; otherwise plain, so that what one pass reads stays in the Infinity
// Cache for the next (the rule is at streams_fit_cache()).
template <bool NT = true, typename T>
__device__ __forceinline__ T nt_load(const T *p)
{
    if constexpr (NT) return __builtin_nontemporal_load(p);
    else return *p;
}

struct SumOp {
    template <typename T> __device__ static T id() { return T(0); }
    template <typename T> __device__ static T comb(T a, T b) { return a + b; }
};
struct MaxOp {
    template <typename T> __device__ static T id() { return T(0); }
    template <typename T> __device__ static T comb(T a, T b) { return a > b ? a : b; }
};

// Tile index of this workgroup.  Workgroups are dispatched round-robin over
// the 8 XCDs (workgroup b runs on XCD b % 8); with per_xcd > 0, XCD x processes
// that many consecutive tiles, so neighbouring segments share that XCD's L2
// (the grid is then 8 per_xcd).
__device__ __forceinline__ int tile_of_block(int per_xcd)
{
    const int b = blockIdx.x;
    return per_xcd ? (b & 7) * per_xcd + (b >> 3) : b;
}

// Lane permutations inside the vector ALU, on 32- or 64-bit values: lane i
// receives the value of another lane of its 16 (data-parallel primitives).
template <int CTRL, int BANKS>
__device__ __forceinline__ uint32_t dpp32(uint32_t old, uint32_t v)
{
    return (uint32_t)__builtin_amdgcn_update_dpp((int)old, (int)v, CTRL, 0xf, BANKS, false);
}
template <int OFF>
__device__ __forceinline__ uint32_t lane_xor32(uint32_t v)
{
    static_assert(OFF == 1 || OFF == 2 || OFF == 4 || OFF == 8, "inside a row of 16 lanes");
    if constexpr (OFF == 1) return dpp32<0xB1, 0xf>(v, v);          // quad_perm [1,0,3,2]
    if constexpr (OFF == 2) return dpp32<0x4E, 0xf>(v, v);          // quad_perm [2,3,0,1]
    if constexpr (OFF == 8) return dpp32<0x128, 0xf>(v, v);         // row_ror:8
    // lanes 0-3 and 8-11 of a row take lane i + 4, the others lane i - 4
    return dpp32<0x114, 0xa>(dpp32<0x104, 0x5>(v, v), v);           // row_shl:4, row_shr:4
}
template <int OFF, typename T>
__device__ __forceinline__ T lane_xor(T v)
{
    if constexpr (sizeof(T) == 4) {
        return __builtin_bit_cast(T, lane_xor32<OFF>(__builtin_bit_cast(uint32_t, v)));
    } else {
        const uint64_t u = __builtin_bit_cast(uint64_t, v);
        const uint64_t hi = lane_xor32<OFF>((uint32_t)(u >> 32));
        return __builtin_bit_cast(T, (hi << 32) | lane_xor32<OFF>((uint32_t)u));
    }
}
// comb(v of this lane, v of lane ^ 16 or ^ 32): the swap leaves one half's
// values in a and the other half's in b, in all lanes (comb commutes).
template <class R, int OFF, typename T>
__device__ __forceinline__ T swap_comb(T v)
{
    auto swap = [](uint32_t u) {
        if constexpr (OFF == 16) return __builtin_amdgcn_permlane16_swap(u, u, false, false);
        else return __builtin_amdgcn_permlane32_swap(u, u, false, false);
    };
    if constexpr (sizeof(T) == 4) {
        const auto p = swap(__builtin_bit_cast(uint32_t, v));
        return R::comb(__builtin_bit_cast(T, (uint32_t)p[0]), __builtin_bit_cast(T, (uint32_t)p[1]));
    } else {
        const uint64_t u = __builtin_bit_cast(uint64_t, v);
        const auto l = swap((uint32_t)u);
        const auto h = swap((uint32_t)(u >> 32));
        return R::comb(__builtin_bit_cast(T, ((uint64_t)h[0] << 32) | l[0]),
                       __builtin_bit_cast(T, ((uint64_t)h[1] << 32) | l[1]));
    }
}

// Butterfly over groups of 2^wl lanes (wl <= 6 and the same in the whole
// wave), widest step first: every lane ends with the same sum.  The steps
// stay in the vector ALU; through LDS permutes (two per 64-bit shuffle, each
// waited for) they were the longest chain of a tile of short segments.
template <class R, typename T>
__device__ __forceinline__ T group_reduce(T v, int wl)
{
    if (wl >= 6) v = swap_comb<R, 32>(v);
    if (wl >= 5) v = swap_comb<R, 16>(v);
    if (wl >= 4) v = R::comb(v, lane_xor<8>(v));
    if (wl >= 3) v = R::comb(v, lane_xor<4>(v));
    if (wl >= 2) v = R::comb(v, lane_xor<2>(v));
    if (wl >= 1) v = R::comb(v, lane_xor<1>(v));
    return v;
}

// Fixed-order workgroup reduction of NQ values; result valid in thread 0.
template <class R, int NQ, typename T>
__device__ __forceinline__ void block_reduce(T (&v)[NQ], T (*s_red)[kBlock / 64])
{
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
#pragma unroll
    for (int q = 0; q < NQ; ++q) {
        T x = group_reduce<R>(v[q], 6);
        if (lane == 0) s_red[q][wave] = x;
    }
    __syncthreads();
    if (threadIdx.x == 0) {
#pragma unroll
        for (int q = 0; q < NQ; ++q) {
            T x = s_red[q][0];
            for (int w = 1; w < kBlock / 64; ++w) x = R::comb(x, s_red[q][w]);
            v[q] = x;
        }
    }
}

template <bool NT = true, typename T>
__device__ __forceinline__ void nt_store(T *p, T v)
{
    if constexpr (NT) __builtin_nontemporal_store(v, p);
    else *p = v;
}

// Generic tile kernel.  Op supplies:
//   MT  matrix value type, AT accumulation type, NR right-hand sides,
//   NQ  per-tile partial quantities (0 = none), R the reduction (Sum/Max),
//   Pre per-segment values loaded before the reduction (prefetch)
//   value(a, j, out[NR])          product for a nonzero a with index j
//   prefetch(seg, pre)            issue the epilogue's vector loads early
//   epilogue(seg, r[NR], pre, acc) per-segment update, adds to acc[NQ]
//   partials                      double* [NQ * ntiles] or null
// Memory-level parallelism: every thread first issues all of its index /
// value loads, the segment-pointer loads and the epilogue prefetches, then
// all of its gathers, so one tile costs about two memory round trips before
// the LDS phases.  PER is the tile size over the 256 threads (tile_loads()):
// a small tile issues no repeated loads and takes little LDS.  With PER = 8
// for every tile size, shuffles through LDS in the segment sums and an LDS
// buffer of their results, an iteration of a 10k-nonzero LP took 10.3 us
// (8.2 without), of a 1M-nonzero LP 34.8 us (28.6; update and output
// included); with the steps since then 6.9 and 23.5.
constexpr int kPre = 2;                         // prefetched segments per thread

template <class Op, int PER, bool NT>
__global__ __launch_bounds__(kBlock) void k_tile(const Tile *__restrict__ tiles,
                                                 const int *__restrict__ blk2tile, int ntiles,
                                                 int per_xcd, const int *__restrict__ idx,
                                                 const typename Op::MT *__restrict__ val,
                                                 const int *__restrict__ seg_ptr, int seg_stride,
                                                 const uint16_t *__restrict__ pos,
                                                 typename Op::AT *__restrict__ carries, Op op0)
{
    using AT = typename Op::AT;
    using MT = typename Op::MT;
    using R = typename Op::R;
    constexpr int NR = Op::NR;
    constexpr int NQ = Op::NQ > 0 ? Op::NQ : 1;
    __shared__ AT s_prod[NR][PER * kBlock];
    __shared__ int s_ptr[kMaxSegs + 1];
    __shared__ double s_red[NQ][kBlock / 64];
    __shared__ AT s_redp[NR][kBlock / 64];

    const int t = blk2tile ? blk2tile[blockIdx.x] : tile_of_block(per_xcd);
    if (t < 0 || t >= ntiles) return;
    const Tile d = tiles[t];
    Op op = op0;
    op.slice = d.slice;
    seg_ptr += (size_t)d.slice * seg_stride;
    const int nnz0 = d.nnz_begin;
    // (a merged tile of -npieces pieces of d.piece nonzeros starts with its first)
    const int cnt = d.npieces < 0 ? d.piece : d.nnz_end - d.nnz_begin;
    const int nseg = d.seg_end - d.seg_begin;
    const bool whole = d.npieces == 0;

    // Every load of phase 1 is unconditional, from an index clamped into the
    // tile (lanes past its end repeat its last element and store nothing),
    // so that each group of loads issues back to back and is waited for
    // once; per-element branches would put a wait after every load.
    // 1a. issue the tile's matrix stream (coalesced, non-temporal)
    int jj[PER];
    MT aa[PER];
    int pp[PER];              // where each product goes in LDS (gather-sorted tiles)
    if (cnt > 0) {
#pragma unroll
        for (int q = 0; q < PER; ++q) {
            const int e = min((int)threadIdx.x + q * kBlock, cnt - 1);
            jj[q] = nt_load<NT>(idx + nnz0 + e);
            aa[q] = nt_load<NT>(val + nnz0 + e);
        }
        if (pos) {
#pragma unroll
            for (int q = 0; q < PER; ++q)
                pp[q] = nt_load<NT>(pos + nnz0 + min((int)threadIdx.x + q * kBlock, cnt - 1));
        } else {
#pragma unroll
            for (int q = 0; q < PER; ++q) pp[q] = threadIdx.x + q * kBlock;
        }
    }
    // 1b. segment pointers to LDS and the epilogue's vector loads; the second
    // set only where the tile has more than kBlock segments (a uniform branch)
    typename Op::Pre pre[kPre];
    if (whole) {
        const int sp0 = seg_ptr[d.seg_begin + min((int)threadIdx.x, nseg)];
        op.template prefetch<NT>(d.seg_begin + min((int)threadIdx.x, nseg - 1), pre[0]);
        if (nseg >= kBlock) {
            constexpr int kPtrIt = (kMaxSegs + kBlock) / kBlock;   // covers nseg + 1 <= kMaxSegs + 1
            int sp[kPtrIt];
#pragma unroll
            for (int i = 1; i < kPtrIt; ++i)
                sp[i] = seg_ptr[d.seg_begin + min((int)threadIdx.x + i * kBlock, nseg)];
            op.template prefetch<NT>(d.seg_begin + min((int)threadIdx.x + kBlock, nseg - 1), pre[1]);
#pragma unroll
            for (int i = 1; i < kPtrIt; ++i) {
                const int s = threadIdx.x + i * kBlock;
                if (s <= nseg) s_ptr[s] = sp[i] - nnz0;
            }
        }
        if ((int)threadIdx.x <= nseg) s_ptr[threadIdx.x] = sp0 - nnz0;
    }
    // graph replays: the run's scalars, whose load and divisions overlap the
    // loads above (in front of the tile's descriptor they held every kernel
    // up by a memory round trip)
    op.resolve();
    // 1c. gathers (all issued before the first product is stored), products to LDS
    if (cnt > 0) {
        AT pv[PER][NR];
#pragma unroll
        for (int q = 0; q < PER; ++q) op.value(aa[q], jj[q], pv[q]);
#pragma unroll
        for (int q = 0; q < PER; ++q) {
            const int e = threadIdx.x + q * kBlock;
            if (e < cnt) {
#pragma unroll
                for (int r = 0; r < NR; ++r) s_prod[r][pp[q]] = pv[q][r];
            }
        }
    }
    __syncthreads();

    double acc[NQ];
#pragma unroll
    for (int q = 0; q < NQ; ++q) acc[q] = 0.0;

    if (whole) {
        // 2. segment sums; a segment's result replaces its first product (only
        // its own lanes read that range).  The order of a sum is that of 2^W
        // strided partial sums and a butterfly over them; 2^(W - h) lanes take
        // a segment, 2^h partial sums each, and the butterfly's first h steps
        // are additions inside a lane: the same sums, with fewer passes over
        // the tile's segments (choose_sum_lanes picks h, and in FP64 another W
        // where a long segment would keep the others waiting).
        const int wide = sizeof(AT) == 8 ? (d.width_log2 >> 12) & 15 : 0;
        const int W = wide ? wide - 1 : d.width_log2 & 15;
        auto sums = [&](auto h_) {
            constexpr int H = decltype(h_)::value, A = 1 << H;
            const int wl = W - H;
            const int lane = threadIdx.x & ((1 << wl) - 1);
            for (int s = threadIdx.x >> wl; s < nseg; s += kBlock >> wl) {
                const int b = s_ptr[s], e = s_ptr[s + 1];
                AT r[A][NR];
#pragma unroll
                for (int u = 0; u < A; ++u)
#pragma unroll
                    for (int q = 0; q < NR; ++q) r[u][q] = R::template id<AT>();
                int p = b + lane;
                if constexpr (H == 0) {
                    const int G = 1 << wl;
                    for (; p + 3 * G < e; p += 4 * G) {       // 4 reads in flight, added in order
                        AT w[4][NR];
#pragma unroll
                        for (int u = 0; u < 4; ++u)
#pragma unroll
                            for (int q = 0; q < NR; ++q) w[u][q] = s_prod[q][p + u * G];
#pragma unroll
                        for (int u = 0; u < 4; ++u)
#pragma unroll
                            for (int q = 0; q < NR; ++q) r[0][q] = R::comb(r[0][q], w[u][q]);
                    }
                }
                for (; p < e; p += 1 << W) {
                    AT w[A][NR];
#pragma unroll
                    for (int u = 0; u < A; ++u)
#pragma unroll
                        for (int q = 0; q < NR; ++q) w[u][q] = s_prod[q][min(p + (u << wl), e - 1)];
#pragma unroll
                    for (int u = 0; u < A; ++u)
#pragma unroll
                        for (int q = 0; q < NR; ++q)
                            r[u][q] = p + (u << wl) < e ? R::comb(r[u][q], w[u][q]) : r[u][q];
                }
#pragma unroll
                for (int o = A / 2; o > 0; o >>= 1)
#pragma unroll
                    for (int u = 0; u < o; ++u)
#pragma unroll
                        for (int q = 0; q < NR; ++q) r[u][q] = R::comb(r[u][q], r[u + o][q]);
#pragma unroll
                for (int q = 0; q < NR; ++q) r[0][q] = group_reduce<R>(r[0][q], wl);
                if (lane == 0 && e > b) {
#pragma unroll
                    for (int q = 0; q < NR; ++q) s_prod[q][b] = r[0][q];
                }
            }
        };
        switch (wide ? 0 : (d.width_log2 >> 8) & 15) {
        case 0: sums(std::integral_constant<int, 0>{}); break;
        case 1: sums(std::integral_constant<int, 1>{}); break;
        default: sums(std::integral_constant<int, 2>{}); break;
        }
        __syncthreads();
        // 3. fused epilogue, one thread per segment (coalesced vector I/O)
        auto finish = [&](int s, const typename Op::Pre &p1) {
            const int b = s_ptr[s], e = s_ptr[s + 1];
            AT r[NR];
#pragma unroll
            for (int z = 0; z < NR; ++z) r[z] = e > b ? s_prod[z][b] : R::template id<AT>();
            op.template epilogue<NT>(d.seg_begin + s, r, p1, acc);
        };
        if ((int)threadIdx.x < nseg) finish(threadIdx.x, pre[0]);
        if ((int)threadIdx.x + kBlock < nseg) finish(threadIdx.x + kBlock, pre[1]);
        for (int s = threadIdx.x + kPre * kBlock; s < nseg; s += kBlock) {
            typename Op::Pre p1;
            op.template prefetch<NT>(d.seg_begin + s, p1);
            finish(s, p1);
        }
        if (Op::NQ > 0) {
            block_reduce<SumOp, NQ>(acc, s_red);
            if (threadIdx.x == 0)
                for (int q = 0; q < Op::NQ; ++q) op.partials[(size_t)q * ntiles + t] = acc[q];
        }
        return;
    }

    // Split segment: reduce this piece and publish it; the pieces are added in
    // piece order after this launch (k_split_fix, or the sliced steps'
    // k_combine: no in-kernel cross-workgroup communication, so no L2-wide
    // fences).
    AT pr[NR];
#pragma unroll
    for (int q = 0; q < NR; ++q) pr[q] = R::template id<AT>();
    for (int e = threadIdx.x; e < cnt; e += kBlock) {
#pragma unroll
        for (int q = 0; q < NR; ++q) pr[q] = R::comb(pr[q], s_prod[q][e]);
    }
    block_reduce<R, NR>(pr, s_redp);
    if (d.npieces > 0) {
        if (threadIdx.x == 0) {
#pragma unroll
            for (int q = 0; q < NR; ++q) carries[(size_t)q * ntiles + t] = pr[q];
        }
        return;
    }
    // A segment of few pieces stays in this workgroup, which takes them one
    // after another (the sums are those of the separate pieces).
    AT tot[NR];
#pragma unroll
    for (int q = 0; q < NR; ++q) tot[q] = R::comb(R::template id<AT>(), pr[q]);
    for (Walk w(nnz0, d.nnz_end, cnt); w.has(); w.step(d.piece)) {
        const uint32_t pb = w.p;
        const int pc = min(d.piece, w.left());
#pragma unroll
        for (int q = 0; q < PER; ++q) {
            const int e = min((int)threadIdx.x + q * kBlock, pc - 1);
            jj[q] = nt_load<NT>(idx + pb + e);
            aa[q] = nt_load<NT>(val + pb + e);
        }
        AT pv[PER][NR];
#pragma unroll
        for (int q = 0; q < PER; ++q) op.value(aa[q], jj[q], pv[q]);
#pragma unroll
        for (int z = 0; z < NR; ++z) {
            pr[z] = R::template id<AT>();
#pragma unroll
            for (int q = 0; q < PER; ++q)
                if ((int)threadIdx.x + q * kBlock < pc) pr[z] = R::comb(pr[z], pv[q][z]);
        }
        __syncthreads();              // s_redp is still being read
        block_reduce<R, NR>(pr, s_redp);
#pragma unroll
        for (int z = 0; z < NR; ++z) tot[z] = R::comb(tot[z], pr[z]);
    }
    if (threadIdx.x == 0) {
        typename Op::Pre p1;
        op.template prefetch<NT>(d.seg_begin, p1);
        op.template epilogue<NT>(d.seg_begin, tot, p1, acc);
        if (Op::NQ > 0)
            for (int q = 0; q < Op::NQ; ++q) op.partials[(size_t)q * ntiles + t] = acc[q];
    }
}

// A segment split over npieces consecutive tiles starting at tile t0.
struct SplitSeg {
    int32_t seg, t0, npieces, slice;
};
// The sum of its pieces in piece order, eight loads at a time.
template <class R, typename AT>
__device__ __forceinline__ AT split_sum(const AT *carries, int npieces)
{
    AT r = R::template id<AT>();
    int pc = 0;
    for (; pc + 8 <= npieces; pc += 8) {
        AT v[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) v[u] = carries[pc + u];
#pragma unroll
        for (int u = 0; u < 8; ++u) r = R::comb(r, v[u]);
    }
    for (; pc < npieces; ++pc) r = R::comb(r, carries[pc]);
    return r;
}

// Finish split segments: one thread per split segment sums its pieces'
// carries in piece order and runs the epilogue; the segment's partial-sum
// contribution goes to the slot of its first piece (the other pieces' slots
// get zero), so every slot is written exactly once per pass.
template <class Op>
__global__ __launch_bounds__(64) void k_split_fix(Op op0, const SplitSeg *__restrict__ splits,
                                                   int nsplit, int ntiles,
                                                   const typename Op::AT *__restrict__ carries)
{
    using AT = typename Op::AT;
    using R = typename Op::R;
    constexpr int NR = Op::NR;
    constexpr int NQ = Op::NQ > 0 ? Op::NQ : 1;
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= nsplit) return;
    const SplitSeg sg = splits[i];
    Op op = op0;
    op.slice = sg.slice;
    op.resolve();
    AT r[NR];
#pragma unroll
    for (int q = 0; q < NR; ++q)
        r[q] = split_sum<R>(carries + (size_t)q * ntiles + sg.t0, sg.npieces);
    double acc[NQ];
#pragma unroll
    for (int q = 0; q < NQ; ++q) acc[q] = 0.0;
    typename Op::Pre p1;
    op.template prefetch<true>(sg.seg, p1);
    op.template epilogue<true>(sg.seg, r, p1, acc);
    if (Op::NQ > 0)
        for (int pc = 0; pc < sg.npieces; ++pc)
            for (int q = 0; q < Op::NQ; ++q)
                op.partials[(size_t)q * ntiles + sg.t0 + pc] = pc == 0 ? acc[q] : 0.0;
}

struct NoPre {};

// Iteration scalars read from device memory by graph-replayed launches:
// the primal / dual step size and the Halpern index of the run's first
// iteration (the launch adds its offset j inside the run).
struct IterDev {
    double tau, sigma;
    long long k0;
};

// ---------------------------------------------------------------------------
// Fused PDHG steps (Sec. 2.2 / Algorithm 1 steps 1-2, with the reflected
// Halpern update of App. A fused in).  T is double (FP64) or float (FP32).

// Primal step over CSC tiles, one segment per column j:
//   g = c~_j - (A~^T y)_j ; xh = clamp(x_j - tau g, l_j, u_j) ; xbar = 2 xh - x_j
//   x_j <- a ((1+gamma) xh - gamma x_j) + b xa_j,  a = (k+1)/(k+2), b = 1/(k+2)
template <typename T>
struct PrimalOp {
    using MT = T; using AT = T; using R = SumOp;
    static constexpr int NR = 1, NQ = 0;
    int slice = 0;
    __device__ void resolve()
    {
        if (!dev) return;
        const double kk = (double)(dev->k0 + j);
        tau = (T)dev->tau;
        a = (T)((kk + 1.0) / (kk + 2.0));
        b = (T)(1.0 / (kk + 2.0));
    }
    const T *__restrict__ y;
    const T *__restrict__ c;
    const T *__restrict__ lo;
    const T *__restrict__ hi;
    const T *__restrict__ xa;
    T *__restrict__ x;
    T *__restrict__ xbar;
    double *__restrict__ xh;      // written when write_hat
    double *__restrict__ dx;      // x_j - xh_j, written when write_hat
    double *partials;
    T tau, a, b, gamma;
    int write_hat;
    const IterDev *dev = nullptr;   // graph replays: tau and k from here
    int j = 0;
    struct Pre { T x, c, lo, hi, xa; };
    __device__ void value(MT v, int j, AT *out) const { out[0] = v * y[j]; }
    template <bool NT> __device__ void prefetch(int j, Pre &p) const
    {
        p.x = nt_load<NT>(x + j); p.c = nt_load<NT>(c + j); p.lo = nt_load<NT>(lo + j);
        p.hi = nt_load<NT>(hi + j); p.xa = nt_load<NT>(xa + j);
    }
    template <bool NT> __device__ void epilogue(int j, const AT *r, const Pre &p, double *) const
    {
        const T g = p.c - r[0];
        const T xk = p.x;
        const T xhv = clampv(xk - tau * g, p.lo, p.hi);
        xbar[j] = T(2) * xhv - xk;
        nt_store<NT>(x + j, a * ((T(1) + gamma) * xhv - gamma * xk) + b * p.xa);
        if (write_hat) {
            xh[j] = (double)xhv;
            dx[j] = (double)xk - (double)xhv;
        }
    }
};

// Primal step of a QP with diagonal Q (Sec. 6) over CSC tiles: the step
// minimises q x^2 / 2 + g x + (x - x_j)^2 / (2 tau) over the box, separately
// per column, so xh = clamp((x_j - tau g) / (1 + tau q_j), l_j, u_j) (a
// convex one-dimensional quadratic); the rest is the LP step.  q is the
// scaled diagonal D_c Q D_c.  A type of its own, so the LP step's kernel
// arguments and code stay as they are.
template <typename T>
struct PrimalQPOp : PrimalOp<T> {
    using Base = PrimalOp<T>;
    const T *__restrict__ q;
    struct Pre { T x, c, lo, hi, xa, q; };
    template <bool NT> __device__ void prefetch(int j, Pre &p) const
    {
        p.x = nt_load<NT>(this->x + j); p.c = nt_load<NT>(this->c + j); p.lo = nt_load<NT>(this->lo + j);
        p.hi = nt_load<NT>(this->hi + j); p.xa = nt_load<NT>(this->xa + j); p.q = nt_load<NT>(q + j);
    }
    template <bool NT> __device__ void epilogue(int j, const T *r, const Pre &p, double *) const
    {
        const T g = p.c - r[0];
        const T xk = p.x;
        const T tau = this->tau;
        const T xhv = clampv((xk - tau * g) / (T(1) + tau * p.q), p.lo, p.hi);
        this->xbar[j] = T(2) * xhv - xk;
        nt_store<NT>(this->x + j, this->a * ((T(1) + this->gamma) * xhv - this->gamma * xk) + this->b * p.xa);
        if (this->write_hat) {
            this->xh[j] = (double)xhv;
            this->dx[j] = (double)xk - (double)xhv;
        }
    }
};

// Dual step over CSR tiles, one segment per row i:
//   q = (A~ xbar)_i ; w = y_i / sigma - q ; yh = sigma (w - clamp(w, -u_i, -l_i))
//   y_i <- a ((1+gamma) yh - gamma y_i) + b ya_i
template <typename T>
struct DualOp {
    using MT = T; using AT = T; using R = SumOp;
    static constexpr int NR = 1, NQ = 0;
    int slice = 0;
    __device__ void resolve()
    {
        if (!dev) return;
        const double kk = (double)(dev->k0 + j);
        sigma = (T)dev->sigma;
        a = (T)((kk + 1.0) / (kk + 2.0));
        b = (T)(1.0 / (kk + 2.0));
    }
    const T *__restrict__ xbar;
    const T *__restrict__ lo;
    const T *__restrict__ hi;
    const T *__restrict__ ya;
    T *__restrict__ y;
    double *__restrict__ yh;
    double *__restrict__ dy;
    double *partials;
    T sigma, a, b, gamma;
    int write_hat;
    const IterDev *dev = nullptr;
    int j = 0;
    struct Pre { T y, lo, hi, ya; };
    __device__ void value(MT v, int j, AT *out) const { out[0] = v * xbar[j]; }
    template <bool NT> __device__ void prefetch(int i, Pre &p) const
    {
        p.y = y[i]; p.lo = nt_load<NT>(lo + i); p.hi = nt_load<NT>(hi + i); p.ya = nt_load<NT>(ya + i);
    }
    template <bool NT> __device__ void epilogue(int i, const AT *r, const Pre &p, double *) const
    {
        const T yk = p.y;
        const T w = yk / sigma - r[0];
        const T yhv = sigma * (w - clampv(w, -p.hi, -p.lo));
        y[i] = a * ((T(1) + gamma) * yhv - gamma * yk) + b * p.ya;
        if (write_hat) {
            yh[i] = (double)yhv;
            dy[i] = (double)yk - (double)yhv;
        }
    }
};

// Per-slice segment sums for the XCD-sliced form of the fused steps:
//   partial[slice * nseg + seg] = sum over the slice's nonzeros of a * v[idx]
template <typename T>
struct PartialOp {
    using MT = T; using AT = T; using R = SumOp;
    static constexpr int NR = 1, NQ = 0;
    int slice = 0;
    __device__ void resolve() {}
    const T *__restrict__ v;
    T *__restrict__ partial;        // one value per compact segment
    double *partials;
    using Pre = NoPre;
    __device__ void value(MT a, int j, AT *o) const { o[0] = a * v[j]; }
    template <bool NT> __device__ void prefetch(int, Pre &) const {}
    template <bool NT> __device__ void epilogue(int g, const AT *r, const Pre &, double *) const
    {
        partial[g] = r[0];
    }
};

// Per-slice segment sums of two right-hand sides (the sliced CSR check
// pass: A~ xh and A~ dx); the second one is stored G entries after the first.
struct PartialOp2 {
    using MT = double; using AT = double; using R = SumOp;
    static constexpr int NR = 2, NQ = 0;
    int slice = 0;
    __device__ void resolve() {}
    const double *__restrict__ v;
    const double *__restrict__ v2;
    double *__restrict__ partial;
    int64_t G;
    double *partials;
    using Pre = NoPre;
    __device__ void value(MT a, int j, AT *o) const
    {
        o[0] = a * v[j];
        o[1] = a * v2[j];
    }
    template <bool NT> __device__ void prefetch(int, Pre &) const {}
    template <bool NT> __device__ void epilogue(int g, const AT *r, const Pre &, double *) const
    {
        partial[g] = r[0];
        partial[G + g] = r[1];
    }
};

// Adds the slice partials of each segment in slice order and runs a fused
// epilogue (PrimalOp / DualOp, or a check pass) on the sums; one thread per
// segment.  The partials are compact (only the slices where the segment has
// nonzeros): the position of segment j's partial in slice s is
// cbase[block * S + s] plus the number of segments of this block before j
// that have slice s, counted with wave ballots over the mask bits.  With
// Op::NR = 2 the second right-hand side's partials start G entries later.
// Ops with NQ > 0 (check passes) leave per-block partial sums in
// op.partials[q * gridDim.x + block].  A block first completes the partials
// of its own split segments from their pieces (splits[first[block] ..
// first[block + 1]), few and in few blocks): as a launch of its own between
// the tiles and the combine that took 5 us per step.
template <class Op, bool NT>
__global__ __launch_bounds__(kBlock) void k_combine(const uint8_t *__restrict__ mask,
                                                    const int *__restrict__ cbase,
                                                    typename Op::AT *partial, int nseg, int S,
                                                    int64_t G, const SplitSeg *__restrict__ splits,
                                                    const int *__restrict__ first, int ntiles,
                                                    const typename Op::AT *__restrict__ carries,
                                                    Op op0)
{
    using AT = typename Op::AT;
    constexpr int NR = Op::NR;
    constexpr int NQ = Op::NQ > 0 ? Op::NQ : 1;
    __shared__ int s_cnt[8][kBlock / 64];
    __shared__ double s_red[NQ][kBlock / 64];
    const int j = blockIdx.x * kBlock + threadIdx.x;
    const bool in = j < nseg;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const unsigned long long below = lane == 0 ? 0ull : (~0ull >> (64 - lane));
    Op op = op0;
    typename Op::Pre p;
    if (in) op.template prefetch<NT>(j, p);
    if (splits) {
        // (stored before the first barrier below, read after it)
        for (int i = first[blockIdx.x] + threadIdx.x; i < first[blockIdx.x + 1]; i += kBlock) {
            const SplitSeg sg = splits[i];
#pragma unroll
            for (int z = 0; z < NR; ++z)
                partial[(size_t)z * G + sg.seg] =
                    split_sum<SumOp>(carries + (size_t)z * ntiles + sg.t0, sg.npieces);
        }
    }
    AT r[NR];
#pragma unroll
    for (int z = 0; z < NR; ++z) r[z] = SumOp::template id<AT>();
    const int *cb = cbase + (size_t)blockIdx.x * S;
    for (int pl = 0; pl < S / 8; ++pl) {
        const unsigned mb = in ? (unsigned)mask[(size_t)pl * nseg + j] : 0u;
        unsigned long long bal[8];
#pragma unroll
        for (int b = 0; b < 8; ++b) {
            bal[b] = __ballot((mb >> b) & 1u);
            if (lane == 0) s_cnt[b][wave] = __popcll(bal[b]);
        }
        __syncthreads();
        // positions of all 8 slices first, then all loads (absent slices
        // load partial[0], always allocated, and add nothing), then the sums
        // in slice order
        int off[8];
#pragma unroll
        for (int b = 0; b < 8; ++b) {
            int o = cb[pl * 8 + b] + __popcll(bal[b] & below);
            for (int w = 0; w < wave; ++w) o += s_cnt[b][w];
            off[b] = ((mb >> b) & 1u) ? o : 0;
        }
        AT pv[8][NR];
#pragma unroll
        for (int b = 0; b < 8; ++b)
#pragma unroll
            for (int z = 0; z < NR; ++z) pv[b][z] = partial[(size_t)z * G + off[b]];
#pragma unroll
        for (int b = 0; b < 8; ++b)
            if ((mb >> b) & 1u)
#pragma unroll
                for (int z = 0; z < NR; ++z) r[z] += pv[b][z];
        __syncthreads();
    }
    double acc[NQ];
#pragma unroll
    for (int q = 0; q < NQ; ++q) acc[q] = 0.0;
    op.resolve();
    if (in) op.template epilogue<NT>(j, r, p, acc);
    if (Op::NQ > 0) {
        block_reduce<SumOp, NQ>(acc, s_red);
        if (threadIdx.x == 0)
            for (int q = 0; q < Op::NQ; ++q) op.partials[(size_t)q * gridDim.x + blockIdx.x] = acc[q];
    }
}

// ---------------------------------------------------------------------------
// Check passes (App. B.4 KKT; App. B.2 / D.2.1 fixed-point residual; App. B.3
// distances to the anchor), FP64 on the FP64 matrix.  TA: anchor type.

// CSR pass with two right-hand sides (xh, dx).  Per-tile partial sums:
//   0 sum r_i^2, r = (A x) - proj_S(A x) in the original space
//   1 sum (l_i y_i^+ - u_i y_i^-)          (= -p(-y), original space)
//   2 sum dy_i^2
//   3 sum (A~ dx)_i dy_i                    (the <A dx, dy> coupling term)
//   4 sum (yh_i - ya_i)^2
template <typename TA>
struct CheckRowOp {
    using MT = double; using AT = double; using R = SumOp;
    static constexpr int NR = 2, NQ = 5;
    int slice = 0;
    __device__ void resolve() {}
    const double *__restrict__ xh;
    const double *__restrict__ dx;
    const double *__restrict__ yh;
    const double *__restrict__ dy;
    const TA *__restrict__ ya;
    const double *__restrict__ dr;
    const double *__restrict__ lo0;
    const double *__restrict__ hi0;
    double *partials;
    __device__ void value(MT v, int j, AT *out) const
    {
        out[0] = v * xh[j];
        out[1] = v * dx[j];
    }
    using Pre = NoPre;
    template <bool NT> __device__ void prefetch(int, Pre &) const {}
    template <bool NT> __device__ void epilogue(int i, const AT *r, const Pre &, double *acc) const
    {
        const double axi = r[0] / dr[i];
        const double res = axi - clampv(axi, lo0[i], hi0[i]);
        acc[0] += res * res;
        const double yi = dr[i] * yh[i];
        if (yi > 0.0) acc[1] += lo0[i] * yi;
        else if (yi < 0.0) acc[1] += hi0[i] * yi;
        const double dyi = dy[i];
        acc[2] += dyi * dyi;
        acc[3] += r[1] * dyi;
        const double an = yh[i] - (double)ya[i];
        acc[4] += an * an;
    }
};

// CSC pass (yh).  Per-tile partial sums:
//   0 sum ((g - s)_j / dc_j)^2, g = c~ - A~^T yh, s from the primal step with tau
//   1 sum c_j x_j   (original space)
//   2 sum s_j x_j   (original space)
//   3 sum dx_j^2
//   4 sum (xh_j - xa_j)^2
template <typename TA>
struct CheckColOp {
    using MT = double; using AT = double; using R = SumOp;
    static constexpr int NR = 1, NQ = 5;
    int slice = 0;
    __device__ void resolve() {}
    const double *__restrict__ yh;
    const double *__restrict__ xh;
    const double *__restrict__ dx;
    const TA *__restrict__ xa;
    const double *__restrict__ c;     // scaled
    const double *__restrict__ c0;    // original
    const double *__restrict__ lo;    // scaled variable bounds
    const double *__restrict__ hi;
    const double *__restrict__ dc;
    const double *__restrict__ q;     // scaled diagonal of Q, or null (an LP)
    double *partials;
    double tau;
    __device__ void value(MT v, int i, AT *out) const { out[0] = v * yh[i]; }
    using Pre = NoPre;
    template <bool NT> __device__ void prefetch(int, Pre &) const {}
    template <bool NT> __device__ void epilogue(int j, const AT *r, const Pre &, double *acc) const
    {
        // a QP (Sec. 6) adds Q x to the gradient, x^T Q x / 2 to the primal
        // objective and takes it off the dual one; q~ x~ = D_c (Q x) and
        // q~ x~^2 = x^T Q x per column
        const double qx = q ? q[j] * xh[j] : 0.0;
        const double g = c[j] + qx - r[0];
        const double u = xh[j] - tau * g;
        const double s = (clampv(u, lo[j], hi[j]) - u) / tau;
        const double dres = (g - s) / dc[j];
        acc[0] += dres * dres;
        const double xj = dc[j] * xh[j];
        const double half_xqx = 0.5 * qx * xh[j];
        acc[1] += c0[j] * xj + half_xqx;
        acc[2] += (s / dc[j]) * xj - half_xqx;
        const double dxj = dx[j];
        acc[3] += dxj * dxj;
        const double an = xh[j] - (double)xa[j];
        acc[4] += an * an;
    }
};

// Plain product out[perm[s]] = sum_p a_p in[idx_p] (perm null: out[s]): the
// caller's order is restored in the same pass (a launch of its own took 4 us).
struct SpmvOp {
    using MT = double; using AT = double; using R = SumOp;
    static constexpr int NR = 1, NQ = 0;
    int slice = 0;
    __device__ void resolve() {}
    const double *__restrict__ in;
    double *__restrict__ out;
    const int *__restrict__ perm;
    double *partials;
    __device__ void value(MT v, int j, AT *o) const { o[0] = v * in[j]; }
    struct Pre { int at; };
    template <bool NT> __device__ void prefetch(int s, Pre &p) const { p.at = perm ? perm[s] : s; }
    template <bool NT> __device__ void epilogue(int, const AT *r, const Pre &p, double *) const
    {
        out[p.at] = r[0];
    }
};

// One half-step of the Golub-Kahan-Lanczos bidiagonalization, with the
// normalisations deferred to the scalars: out <- (A in) / nin - (nin / nprev)
// out (first: no second term); per-tile partials of sum out^2.
struct LanczosOp {
    using MT = double; using AT = double; using R = SumOp;
    static constexpr int NR = 1, NQ = 1;
    int slice = 0;
    __device__ void resolve() {}
    const double *__restrict__ in;
    double *__restrict__ out;
    const double *nin;              // ||in|| (device scalar)
    const double *nprev;            // norm of the previous out (device scalar)
    int first;
    double *partials;
    __device__ void value(MT v, int j, AT *o) const { o[0] = v * in[j]; }
    struct Pre { double o; };
    template <bool NT> __device__ void prefetch(int s, Pre &p) const { p.o = first ? 0.0 : out[s]; }
    template <bool NT> __device__ void epilogue(int s, const AT *r, const Pre &p, double *acc) const
    {
        const double a = *nin;
        double v = r[0] / a;
        if (!first) v -= (a / *nprev) * p.o;
        out[s] = v;
        acc[0] += v * v;
    }
};

// Rescaling reductions: Ruiz (max |a|) and Pock-Chambolle (sum |a|^p);
// epilogue writes the factor 1/sqrt(.) (1 for an empty / zero segment).
struct AbsMaxOp {
    using MT = double; using AT = double; using R = MaxOp;
    static constexpr int NR = 1, NQ = 0;
    int slice = 0;
    __device__ void resolve() {}
    double *__restrict__ f;
    double *partials;
    __device__ void value(MT v, int, AT *o) const { o[0] = fabs(v); }
    using Pre = NoPre;
    template <bool NT> __device__ void prefetch(int, Pre &) const {}
    template <bool NT> __device__ void epilogue(int s, const AT *r, const Pre &, double *) const
    {
        f[s] = r[0] > 0.0 ? 1.0 / sqrt(r[0]) : 1.0;
    }
};
struct AbsPowSumOp {
    using MT = double; using AT = double; using R = SumOp;
    static constexpr int NR = 1, NQ = 0;
    int slice = 0;
    __device__ void resolve() {}
    double *__restrict__ f;
    double *partials;
    double p;
    __device__ void value(MT v, int, AT *o) const { o[0] = p == 1.0 ? fabs(v) : pow(fabs(v), p); }
    using Pre = NoPre;
    template <bool NT> __device__ void prefetch(int, Pre &) const {}
    template <bool NT> __device__ void epilogue(int s, const AT *r, const Pre &, double *) const
    {
        f[s] = r[0] > 0.0 ? 1.0 / sqrt(r[0]) : 1.0;
    }
};

}  // namespace dpdlp
