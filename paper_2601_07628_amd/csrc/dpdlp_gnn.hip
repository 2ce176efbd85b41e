// Learned warm start: a bipartite message-passing network on the row/column
// graph of the scaled constraint matrix A~, trained on the GPU by the kernels
// in this file, predicting a start point (x0, y0) for the PDHG solver.
//
// Network (hidden width H = 128, L layers, BF16 activations and weights,
// FP32 accumulation; FP32 master weights, gradients and Adam moments):
//   H_c^0 = relu(X_c W_cin)                 X_c: n x 16 column features
//   H_r^0 = relu(X_r W_rin)                 X_r: m x 16 row features
//   layer l = 1..L:
//     S_r = A~ H_c^{l-1}                    (CSR SpMM)
//     H_r^l = relu([H_r^{l-1}, S_r] W_r^l)  (256 x 128 weights, MFMA GEMM)
//     S_c = A~^T H_r^l                      (CSC SpMM)
//     H_c^l = relu([H_c^{l-1}, S_c] W_c^l)
//   x~0 = x~ref + H_c^L w_x,  y~0 = y~ref + H_r^L w_y   (scaled space)
// (x~ref, y~ref) is a reference point supplied by the caller (the family's
// mean solution); with w_x = w_y = 0 the network returns it exactly.
// Loss: mean((x~0 - x~*)^2) + mean((y~0 - y~*)^2).
//
// Activations are stored so that each layer's GEMM input [H^{l-1}, S] is one
// contiguous m x 256 (n x 256) BF16 array: a layer writes its output straight
// into the left half of the next layer's input.  Every reduction runs in a
// fixed order (no atomics), so training is bitwise reproducible.
#include <hip/hip_runtime.h>

#include <cmath>
#include <cstring>
#include <algorithm>
#include <memory>
#include <string>
#include <type_traits>
#include <vector>

#include "dpdlp_internal.h"

namespace dpdlp {
namespace gnn {

constexpr int kH = 128;
constexpr int kF = 16;
constexpr int kKC = 2048;             // split-K chunk of the weight-gradient GEMMs
typedef uint16_t bf16;
typedef short short4v __attribute__((ext_vector_type(4)));
typedef float float4v __attribute__((ext_vector_type(4)));

__device__ __forceinline__ bf16 f2bf(float f)
{
    uint32_t u = __float_as_uint(f);
    if ((u & 0x7f800000u) == 0x7f800000u)                  // inf / nan
        return (bf16)((u >> 16) | ((u & 0xffffu) ? 0x40u : 0u));
    u += 0x7fffu + ((u >> 16) & 1u);                       // round to nearest even
    return (bf16)(u >> 16);
}
__device__ __forceinline__ float bf2f(bf16 h) { return __uint_as_float(((uint32_t)h) << 16); }

// C[M x Nc] = A[M x K] B[K x Nc] with general strides, for dpdlp_gnn_gemm_test
// only: A(i,k) = A[i*a_rs + k*a_cs], B(k,j) = B[k*b_rs + j*b_cs].  A workgroup
// (4 wave64) owns a 64 x 64 output tile, each wave a 32 x 32 sub-tile (2 x 2
// MFMA tiles); 64 x 32 slices of A and B are staged in LDS per K step.
__global__ __launch_bounds__(256) void k_gemm(const bf16 *__restrict__ A, long a_rs, long a_cs,
                                              const bf16 *__restrict__ B, long b_rs, long b_cs,
                                              float *__restrict__ C, long ldc, int M, int Nc,
                                              int K)
{
    __shared__ bf16 As[64][40];
    __shared__ bf16 Bs[64][40];
    const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
    const int bm = blockIdx.x * 64, bn = blockIdx.y * 64;
    const int wm = (w & 1) * 32, wn = (w >> 1) * 32;
    float4v acc[2][2];
    for (int a = 0; a < 2; ++a)
        for (int b = 0; b < 2; ++b) acc[a][b] = float4v{0.f, 0.f, 0.f, 0.f};
    for (int kk = 0; kk < K; kk += 32) {
        for (int e = tid; e < 64 * 32; e += 256) {
            int i, k;
            if (a_cs == 1) { i = e >> 5; k = e & 31; } else { i = e & 63; k = e >> 6; }
            const int gi = bm + i, gk = kk + k;
            As[i][k] = (gi < M && gk < K) ? A[(long)gi * a_rs + (long)gk * a_cs] : (bf16)0;
        }
        for (int e = tid; e < 64 * 32; e += 256) {
            int j, k;
            if (b_cs == 1) { j = e & 63; k = e >> 6; } else { j = e >> 5; k = e & 31; }
            const int gj = bn + j, gk = kk + k;
            Bs[j][k] = (gj < Nc && gk < K) ? B[(long)gk * b_rs + (long)gj * b_cs] : (bf16)0;
        }
        __syncthreads();
#pragma unroll
        for (int ks = 0; ks < 32; ks += 16) {
            short4v fa[2], fb[2];
#pragma unroll
            for (int t = 0; t < 2; ++t) {
                const bf16 *pa = &As[wm + t * 16 + (lane & 15)][ks + 4 * (lane >> 4)];
                fa[t] = short4v{(short)pa[0], (short)pa[1], (short)pa[2], (short)pa[3]};
                const bf16 *pb = &Bs[wn + t * 16 + (lane & 15)][ks + 4 * (lane >> 4)];
                fb[t] = short4v{(short)pb[0], (short)pb[1], (short)pb[2], (short)pb[3]};
            }
#pragma unroll
            for (int a = 0; a < 2; ++a)
#pragma unroll
                for (int b = 0; b < 2; ++b)
                    acc[a][b] = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(fa[a], fb[b], acc[a][b], 0, 0, 0);
        }
        __syncthreads();
    }
#pragma unroll
    for (int a = 0; a < 2; ++a)
#pragma unroll
        for (int b = 0; b < 2; ++b)
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                const int i = bm + wm + a * 16 + 4 * (lane >> 4) + v;
                const int j = bn + wn + b * 16 + (lane & 15);
                if (i < M && j < Nc) C[(long)i * ldc + j] = acc[a][b][v];
            }
}

// ---- the network's matrix products -----------------------------------------
// All of them use v_mfma_f32_16x16x16_bf16 in ascending steps of 16 along the
// contraction, with the operands swapped (the weights or dZ as A): a lane then
// holds 4 consecutive features of one node, one 8- or 16-byte store.
//
// A fragment is 64 lanes x 4 BF16: lane (g, i) = (lane >> 4, lane & 15) holds
// the elements k = 4 g .. 4 g + 3 of row or column i.  Weights are kept packed
// in fragments, twice: for X W (fragment [k step][column tile]) and, for the
// 256 x 128 ones, for dZ W^T (fragment [feature step][row tile]).

__device__ __forceinline__ float4v mfma(uint2 a, uint2 b, float4v c)
{
    return __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(__builtin_bit_cast(short4v, a),
                                                     __builtin_bit_cast(short4v, b), c, 0, 0, 0);
}
__device__ __forceinline__ uint2 pack4(const float *f)
{
    return make_uint2((uint32_t)f2bf(f[0]) | ((uint32_t)f2bf(f[1]) << 16),
                      (uint32_t)f2bf(f[2]) | ((uint32_t)f2bf(f[3]) << 16));
}
// relu of 4 accumulators as BF16
__device__ __forceinline__ uint2 relu4(float4v c)
{
    const float f[4] = {fmaxf(c[0], 0.f), fmaxf(c[1], 0.f), fmaxf(c[2], 0.f), fmaxf(c[3], 0.f)};
    return pack4(f);
}

// Where element (k, j) of a matrix with 16 ks rows and 128 columns goes in
// its two packed copies.
__device__ __forceinline__ long packed_fwd(int k, int j)
{
    return ((long)((k >> 4) * 8 + (j >> 4)) * 64 + ((k & 15) >> 2) * 16 + (j & 15)) * 4 + (k & 3);
}
__device__ __forceinline__ long packed_bwd(int k, int j)
{
    return ((long)((j >> 4) * 16 + (k >> 4)) * 64 + ((j & 15) >> 2) * 16 + (k & 15)) * 4 + (j & 3);
}

// Input embedding H = relu(X W), X with 16 features: one MFMA per 16 nodes and
// 16 features; column nodes first, then row nodes.
__global__ __launch_bounds__(256) void k_embed(int n, const bf16 *__restrict__ Xc,
                                               const bf16 *__restrict__ Wc, bf16 *__restrict__ Hc,
                                               int m, const bf16 *__restrict__ Xr,
                                               const bf16 *__restrict__ Wr, bf16 *__restrict__ Hr)
{
    const int nbx = (n + 63) / 64;
    const bool col = (int)blockIdx.x < nbx;
    const int N = col ? n : m;
    const uint2 *X = (const uint2 *)(col ? Xc : Xr), *W = (const uint2 *)(col ? Wc : Wr);
    bf16 *H = col ? Hc : Hr;
    const int lane = threadIdx.x & 63, g = lane >> 4;
    const int row = ((col ? blockIdx.x : blockIdx.x - nbx) * 4 + (threadIdx.x >> 6)) * 16 + (lane & 15);
    const uint2 x = X[(long)min(row, N - 1) * (kF / 4) + g];
    uint2 w[8];
#pragma unroll
    for (int t = 0; t < 8; ++t) w[t] = W[t * 64 + lane];
#pragma unroll
    for (int t = 0; t < 8; ++t) {
        const float4v c = mfma(w[t], x, float4v{0.f, 0.f, 0.f, 0.f});
        if (row < N) *(uint2 *)(H + (long)row * 2 * kH + t * 16 + 4 * g) = relu4(c);
    }
}

// Layer update out = relu(IN W), IN with 256 features.  Bound by memory: 768
// bytes per node.  Persistent workgroups hold the packed W (64 KB) in LDS; a
// wave takes 16 nodes at a time and has the next 16 nodes' loads in flight
// while it multiplies.
__global__ __launch_bounds__(256, 2) void k_dense(int N, const bf16 *__restrict__ IN,
                                                  const bf16 *__restrict__ W, bf16 *__restrict__ out,
                                                  long ld)
{
    __shared__ uint2 sW[16 * 8 * 64];
    const int lane = threadIdx.x & 63, g = lane >> 4;
    const int tiles = (N + 15) / 16, step = gridDim.x * 4;
    int tile = blockIdx.x * 4 + (threadIdx.x >> 6);
    auto load = [&](int t, uint2 (&x)[16]) {
        const uint2 *p = (const uint2 *)(IN + (long)min(t * 16 + (lane & 15), N - 1) * 2 * kH) + g;
#pragma unroll
        for (int ks = 0; ks < 16; ++ks) x[ks] = p[ks * 4];
    };
    uint2 x[16];
    load(min(tile, tiles - 1), x);
    for (int e = threadIdx.x; e < 16 * 8 * 32; e += 256) ((uint4 *)sW)[e] = ((const uint4 *)W)[e];
    __syncthreads();
    for (; tile < tiles; tile += step) {
        uint2 nx[16];
        load(min(tile + step, tiles - 1), nx);
        int w0 = lane;
        asm volatile("" : "+v"(w0));      // keeps the reads of W inside the loop
        float4v acc[8];
#pragma unroll
        for (int t = 0; t < 8; ++t) acc[t] = float4v{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int ks = 0; ks < 16; ++ks)
#pragma unroll
            for (int t = 0; t < 8; ++t) acc[t] = mfma(sW[(ks * 8 + t) * 64 + w0], x[ks], acc[t]);
        const int row = tile * 16 + (lane & 15);
        if (row < N)
#pragma unroll
            for (int t = 0; t < 8; ++t) *(uint2 *)(out + (long)row * ld + t * 16 + 4 * g) = relu4(acc[t]);
#pragma unroll
        for (int ks = 0; ks < 16; ++ks) x[ks] = nx[ks];
    }
}

// The same update for few nodes, where a launch is one round trip: a wave
// takes 16 nodes and 32 features and loads both operands straight into
// registers, all at once.
__global__ __launch_bounds__(256) void k_dense_few(int N, const bf16 *__restrict__ IN,
                                                   const bf16 *__restrict__ W,
                                                   bf16 *__restrict__ out, long ld)
{
    const int lane = threadIdx.x & 63, g = lane >> 4, t0 = (threadIdx.x >> 6) * 2;
    const int row = blockIdx.x * 16 + (lane & 15);
    const uint2 *p = (const uint2 *)(IN + (long)min(row, N - 1) * 2 * kH) + g;
    uint2 x[16], w[16][2];
#pragma unroll
    for (int ks = 0; ks < 16; ++ks) {
        x[ks] = p[ks * 4];
#pragma unroll
        for (int t = 0; t < 2; ++t) w[ks][t] = ((const uint2 *)W)[(ks * 8 + t0 + t) * 64 + lane];
    }
    float4v acc[2] = {float4v{0.f, 0.f, 0.f, 0.f}, float4v{0.f, 0.f, 0.f, 0.f}};
#pragma unroll
    for (int ks = 0; ks < 16; ++ks)
#pragma unroll
        for (int t = 0; t < 2; ++t) acc[t] = mfma(w[ks][t], x[ks], acc[t]);
    if (row < N)
#pragma unroll
        for (int t = 0; t < 2; ++t)
            *(uint2 *)(out + (long)row * ld + (t0 + t) * 16 + 4 * g) = relu4(acc[t]);
}

// dZ = dH * [H > 0] (the ReLU derivative on the stored output) as a BF16 pair
// hi + lo with hi = bf16(dZ), lo = bf16(dZ - hi): the gradient products run
// both on the matrix cores and add them in FP32 (about 16 mantissa bits).
__device__ __forceinline__ void relu_grad(float4 d, uint2 h, uint2 &hi, uint2 &lo)
{
    const float f[4] = {d.x, d.y, d.z, d.w};
    const uint32_t hb[4] = {h.x & 0xffffu, h.x >> 16, h.y & 0xffffu, h.y >> 16};
    float gr[4], res[4];
#pragma unroll
    for (int v = 0; v < 4; ++v) gr[v] = bf2f((bf16)hb[v]) > 0.f ? f[v] : 0.f;
    hi = pack4(gr);
    const uint32_t ib[4] = {hi.x & 0xffffu, hi.x >> 16, hi.y & 0xffffu, hi.y >> 16};
#pragma unroll
    for (int v = 0; v < 4; ++v) res[v] = gr[v] - bf2f((bf16)ib[v]);
    lo = pack4(res);
}

// Data gradient of a layer update: dZ from dH and the stored output, written
// out for the weight gradient, and [dH, dS] = dZ W^T (256 features, FP32; the
// left half replaces dH in place, each wave reading its nodes before it
// writes them).  Bound by memory: 2304 bytes per node.  Persistent workgroups
// with the packed W^T (64 KB) in LDS, as in k_dense.
__global__ __launch_bounds__(256, 2) void k_dgrad(int N, float *dH, const bf16 *__restrict__ H,
                                                  long hld, const bf16 *__restrict__ Wt,
                                                  bf16 *__restrict__ dZ, bf16 *__restrict__ dZlo,
                                                  float *__restrict__ dS)
{
    __shared__ uint2 sW[8 * 16 * 64];
    const int lane = threadIdx.x & 63, g = lane >> 4;
    const int tiles = (N + 15) / 16, step = gridDim.x * 4;
    for (int e = threadIdx.x; e < 8 * 16 * 32; e += 256) ((uint4 *)sW)[e] = ((const uint4 *)Wt)[e];
    __syncthreads();
    for (int tile = blockIdx.x * 4 + (threadIdx.x >> 6); tile < tiles; tile += step) {
        const int row = tile * 16 + (lane & 15);
        const long r = min(row, N - 1);
        int w0 = lane;
        asm volatile("" : "+v"(w0));      // keeps the reads of W inside the loop
        float4 d[8];
        uint2 h[8], hi[8], lo[8];
#pragma unroll
        for (int ks = 0; ks < 8; ++ks) {
            d[ks] = *(const float4 *)(dH + r * kH + ks * 16 + 4 * g);
            h[ks] = *(const uint2 *)(H + r * hld + ks * 16 + 4 * g);
        }
#pragma unroll
        for (int ks = 0; ks < 8; ++ks) {
            relu_grad(d[ks], h[ks], hi[ks], lo[ks]);
            if (row < N) {
                *(uint2 *)(dZ + r * kH + ks * 16 + 4 * g) = hi[ks];
                *(uint2 *)(dZlo + r * kH + ks * 16 + 4 * g) = lo[ks];
            }
        }
#pragma unroll
        for (int half = 0; half < 2; ++half) {
            float4v ah[8], al[8];
#pragma unroll
            for (int t = 0; t < 8; ++t) ah[t] = al[t] = float4v{0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int ks = 0; ks < 8; ++ks)
#pragma unroll
                for (int t = 0; t < 8; ++t) {
                    const uint2 w = sW[(ks * 16 + half * 8 + t) * 64 + w0];
                    ah[t] = mfma(w, hi[ks], ah[t]);
                    al[t] = mfma(w, lo[ks], al[t]);
                }
            float *o = (half == 0 ? dH : dS) + r * kH + 4 * g;
            if (row < N)
#pragma unroll
                for (int t = 0; t < 8; ++t) {
                    const float4v c = al[t] + ah[t];
                    *(float4 *)(o + t * 16) = make_float4(c[0], c[1], c[2], c[3]);
                }
        }
    }
}

// Weight gradients out = A^T dZ of both node kinds in one launch (kind 0:
// columns).
struct WgradArgs {
    const bf16 *A[2], *dZ[2], *dZlo[2];
    int M;                        // features of A
    int K[2], nz[2];              // nodes and their chunks
    float *part[2], *out[2];
};

// The partials over chunks of kKC nodes, for both halves of dZ:
// part[(2 z + half) M 128 + ...].  A workgroup owns 16 MT features of A and
// 16 NT of dZ and walks its chunk in steps of 64 nodes: 4 nodes x 4 features
// per thread and operand are transposed in registers into fragments in LDS,
// with the loads two steps ahead (a chunk's steps are serial).  The layers'
// tiles are 128 x 128 on 8 waves: at 64 x 64 on 4 waves every row was read
// and packed eight times and 150k nodes took 70-80 us, now 64 (bound by the
// MFMA of the chunks' workgroups, 148 for 256 CUs; the chunk size fixes the
// order of the sums).  Both node kinds share a launch (36 + 44 us apart); the
// tiles of one chunk run on one XCD.
template <int MT, int NT>
__global__ __launch_bounds__(64 * NT) void k_wgrad(WgradArgs a)
{
    constexpr int WM = MT == 8 ? 2 : 1, WN = NT / WM;              // the waves' grid
    constexpr int MW = MT / WM, NW = NT / WN;                      // tiles of one wave
    constexpr int FG = 4 * NT;                                     // threads per 4 nodes
    constexpr int kALd = MT == 8 ? 2 * kH : kF;                    // A's row length
    static_assert(WN * WM == NT && MT <= NT, "one wave per 16 features of dZ");
    __shared__ uint2 sD[2][2][4][NT][64];
    __shared__ uint2 sA[2][4][MT][64];
    constexpr int n_tiles = kH / (16 * NT);
    const int tiles = a.M / (16 * MT) * n_tiles;
    const int first = (a.nz[0] + 7) / 8 * 8 * tiles;        // kind 0's workgroups
    const int kind = (int)blockIdx.x < first ? 0 : 1;
    const int b = kind ? blockIdx.x - first : blockIdx.x;
    const int tile = (b >> 3) % tiles;
    const int z = (b >> 3) / tiles * 8 + (b & 7);
    if (z >= a.nz[kind]) return;
    const bf16 *__restrict__ A = a.A[kind], *__restrict__ dZ = a.dZ[kind], *__restrict__ dZlo = a.dZlo[kind];
    const int fb = tile / n_tiles * 16 * MT, jb = tile % n_tiles * 16 * NT;
    const int k0 = z * kKC, k1 = min(a.K[kind], k0 + kKC);
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    // (16 neighbouring lanes read one 128-byte line of a row)
    const int q = tid / FG, fg = tid % FG;
    const bool loads_a = MT == NT || fg < 4 * MT;
    const int mt0 = (wave % WM) * MW, nt0 = (wave / WM) * NW;
    struct Regs { uint2 hi[4], lo[4], a[4]; };
    // A step costs about as many cycles of address and packing instructions as
    // of MFMA, so in a full chunk a step's 12 loads share three base addresses
    // and nothing is checked; a chunk with fewer than kKC nodes reads rows past
    // its end as zeros.
    const int ca = fb + 4 * (loads_a ? fg : 0);
    auto load = [&](auto full, int k, Regs &v) {
        if constexpr (decltype(full)::value) k = min(k, k1 - 64);      // loads ahead of the last steps
        const long row = k + 4 * q;
        const bf16 *h = dZ + row * kH + jb + 4 * fg, *l = dZlo + row * kH + jb + 4 * fg;
        const bf16 *p = A + row * kALd + ca;
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            if constexpr (!decltype(full)::value) {
                v.hi[r] = v.lo[r] = v.a[r] = make_uint2(0, 0);
                if (row + r >= k1) continue;
            }
            v.hi[r] = *(const uint2 *)(h + r * kH);
            v.lo[r] = *(const uint2 *)(l + r * kH);
            v.a[r] = *(const uint2 *)(p + r * kALd);
        }
    };
    // 4 nodes x 4 features -> the 4 features' fragments, which are neighbours
    // in tile fg >> 2; tile t's slots are rotated by 16 t, so that a store's 16
    // lanes meet two to a bank instead of four
    const int t4 = fg >> 2;
    auto put = [&](uint2 (&t)[64], const uint2 (&v)[4]) {
        uint4 *o = (uint4 *)&t[((q & 3) * 16 + (fg & 3) * 4 + 16 * t4) & 63];
        constexpr uint32_t lo = 0x05040100u, hi = 0x07060302u;     // low / high halves of two words
        auto two = [](uint32_t x, uint32_t y, uint32_t sel) { return __builtin_amdgcn_perm(y, x, sel); };
        o[0] = make_uint4(two(v[0].x, v[1].x, lo), two(v[2].x, v[3].x, lo), two(v[0].x, v[1].x, hi),
                          two(v[2].x, v[3].x, hi));
        o[1] = make_uint4(two(v[0].y, v[1].y, lo), two(v[2].y, v[3].y, lo), two(v[0].y, v[1].y, hi),
                          two(v[2].y, v[3].y, hi));
    };
    float4v acc[2][NW][MW];
#pragma unroll
    for (int h = 0; h < 2; ++h)
#pragma unroll
        for (int c = 0; c < NW; ++c)
#pragma unroll
            for (int r = 0; r < MW; ++r) acc[h][c][r] = float4v{0.f, 0.f, 0.f, 0.f};
    // one step: the loaded rows to LDS, the loads of two steps on, the products
    // (one barrier per step: the two LDS buffers alternate)
    auto step = [&](auto full, int k, auto buf_, Regs &v) {
        constexpr int buf = decltype(buf_)::value;
        put(sD[buf][0][q >> 2][t4], v.hi);
        put(sD[buf][1][q >> 2][t4], v.lo);
        if (loads_a) put(sA[buf][q >> 2][t4], v.a);
        load(full, k + 128, v);
        __syncthreads();
#pragma unroll
        for (int ks = 0; ks < 4; ++ks) {
            uint2 fa[MW], fd[2][NW];
#pragma unroll
            for (int r = 0; r < MW; ++r) fa[r] = sA[buf][ks][mt0 + r][(lane + 16 * (mt0 + r)) & 63];
#pragma unroll
            for (int h = 0; h < 2; ++h)
#pragma unroll
                for (int c = 0; c < NW; ++c) fd[h][c] = sD[buf][h][ks][nt0 + c][(lane + 16 * (nt0 + c)) & 63];
#pragma unroll
            for (int h = 0; h < 2; ++h)
#pragma unroll
                for (int c = 0; c < NW; ++c)
#pragma unroll
                    for (int r = 0; r < MW; ++r) acc[h][c][r] = mfma(fd[h][c], fa[r], acc[h][c][r]);
        }
    };
    // pairs of steps (a step past the end adds zeros)
    auto walk = [&](auto full) {
        Regs v0, v1;
        load(full, k0, v0);
        load(full, k0 + 64, v1);
        for (int k = k0; k < k1; k += 128) {
            step(full, k, std::integral_constant<int, 0>{}, v0);
            step(full, k + 64, std::integral_constant<int, 1>{}, v1);
        }
    };
    if (k1 - k0 == kKC) walk(std::true_type{});
    else walk(std::false_type{});
#pragma unroll
    for (int h = 0; h < 2; ++h)
#pragma unroll
        for (int c = 0; c < NW; ++c)
#pragma unroll
            for (int r = 0; r < MW; ++r) {
                const float4v p = acc[h][c][r];
                const long f = fb + (mt0 + r) * 16 + (lane & 15);
                float *o = a.part[kind] + ((long)(2 * z + h) * a.M + f) * kH + jb + (nt0 + c) * 16 + 4 * (lane >> 4);
                *(float4 *)o = make_float4(p[0], p[1], p[2], p[3]);
            }
}

// out = (sum of the hi partials in chunk order) + (sum of the lo partials);
// blockIdx.y: the node kind.
__global__ __launch_bounds__(256) void k_sum_wgrad(WgradArgs a)
{
    const int kind = blockIdx.y, nz = a.nz[kind];
    const long stride = (long)a.M * kH, e = (long)blockIdx.x * 256 + threadIdx.x;
    if (e >= stride) return;
    const float *__restrict__ part = a.part[kind] + e;
    float s = 0.f, t = 0.f;
    int z = 0;
    for (; z + 8 <= nz; z += 8) {
        float h[8], l[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) {
            h[u] = part[(long)(2 * (z + u)) * stride];
            l[u] = part[(long)(2 * (z + u) + 1) * stride];
        }
#pragma unroll
        for (int u = 0; u < 8; ++u) { s += h[u]; t += l[u]; }
    }
    for (; z < nz; ++z) {
        s += part[(long)(2 * z) * stride];
        t += part[(long)(2 * z + 1) * stride];
    }
    a.out[kind][e] = s + t;
}

// ---- the sparse products ---------------------------------------------------------
// The value of lane N of each 16 lanes.
template <int N>
__device__ __forceinline__ uint32_t row_bcast(uint32_t v)
{
    return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x150 + N, 0xf, 0xf, true);
}

// out[s, :] (+)= sum_{p in segment s} a_p in[idx_p, :], FP32 accumulation in
// stored order.  LPS lanes own a segment and 16 bytes of every gathered row
// (16 lanes: BF16 rows of 256 bytes; 32 lanes: FP32 rows of 512 bytes); they
// read 16 (index, value) pairs at once, hand them out by lane permutations and
// keep 8 gathers in flight.
template <int LPS, typename Fma>
__device__ __forceinline__ void spmm_segment(const int *__restrict__ idx, const float *__restrict__ val,
                                             int p, int pe, const char *__restrict__ in, long in_bytes,
                                             Fma &&fma8)
{
    const int l = threadIdx.x & 15;
    in += 16 * (threadIdx.x & (LPS - 1));
    for (Walk w(p, pe, 0); __any(w.has()); w.step(16)) {
        uint32_t j = 0, a = 0;
        if (w.has(l)) {
            j = (uint32_t)idx[w.p + l];
            a = __float_as_uint(val[w.p + l]);
        }
        auto half = [&](auto h) {
            constexpr int B = decltype(h)::value * 8;
            if (!__any(w.has(B))) return;
            const uint32_t jb[8] = {row_bcast<B>(j), row_bcast<B + 1>(j), row_bcast<B + 2>(j),
                                    row_bcast<B + 3>(j), row_bcast<B + 4>(j), row_bcast<B + 5>(j),
                                    row_bcast<B + 6>(j), row_bcast<B + 7>(j)};
            const uint32_t ab[8] = {row_bcast<B>(a), row_bcast<B + 1>(a), row_bcast<B + 2>(a),
                                    row_bcast<B + 3>(a), row_bcast<B + 4>(a), row_bcast<B + 5>(a),
                                    row_bcast<B + 6>(a), row_bcast<B + 7>(a)};
            uint4 r[8];
#pragma unroll
            for (int u = 0; u < 8; ++u) r[u] = *(const uint4 *)(in + (long)jb[u] * in_bytes);
#pragma unroll
            for (int u = 0; u < 8; ++u)
                if (w.has(B + u)) fma8(__uint_as_float(ab[u]), r[u]);
        };
        half(std::integral_constant<int, 0>{});
        half(std::integral_constant<int, 1>{});
    }
}

__global__ __launch_bounds__(256) void k_spmm_bf16(const int *__restrict__ ptr,
                                                   const int *__restrict__ idx,
                                                   const float *__restrict__ val, int nseg,
                                                   const bf16 *__restrict__ in, long in_ld,
                                                   bf16 *__restrict__ out, long out_ld)
{
    const int seg = blockIdx.x * 16 + (threadIdx.x >> 4);
    const bool on = seg < nseg;
    float acc[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
    spmm_segment<16>(idx, val, on ? ptr[seg] : 0, on ? ptr[seg + 1] : 0, (const char *)in,
                     in_ld * sizeof(bf16), [&](float a, uint4 r) {
                         const uint32_t u[4] = {r.x, r.y, r.z, r.w};
#pragma unroll
                         for (int q = 0; q < 4; ++q) {
                             acc[2 * q] += a * bf2f((bf16)(u[q] & 0xffffu));
                             acc[2 * q + 1] += a * bf2f((bf16)(u[q] >> 16));
                         }
                     });
    if (!on) return;
    const uint2 lo = pack4(acc), hi = pack4(acc + 4);
    *(uint4 *)(out + (long)seg * out_ld + 8 * (threadIdx.x & 15)) = make_uint4(lo.x, lo.y, hi.x, hi.y);
}

// out += (the gradient products), rows of 128 FP32
__global__ __launch_bounds__(256) void k_spmm_f32_add(const int *__restrict__ ptr,
                                                      const int *__restrict__ idx,
                                                      const float *__restrict__ val, int nseg,
                                                      const float *__restrict__ in,
                                                      float *__restrict__ out)
{
    const int seg = blockIdx.x * 8 + (threadIdx.x >> 5);
    const bool on = seg < nseg;
    float4 *o = (float4 *)(out + (long)(on ? seg : 0) * kH) + (threadIdx.x & 31);
    const float4 old = *o;
    float acc[4] = {0.f, 0.f, 0.f, 0.f};
    spmm_segment<32>(idx, val, on ? ptr[seg] : 0, on ? ptr[seg + 1] : 0, (const char *)in,
                     kH * sizeof(float), [&](float a, uint4 r) {
                         acc[0] += a * __uint_as_float(r.x);
                         acc[1] += a * __uint_as_float(r.y);
                         acc[2] += a * __uint_as_float(r.z);
                         acc[3] += a * __uint_as_float(r.w);
                     });
    if (on) *o = make_float4(acc[0] + old.x, acc[1] + old.y, acc[2] + old.z, acc[3] + old.w);
}

__global__ void k_d2f(const double *__restrict__ a, float *__restrict__ b, long n)
{
    long i = (long)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) b[i] = (float)a[i];
}
// Parameter i's places in the packed BF16 copies: both matrices' layouts keep
// a matrix inside its own range of the parameter vector; the heads stay FP32.
__device__ __forceinline__ void store_packed(long i, long heads, float v, bf16 *wf, bf16 *wt)
{
    if (i >= heads) return;
    const bf16 h = f2bf(v);
    const long embed = 2L * kF * kH;
    if (i < embed) {
        const int e = (int)(i % (kF * kH));
        wf[i - e + packed_fwd(e / kH, e % kH)] = h;
    } else {
        const int e = (int)((i - embed) % (2 * kH * kH));
        wf[i - e + packed_fwd(e / kH, e % kH)] = h;
        wt[i - e + packed_bwd(e / kH, e % kH)] = h;
    }
}
__global__ void k_pack(const float *__restrict__ w, bf16 *__restrict__ wf, bf16 *__restrict__ wt,
                       long heads)
{
    const long i = (long)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < heads) store_packed(i, heads, w[i], wf, wt);
}

// Features (permuted order, scaled space; see dpdlp.h), column nodes first:
//   column [c~, c~ - c~ref, x~ref, has_lo, has_hi, lo~ or 0, hi~ or 0, 1, 0 ...]
//   row    [b~, b~ - b~ref, y~ref, is_eq, has_lo, has_hi, 0, 1, 0 ...],
//          b = finite lo, else finite hi, else 0
struct FeatArgs {
    int n, m;
    const int *pc, *pr;
    const double *dc, *dr, *c, *cref, *xref, *vlo0, *vhi0, *lo, *hi, *bref, *yref;
    bf16 *Xc, *Xr;
    float *xref_s, *yref_s;
};
__global__ __launch_bounds__(256) void k_features(FeatArgs a)
{
    const int nbx = (a.n + 255) / 256;
    const bool col = (int)blockIdx.x < nbx;
    const int j = (col ? blockIdx.x : blockIdx.x - nbx) * 256 + threadIdx.x;
    if (j >= (col ? a.n : a.m)) return;
    float f[kF] = {0};
    if (col) {
        const int o = a.pc[j];
        const double d = a.dc[j];
        const double lo = a.vlo0[j], hi = a.vhi0[j];
        f[0] = (float)(d * a.c[o]);
        f[1] = (float)(d * (a.c[o] - a.cref[o]));
        f[2] = (float)(a.xref[o] / d);
        f[3] = isfinite(lo) ? 1.f : 0.f;
        f[4] = isfinite(hi) ? 1.f : 0.f;
        f[5] = isfinite(lo) ? (float)fmin(fmax(lo / d, -1e4), 1e4) : 0.f;
        f[6] = isfinite(hi) ? (float)fmin(fmax(hi / d, -1e4), 1e4) : 0.f;
        a.xref_s[j] = f[2];
    } else {
        const int o = a.pr[j];
        const double d = a.dr[j];
        const double l = a.lo[o], h = a.hi[o];
        const double b = isfinite(l) ? l : (isfinite(h) ? h : 0.0);
        f[0] = (float)(d * b);
        f[1] = (float)(d * (b - a.bref[o]));
        f[2] = (float)(a.yref[o] / d);
        f[3] = (isfinite(l) && isfinite(h) && l == h) ? 1.f : 0.f;
        f[4] = isfinite(l) ? 1.f : 0.f;
        f[5] = isfinite(h) ? 1.f : 0.f;
        a.yref_s[j] = f[2];
    }
    f[7] = 1.f;
    uint2 *X = (uint2 *)((col ? a.Xc : a.Xr) + (long)j * kF);
#pragma unroll
    for (int q = 0; q < kF / 4; ++q) X[q] = pack4(f + 4 * q);
}

// The heads and their backward, both node kinds in one launch (kind 0:
// columns, x; kind 1: rows, y).
struct HeadArgs {
    int N[2];
    const bf16 *H[2];            // last activations, rows of 128
    const float *w[2], *ref[2];
    float *pred[2];
    double *out[2];              // prediction in the original order and space, or null
    const int *perm[2];
    const double *scale[2];
    const float *tgt[2];
    float *dpred[2], *dH[2];
    double *part[2];
};
__device__ __forceinline__ int head_side(const HeadArgs &a, int per, int &block)
{
    const int nbx = (a.N[0] + per - 1) / per;
    block = (int)blockIdx.x < nbx ? blockIdx.x : blockIdx.x - nbx;
    return (int)blockIdx.x < nbx ? 0 : 1;
}

// pred_j = ref_j + sum_f H[j, f] w[f]   (sequential over f), and
// out[perm[j]] = scale[j] pred_j  (scaled, permuted -> original: x = D_c x~,
// y = D_r y~)
__global__ __launch_bounds__(256) void k_head(HeadArgs a)
{
    int block;
    const int k = head_side(a, 256, block);
    const int j = block * 256 + threadIdx.x;
    if (j >= a.N[k]) return;
    const uint4 *h = (const uint4 *)(a.H[k] + (long)j * kH);
    const float *w = a.w[k];
    uint4 r[kH / 8];
#pragma unroll
    for (int q = 0; q < kH / 8; ++q) r[q] = h[q];
    float s = 0.f;
#pragma unroll
    for (int q = 0; q < kH / 8; ++q) {
        const uint32_t u[4] = {r[q].x, r[q].y, r[q].z, r[q].w};
#pragma unroll
        for (int v = 0; v < 4; ++v) {
            s += bf2f((bf16)(u[v] & 0xffffu)) * w[q * 8 + 2 * v];
            s += bf2f((bf16)(u[v] >> 16)) * w[q * 8 + 2 * v + 1];
        }
    }
    const float p = a.ref[k][j] + s;
    a.pred[k][j] = p;
    if (a.out[k]) a.out[k][a.perm[k][j]] = a.scale[k][j] * (double)p;
}

// Loss gradient of the heads: d_j = 2 (pred_j - target_j) / N, dH[j, f] = d_j w[f];
// per-block partial sums of the squared error (for the loss) go to part[block].
__global__ __launch_bounds__(256) void k_head_bwd(HeadArgs a)
{
    __shared__ double s[256];
    __shared__ float sd[256];
    int block;
    const int k = head_side(a, 256, block);
    const int n = a.N[k], j0 = block * 256, j = j0 + threadIdx.x;
    double e2 = 0.0;
    float d = 0.f;
    if (j < n) {
        const float r = a.pred[k][j] - a.tgt[k][j];
        e2 = (double)r * (double)r;
        d = 2.f * r / (float)n;
        a.dpred[k][j] = d;
    }
    s[threadIdx.x] = e2;
    sd[threadIdx.x] = d;
    __syncthreads();
    const int f4 = threadIdx.x & 31;
    const float4 w = ((const float4 *)a.w[k])[f4];
    for (int i = threadIdx.x >> 5; i < 256 && j0 + i < n; i += 8) {
        const float di = sd[i];
        ((float4 *)(a.dH[k] + (long)(j0 + i) * kH))[f4] = make_float4(di * w.x, di * w.y, di * w.z, di * w.w);
    }
    for (int o = 128; o > 0; o >>= 1) {
        if (threadIdx.x < o) s[threadIdx.x] += s[threadIdx.x + o];
        __syncthreads();
    }
    if (threadIdx.x == 0) a.part[k][block] = s[0];
}

// dw[f] partials over chunks of kHeadChunk nodes, in node order:
// part[c * kH + f] = sum_{j in chunk c} d_j H[j, f]; column chunks first.  One
// wave per chunk, two features per lane; a serial sum, so its loads go out 32
// nodes ahead.
constexpr int kHeadChunk = 1024;
__global__ __launch_bounds__(64) void k_head_wgrad(HeadArgs a, float *__restrict__ part)
{
    int c;
    const int k = head_side(a, kHeadChunk, c);
    const int j0 = c * kHeadChunk, j1 = min(a.N[k], j0 + kHeadChunk);
    const uint32_t *h = (const uint32_t *)a.H[k] + threadIdx.x;
    const float *d = a.dpred[k];
    float s0 = 0.f, s1 = 0.f;
    int j = j0;
    for (; j + 32 <= j1; j += 32) {
        uint32_t u[32];
#pragma unroll
        for (int q = 0; q < 32; ++q) u[q] = h[(long)(j + q) * (kH / 2)];
#pragma unroll
        for (int q = 0; q < 32; ++q) {
            s0 += d[j + q] * bf2f((bf16)(u[q] & 0xffffu));
            s1 += d[j + q] * bf2f((bf16)(u[q] >> 16));
        }
    }
    for (; j < j1; ++j) {
        const uint32_t u = h[(long)j * (kH / 2)];
        s0 += d[j] * bf2f((bf16)(u & 0xffffu));
        s1 += d[j] * bf2f((bf16)(u >> 16));
    }
    ((float2 *)(part + (long)blockIdx.x * kH))[threadIdx.x] = make_float2(s0, s1);
}
// dw of both heads: the chunks added in order (block 0: columns, 1: rows).
__global__ __launch_bounds__(kH) void k_sum_head(const float *__restrict__ part, int ncx, int ncy,
                                                 float *__restrict__ gx, float *__restrict__ gy)
{
    const int c0 = blockIdx.x == 0 ? 0 : ncx, c1 = blockIdx.x == 0 ? ncx : ncx + ncy;
    float s = 0.f;
    int c = c0;
    for (; c + 16 <= c1; c += 16) {
        float a[16];
#pragma unroll
        for (int u = 0; u < 16; ++u) a[u] = part[(long)(c + u) * kH + threadIdx.x];
#pragma unroll
        for (int u = 0; u < 16; ++u) s += a[u];
    }
    for (; c < c1; ++c) s += part[(long)c * kH + threadIdx.x];
    (blockIdx.x == 0 ? gx : gy)[threadIdx.x] = s;
}

// dZ pair of the embeddings (their inputs need no gradient), 4 features per
// thread, column nodes first.
__global__ __launch_bounds__(256) void k_relu_bwd(long n, const float *__restrict__ dHc,
                                                  const bf16 *__restrict__ Hc, bf16 *__restrict__ dZc,
                                                  bf16 *__restrict__ dZclo, long m,
                                                  const float *__restrict__ dHr,
                                                  const bf16 *__restrict__ Hr, bf16 *__restrict__ dZr,
                                                  bf16 *__restrict__ dZrlo)
{
    long e = (long)blockIdx.x * 256 + threadIdx.x;
    const bool col = e < n * 32;
    if (!col) e -= n * 32;
    if (!col && e >= m * 32) return;
    const long r = e >> 5, f4 = e & 31;
    uint2 hi, lo;
    relu_grad(((const float4 *)(col ? dHc : dHr))[e], ((const uint2 *)((col ? Hc : Hr) + r * 2 * kH))[f4], hi, lo);
    ((uint2 *)(col ? dZc : dZr))[e] = hi;
    ((uint2 *)(col ? dZclo : dZrlo))[e] = lo;
}

__global__ void k_adam(long n, float *__restrict__ w, const float *__restrict__ g,
                       float *__restrict__ m1, float *__restrict__ m2, bf16 *__restrict__ wf,
                       bf16 *__restrict__ wt, long heads, float lr, float b1, float b2, float eps,
                       float c1, float c2)
{
    long i = (long)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    const float gi = g[i];
    const float a = b1 * m1[i] + (1.f - b1) * gi;
    const float b = b2 * m2[i] + (1.f - b2) * gi * gi;
    m1[i] = a;
    m2[i] = b;
    const float wi = w[i] - lr * (a / c1) / (sqrtf(b / c2) + eps);
    w[i] = wi;
    store_packed(i, heads, wi, wf, wt);
}

// Targets: original -> scaled, permuted, out[j] = x[perm[j]] / scale[j]; column
// nodes first.
__global__ __launch_bounds__(256) void k_targets(int n, const double *x, const int *pc,
                                                 const double *dc, float *tx, int m, const double *y,
                                                 const int *pr, const double *dr, float *ty)
{
    const int nbx = (n + 255) / 256;
    const bool col = (int)blockIdx.x < nbx;
    const int j = (col ? blockIdx.x : blockIdx.x - nbx) * 256 + threadIdx.x;
    if (j >= (col ? n : m)) return;
    if (col) tx[j] = (float)(x[pc[j]] / dc[j]);
    else ty[j] = (float)(y[pr[j]] / dr[j]);
}
// out[b] = the sum of the b-th of two runs of partials (np0, then np1 of them)
__global__ __launch_bounds__(256) void k_sum_double(const double *part, int np0, int np1, double *out)
{
    __shared__ double s[256];
    const double *p = part + (blockIdx.x == 0 ? 0 : np0);
    const int np = blockIdx.x == 0 ? np0 : np1;
    double a = 0.0;
    for (int i = threadIdx.x; i < np; i += 256) a += p[i];
    s[threadIdx.x] = a;
    __syncthreads();
    for (int o = 128; o > 0; o >>= 1) {
        if (threadIdx.x < o) s[threadIdx.x] += s[threadIdx.x + o];
        __syncthreads();
    }
    if (threadIdx.x == 0) out[blockIdx.x] = s[0];
}

}  // namespace gnn
}  // namespace dpdlp

using namespace dpdlp;
using namespace dpdlp::gnn;

struct dpdlp_gnn {
    ProblemView pv;
    hipStream_t s = nullptr;
    int L = 3;
    long n_params = 0;
    std::vector<void *> mem;
    // parameters
    float *w = nullptr, *g = nullptr, *m1 = nullptr, *m2 = nullptr;
    bf16 *wf = nullptr, *wt = nullptr;     // packed BF16 weights, for X W and for dZ W^T
    long off_cin = 0, off_rin = 0, off_wx = 0, off_wy = 0;
    std::vector<long> off_c, off_r;
    int adam_t = 0;
    // graph values in FP32
    float *vf = nullptr, *vtf = nullptr;
    // features, references, activations
    bf16 *Xc = nullptr, *Xr = nullptr;
    float *xref = nullptr, *yref = nullptr, *px = nullptr, *py = nullptr;
    float *tx = nullptr, *ty = nullptr, *dpx = nullptr, *dpy = nullptr;
    std::vector<bf16 *> INc, INr;          // index 1..L
    bf16 *Hc_last = nullptr, *Hr_last = nullptr;
    float *dHc = nullptr, *dHr = nullptr, *dSc = nullptr, *dSr = nullptr;
    bf16 *dZc = nullptr, *dZr = nullptr, *dZc_lo = nullptr, *dZr_lo = nullptr;
    float *wpart = nullptr;
    double *lpart = nullptr, *lsum = nullptr;
    double *ref_c = nullptr, *ref_b = nullptr, *ref_x = nullptr, *ref_y = nullptr;
    double *tmp_n = nullptr, *tmp_m = nullptr, *tmp_n2 = nullptr, *tmp_m2 = nullptr, *tmp_m3 = nullptr;
    bool have_ref = false, have_inst = false;
    ~dpdlp_gnn() { for (void *p : mem) (void)hipFree(p); }
};

namespace {

int gfail(hipError_t e, const char *what)
{
    set_error(std::string(what) + ": " + hipGetErrorString(e));
    return e == hipErrorOutOfMemory ? DPDLP_E_OOM : DPDLP_E_HIP;
}
#define GCHK(expr)                                           \
    do {                                                     \
        hipError_t _e = (expr);                              \
        if (_e != hipSuccess) return gfail(_e, #expr);       \
    } while (0)
#define RCHK(expr)                      \
    do {                                \
        int _r = (expr);                \
        if (_r != DPDLP_OK) return _r;  \
    } while (0)

template <typename T>
int galloc(dpdlp_gnn *G, T **p, size_t count)
{
    void *q = nullptr;
    hipError_t e = hipMalloc(&q, std::max<size_t>(count, 1) * sizeof(T));
    if (e != hipSuccess) return gfail(e, "hipMalloc");
    G->mem.push_back(q);
    *p = (T *)q;
    return DPDLP_OK;
}

inline unsigned nb(long n, int b = 256) { return (unsigned)((n + b - 1) / b); }

// persistent workgroups of the dense kernels: two per CU (their LDS), fewer
// where there are fewer than 64 nodes for each
unsigned dense_grid(int N) { return std::min(512u, nb(N, 64)); }

// out = relu(IN W).  Below kFewNodes one wave per 16 nodes and 32 features (a
// launch is then one round trip, and filling 64 KB of LDS with W would be the
// longest part of it), beyond it the persistent form.  A prediction with six
// layer updates of N nodes each, few / persistent, us: N 1024 86 / 100, 4096
// 85 / 112, 8192 99 / 115, 12288 117 / 119, 16384 137 / 124, 20480 159 / 140,
// 32768 222 / 165, 65536 392 / 249.
constexpr int kFewNodes = 12288;
void dense(dpdlp_gnn *G, int N, const bf16 *IN, long off, bf16 *out, long ld)
{
    if (N < kFewNodes)
        hipLaunchKernelGGL(k_dense_few, dim3(nb(N, 16)), dim3(256), 0, G->s, N, IN, G->wf + off, out, ld);
    else
        hipLaunchKernelGGL(k_dense, dim3(dense_grid(N)), dim3(256), 0, G->s, N, IN, G->wf + off, out, ld);
}

// weight gradients of a layer (MT = 8) or of the embeddings (MT = 1)
template <int MT, int NT>
void wgrad(dpdlp_gnn *G, const bf16 *Ac, const bf16 *Ar, int M, float *out_c, float *out_r)
{
    WgradArgs a{};
    a.A[0] = Ac; a.A[1] = Ar;
    a.dZ[0] = G->dZc; a.dZ[1] = G->dZr;
    a.dZlo[0] = G->dZc_lo; a.dZlo[1] = G->dZr_lo;
    a.M = M;
    a.K[0] = G->pv.n; a.K[1] = G->pv.m;
    int wgs = 0;
    for (int k = 0; k < 2; ++k) {
        a.nz[k] = (a.K[k] + kKC - 1) / kKC;
        wgs += (a.nz[k] + 7) / 8 * 8 * (M / (16 * MT) * (kH / (16 * NT)));
    }
    a.part[0] = G->wpart;
    a.part[1] = G->wpart + (long)a.nz[0] * 2 * M * kH;
    a.out[0] = out_c; a.out[1] = out_r;
    hipLaunchKernelGGL((k_wgrad<MT, NT>), dim3(wgs), dim3(64 * NT), 0, G->s, a);
    hipLaunchKernelGGL(k_sum_wgrad, dim3(nb((long)M * kH), 2), dim3(256), 0, G->s, a);
}

void spmm_bf16(dpdlp_gnn *G, bool csr, const bf16 *in, long in_ld, bf16 *out)
{
    const ProblemView &P = G->pv;
    const int nseg = csr ? P.m : P.n;
    hipLaunchKernelGGL(k_spmm_bf16, dim3(nb(nseg, 16)), dim3(256), 0, G->s, csr ? P.rp : P.cp,
                       csr ? P.ci : P.ri, csr ? G->vf : G->vtf, nseg, in, in_ld, out, 2L * kH);
}
void spmm_add(dpdlp_gnn *G, bool csr, const float *in, float *out)
{
    const ProblemView &P = G->pv;
    const int nseg = csr ? P.m : P.n;
    hipLaunchKernelGGL(k_spmm_f32_add, dim3(nb(nseg, 8)), dim3(256), 0, G->s, csr ? P.rp : P.cp,
                       csr ? P.ci : P.ri, csr ? G->vf : G->vtf, nseg, in, out);
}

const bf16 *Hc_of(dpdlp_gnn *G, int l, long *ld)
{
    if (l < G->L) { *ld = 2 * kH; return G->INc[(size_t)l + 1]; }
    *ld = kH;
    return G->Hc_last;
}
const bf16 *Hr_of(dpdlp_gnn *G, int l, long *ld)
{
    if (l < G->L) { *ld = 2 * kH; return G->INr[(size_t)l + 1]; }
    *ld = kH;
    return G->Hr_last;
}

HeadArgs head_args(dpdlp_gnn *G, double *x0, double *y0)
{
    HeadArgs a{};
    a.N[0] = G->pv.n; a.N[1] = G->pv.m;
    a.H[0] = G->Hc_last; a.H[1] = G->Hr_last;
    a.w[0] = G->w + G->off_wx; a.w[1] = G->w + G->off_wy;
    a.ref[0] = G->xref; a.ref[1] = G->yref;
    a.pred[0] = G->px; a.pred[1] = G->py;
    a.out[0] = x0; a.out[1] = y0;
    a.perm[0] = G->pv.perm_col; a.perm[1] = G->pv.perm_row;
    a.scale[0] = G->pv.dc; a.scale[1] = G->pv.dr;
    a.tgt[0] = G->tx; a.tgt[1] = G->ty;
    a.dpred[0] = G->dpx; a.dpred[1] = G->dpy;
    a.dH[0] = G->dHc; a.dH[1] = G->dHr;
    a.part[0] = G->lpart; a.part[1] = G->lpart + nb(G->pv.n);
    return a;
}

// x0, y0: device vectors for the prediction in the original order and space
// (null where it is not wanted)
void forward(dpdlp_gnn *G, double *x0, double *y0)
{
    const int m = G->pv.m, n = G->pv.n, L = G->L;
    hipLaunchKernelGGL(k_embed, dim3(nb(n, 64) + nb(m, 64)), dim3(256), 0, G->s, n, G->Xc,
                       G->wf + G->off_cin, G->INc[1], m, G->Xr, G->wf + G->off_rin, G->INr[1]);
    for (int l = 1; l <= L; ++l) {
        spmm_bf16(G, true, G->INc[l], 2 * kH, G->INr[l] + kH);
        long ldr;
        bf16 *Hr = (bf16 *)Hr_of(G, l, &ldr);
        dense(G, m, G->INr[l], G->off_r[(size_t)l - 1], Hr, ldr);
        spmm_bf16(G, false, Hr, ldr, G->INc[l] + kH);
        long ldc;
        bf16 *Hc = (bf16 *)Hc_of(G, l, &ldc);
        dense(G, n, G->INc[l], G->off_c[(size_t)l - 1], Hc, ldc);
    }
    hipLaunchKernelGGL(k_head, dim3(nb(n) + nb(m)), dim3(256), 0, G->s, head_args(G, x0, y0));
}

void backward(dpdlp_gnn *G)
{
    const int m = G->pv.m, n = G->pv.n, L = G->L;
    const HeadArgs ha = head_args(G, nullptr, nullptr);
    hipLaunchKernelGGL(k_head_bwd, dim3(nb(n) + nb(m)), dim3(256), 0, G->s, ha);
    hipLaunchKernelGGL(k_sum_double, dim3(2), dim3(256), 0, G->s, G->lpart, (int)nb(n), (int)nb(m), G->lsum);
    const int ncx = (int)nb(n, kHeadChunk), ncy = (int)nb(m, kHeadChunk);
    hipLaunchKernelGGL(k_head_wgrad, dim3(ncx + ncy), dim3(64), 0, G->s, ha, G->wpart);
    hipLaunchKernelGGL(k_sum_head, dim3(2), dim3(kH), 0, G->s, G->wpart, ncx, ncy, G->g + G->off_wx,
                       G->g + G->off_wy);

    for (int l = L; l >= 1; --l) {
        long ldc, ldr;
        const bf16 *Hc = Hc_of(G, l, &ldc);
        const bf16 *Hr = Hr_of(G, l, &ldr);
        const long oc = G->off_c[(size_t)l - 1], orow = G->off_r[(size_t)l - 1];
        // column update of layer l; dH_c becomes that of layer l - 1 (without
        // the row update's part, added below)
        hipLaunchKernelGGL(k_dgrad, dim3(dense_grid(n)), dim3(256), 0, G->s, n, G->dHc, Hc, ldc,
                           G->wt + oc, G->dZc, G->dZc_lo, G->dSc);
        spmm_add(G, true, G->dSc, G->dHr);                          // dH_r^l += A~ dS_c
        // row update of layer l
        hipLaunchKernelGGL(k_dgrad, dim3(dense_grid(m)), dim3(256), 0, G->s, m, G->dHr, Hr, ldr,
                           G->wt + orow, G->dZr, G->dZr_lo, G->dSr);
        wgrad<8, 8>(G, G->INc[l], G->INr[l], 2 * kH, G->g + oc, G->g + orow);
        spmm_add(G, false, G->dSr, G->dHc);                         // dH_c^{l-1} += A~^T dS_r
    }
    // embeddings
    hipLaunchKernelGGL(k_relu_bwd, dim3(nb(((long)n + m) * 32)), dim3(256), 0, G->s, (long)n, G->dHc,
                       G->INc[1], G->dZc, G->dZc_lo, (long)m, G->dHr, G->INr[1], G->dZr, G->dZr_lo);
    wgrad<1, 4>(G, G->Xc, G->Xr, kF, G->g + G->off_cin, G->g + G->off_rin);
}

// host or device double vector -> device (staging through tmp when host)
int to_dev(dpdlp_gnn *G, const double *src, int mem_kind, double *stage, long k, const double **out)
{
    if (!src) { *out = nullptr; return DPDLP_OK; }
    if (mem_kind == DPDLP_MEM_HOST) {
        GCHK(hipMemcpyAsync(stage, src, sizeof(double) * (size_t)k, hipMemcpyHostToDevice, G->s));
        *out = stage;
    } else {
        *out = src;
    }
    return DPDLP_OK;
}

}  // namespace

extern "C" {

int dpdlp_gnn_create(dpdlp_problem *prob, int32_t layers, void *stream, dpdlp_gnn **out)
{
    if (!prob || !out || layers < 1 || layers > 8) {
        set_error("bad arguments");
        return DPDLP_E_INVALID_ARG;
    }
    *out = nullptr;
    auto G = std::make_unique<dpdlp_gnn>();
    RCHK(problem_view(prob, &G->pv));
    G->s = (hipStream_t)stream;
    G->L = layers;
    const long m = G->pv.m, n = G->pv.n, nnz = G->pv.nnz;
    // parameter layout
    long off = 0;
    G->off_cin = off; off += (long)kF * kH;
    G->off_rin = off; off += (long)kF * kH;
    for (int l = 0; l < layers; ++l) {
        G->off_c.push_back(off); off += 2L * kH * kH;
        G->off_r.push_back(off); off += 2L * kH * kH;
    }
    G->off_wx = off; off += kH;
    G->off_wy = off; off += kH;
    G->n_params = off;
    RCHK(galloc(G.get(), &G->w, (size_t)off));
    RCHK(galloc(G.get(), &G->g, (size_t)off));
    RCHK(galloc(G.get(), &G->m1, (size_t)off));
    RCHK(galloc(G.get(), &G->m2, (size_t)off));
    RCHK(galloc(G.get(), &G->wf, (size_t)off));
    RCHK(galloc(G.get(), &G->wt, (size_t)off));
    GCHK(hipMemsetAsync(G->w, 0, sizeof(float) * off, G->s));
    GCHK(hipMemsetAsync(G->g, 0, sizeof(float) * off, G->s));
    GCHK(hipMemsetAsync(G->m1, 0, sizeof(float) * off, G->s));
    GCHK(hipMemsetAsync(G->m2, 0, sizeof(float) * off, G->s));
    GCHK(hipMemsetAsync(G->wf, 0, sizeof(bf16) * off, G->s));
    GCHK(hipMemsetAsync(G->wt, 0, sizeof(bf16) * off, G->s));
    RCHK(galloc(G.get(), &G->vf, (size_t)nnz));
    RCHK(galloc(G.get(), &G->vtf, (size_t)nnz));
    if (nnz) {
        hipLaunchKernelGGL(k_d2f, dim3(nb(nnz)), dim3(256), 0, G->s, G->pv.v, G->vf, nnz);
        hipLaunchKernelGGL(k_d2f, dim3(nb(nnz)), dim3(256), 0, G->s, G->pv.vt, G->vtf, nnz);
    }
    RCHK(galloc(G.get(), &G->Xc, (size_t)n * kF));
    RCHK(galloc(G.get(), &G->Xr, (size_t)m * kF));
    float **fv[] = {&G->xref, &G->px, &G->tx, &G->dpx};
    for (auto p : fv) RCHK(galloc(G.get(), p, (size_t)n));
    float **fm[] = {&G->yref, &G->py, &G->ty, &G->dpy};
    for (auto p : fm) RCHK(galloc(G.get(), p, (size_t)m));
    G->INc.assign((size_t)layers + 1, nullptr);
    G->INr.assign((size_t)layers + 1, nullptr);
    for (int l = 1; l <= layers; ++l) {
        RCHK(galloc(G.get(), &G->INc[(size_t)l], (size_t)n * 2 * kH));
        RCHK(galloc(G.get(), &G->INr[(size_t)l], (size_t)m * 2 * kH));
    }
    RCHK(galloc(G.get(), &G->Hc_last, (size_t)n * kH));
    RCHK(galloc(G.get(), &G->Hr_last, (size_t)m * kH));
    RCHK(galloc(G.get(), &G->dHc, (size_t)n * kH));
    RCHK(galloc(G.get(), &G->dHr, (size_t)m * kH));
    RCHK(galloc(G.get(), &G->dSc, (size_t)n * kH));
    RCHK(galloc(G.get(), &G->dSr, (size_t)m * kH));
    RCHK(galloc(G.get(), &G->dZc, (size_t)n * kH));
    RCHK(galloc(G.get(), &G->dZr, (size_t)m * kH));
    RCHK(galloc(G.get(), &G->dZc_lo, (size_t)n * kH));
    RCHK(galloc(G.get(), &G->dZr_lo, (size_t)m * kH));
    const long chunks = (n + kKC - 1) / kKC + (m + kKC - 1) / kKC;
    RCHK(galloc(G.get(), &G->wpart, (size_t)std::max<long>(chunks * 4 * kH * kH, ((n + m) / kHeadChunk + 2) * kH)));
    RCHK(galloc(G.get(), &G->lpart, (size_t)(nb(n) + nb(m))));
    RCHK(galloc(G.get(), &G->lsum, 2));
    double **dn[] = {&G->ref_c, &G->ref_x, &G->tmp_n, &G->tmp_n2};
    for (auto p : dn) RCHK(galloc(G.get(), p, (size_t)n));
    double **dm[] = {&G->ref_b, &G->ref_y, &G->tmp_m, &G->tmp_m2, &G->tmp_m3};
    for (auto p : dm) RCHK(galloc(G.get(), p, (size_t)m));
    GCHK(hipGetLastError());
    GCHK(hipStreamSynchronize(G->s));
    *out = G.release();
    return DPDLP_OK;
}

int dpdlp_gnn_destroy(dpdlp_gnn *G)
{
    if (!G) return DPDLP_OK;
    (void)hipStreamSynchronize(G->s);
    delete G;
    return DPDLP_OK;
}

int64_t dpdlp_gnn_num_params(dpdlp_gnn *G) { return G ? G->n_params : -1; }

int dpdlp_gnn_set_params(dpdlp_gnn *G, const float *params, int64_t count, void *stream)
{
    if (!G || !params || count != G->n_params) { set_error("bad arguments"); return DPDLP_E_INVALID_ARG; }
    G->s = (hipStream_t)stream;
    GCHK(hipMemcpyAsync(G->w, params, sizeof(float) * count, hipMemcpyHostToDevice, G->s));
    hipLaunchKernelGGL(k_pack, dim3(nb(G->off_wx)), dim3(256), 0, G->s, G->w, G->wf, G->wt, G->off_wx);
    GCHK(hipMemsetAsync(G->m1, 0, sizeof(float) * count, G->s));
    GCHK(hipMemsetAsync(G->m2, 0, sizeof(float) * count, G->s));
    G->adam_t = 0;
    GCHK(hipStreamSynchronize(G->s));
    return DPDLP_OK;
}

int dpdlp_gnn_get_params(dpdlp_gnn *G, float *params, float *grads, int64_t count, void *stream)
{
    if (!G || count != G->n_params) { set_error("bad arguments"); return DPDLP_E_INVALID_ARG; }
    G->s = (hipStream_t)stream;
    if (params) GCHK(hipMemcpyAsync(params, G->w, sizeof(float) * count, hipMemcpyDeviceToHost, G->s));
    if (grads) GCHK(hipMemcpyAsync(grads, G->g, sizeof(float) * count, hipMemcpyDeviceToHost, G->s));
    GCHK(hipStreamSynchronize(G->s));
    return DPDLP_OK;
}

int dpdlp_gnn_set_reference(dpdlp_gnn *G, const double *c_ref, const double *b_ref,
                            const double *x_ref, const double *y_ref, int32_t mem_kind, void *stream)
{
    if (!G || !c_ref || !b_ref || !x_ref || !y_ref) { set_error("NULL argument"); return DPDLP_E_INVALID_ARG; }
    if (!mem_kind_ok(mem_kind)) return bad_mem_kind();
    G->s = (hipStream_t)stream;
    const long m = G->pv.m, n = G->pv.n;
    const int k = mem_kind == DPDLP_MEM_HOST ? (int)hipMemcpyHostToDevice : (int)hipMemcpyDeviceToDevice;
    GCHK(hipMemcpyAsync(G->ref_c, c_ref, sizeof(double) * n, (hipMemcpyKind)k, G->s));
    GCHK(hipMemcpyAsync(G->ref_x, x_ref, sizeof(double) * n, (hipMemcpyKind)k, G->s));
    GCHK(hipMemcpyAsync(G->ref_b, b_ref, sizeof(double) * m, (hipMemcpyKind)k, G->s));
    GCHK(hipMemcpyAsync(G->ref_y, y_ref, sizeof(double) * m, (hipMemcpyKind)k, G->s));
    GCHK(hipStreamSynchronize(G->s));
    G->have_ref = true;
    return DPDLP_OK;
}

int dpdlp_gnn_set_instance(dpdlp_gnn *G, const double *c, const double *con_lo, const double *con_hi,
                           int32_t mem_kind, void *stream)
{
    if (!G || !c || !con_lo || !con_hi) { set_error("NULL argument"); return DPDLP_E_INVALID_ARG; }
    if (!mem_kind_ok(mem_kind)) return bad_mem_kind();
    if (!G->have_ref) { set_error("dpdlp_gnn_set_reference first"); return DPDLP_E_INVALID_ARG; }
    G->s = (hipStream_t)stream;
    const int m = G->pv.m, n = G->pv.n;
    const double *dc_, *dlo, *dhi;
    RCHK(to_dev(G, c, mem_kind, G->tmp_n, n, &dc_));
    RCHK(to_dev(G, con_lo, mem_kind, G->tmp_m, m, &dlo));
    RCHK(to_dev(G, con_hi, mem_kind, G->tmp_m2, m, &dhi));
    FeatArgs f{n, m, G->pv.perm_col, G->pv.perm_row, G->pv.dc, G->pv.dr, dc_, G->ref_c, G->ref_x,
               G->pv.vlo0, G->pv.vhi0, dlo, dhi, G->ref_b, G->ref_y, G->Xc, G->Xr, G->xref, G->yref};
    hipLaunchKernelGGL(k_features, dim3(nb(n) + nb(m)), dim3(256), 0, G->s, f);
    GCHK(hipGetLastError());
    GCHK(hipStreamSynchronize(G->s));
    G->have_inst = true;
    return DPDLP_OK;
}

int dpdlp_gnn_forward(dpdlp_gnn *G, double *x0, double *y0, int32_t mem_kind, void *stream)
{
    if (!G) { set_error("NULL argument"); return DPDLP_E_INVALID_ARG; }
    if (!mem_kind_ok(mem_kind)) return bad_mem_kind();
    if (!G->have_inst) { set_error("dpdlp_gnn_set_instance first"); return DPDLP_E_INVALID_ARG; }
    G->s = (hipStream_t)stream;
    const int m = G->pv.m, n = G->pv.n;
    const bool host = mem_kind == DPDLP_MEM_HOST;
    double *dx = x0 ? (host ? G->tmp_n2 : x0) : nullptr;
    double *dy = y0 ? (host ? G->tmp_m3 : y0) : nullptr;
    forward(G, dx, dy);
    if (host && x0) GCHK(hipMemcpyAsync(x0, dx, sizeof(double) * n, hipMemcpyDeviceToHost, G->s));
    if (host && y0) GCHK(hipMemcpyAsync(y0, dy, sizeof(double) * m, hipMemcpyDeviceToHost, G->s));
    GCHK(hipGetLastError());
    GCHK(hipStreamSynchronize(G->s));
    return DPDLP_OK;
}

int dpdlp_gnn_backward(dpdlp_gnn *G, const double *x_target, const double *y_target, int32_t mem_kind,
                       double *loss2, void *stream)
{
    if (!G || !x_target || !y_target) { set_error("NULL argument"); return DPDLP_E_INVALID_ARG; }
    if (!mem_kind_ok(mem_kind)) return bad_mem_kind();
    if (!G->have_inst) { set_error("dpdlp_gnn_set_instance first"); return DPDLP_E_INVALID_ARG; }
    G->s = (hipStream_t)stream;
    const int m = G->pv.m, n = G->pv.n;
    const double *dx, *dy;
    RCHK(to_dev(G, x_target, mem_kind, G->tmp_n, n, &dx));
    RCHK(to_dev(G, y_target, mem_kind, G->tmp_m, m, &dy));
    hipLaunchKernelGGL(k_targets, dim3(nb(n) + nb(m)), dim3(256), 0, G->s, n, dx, G->pv.perm_col,
                       G->pv.dc, G->tx, m, dy, G->pv.perm_row, G->pv.dr, G->ty);
    forward(G, nullptr, nullptr);
    backward(G);
    double h[2];
    GCHK(hipMemcpyAsync(h, G->lsum, sizeof(h), hipMemcpyDeviceToHost, G->s));
    GCHK(hipGetLastError());
    GCHK(hipStreamSynchronize(G->s));
    if (loss2) { loss2[0] = h[0] / n; loss2[1] = h[1] / m; }
    return DPDLP_OK;
}

int dpdlp_gnn_adam_step(dpdlp_gnn *G, double lr, double beta1, double beta2, double eps, void *stream)
{
    if (!G) { set_error("NULL argument"); return DPDLP_E_INVALID_ARG; }
    G->s = (hipStream_t)stream;
    G->adam_t += 1;
    const float c1 = (float)(1.0 - std::pow(beta1, G->adam_t));
    const float c2 = (float)(1.0 - std::pow(beta2, G->adam_t));
    hipLaunchKernelGGL(k_adam, dim3(nb(G->n_params)), dim3(256), 0, G->s, G->n_params, G->w, G->g,
                       G->m1, G->m2, G->wf, G->wt, G->off_wx, (float)lr, (float)beta1, (float)beta2,
                       (float)eps, c1, c2);
    GCHK(hipGetLastError());
    return DPDLP_OK;
}

int dpdlp_gnn_gemm_test(const uint16_t *A, long a_rs, long a_cs, const uint16_t *B, long b_rs,
                        long b_cs, float *C, long ldc, int32_t M, int32_t Nc, int32_t K, void *stream)
{
    if (!A || !B || !C || M < 1 || Nc < 1 || K < 1) { set_error("bad arguments"); return DPDLP_E_INVALID_ARG; }
    hipLaunchKernelGGL(k_gemm, dim3(nb(M, 64), nb(Nc, 64)), dim3(256), 0, (hipStream_t)stream, A, a_rs,
                       a_cs, B, b_rs, b_cs, C, ldc, M, Nc, K);
    GCHK(hipGetLastError());
    GCHK(hipStreamSynchronize((hipStream_t)stream));
    return DPDLP_OK;
}

}  // extern "C"
