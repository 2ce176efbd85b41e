// Internal declarations shared by the host preprocessing (dpdlp_host.cpp)
// and the device solver (dpdlp_solver.hip).
#pragma once
#include <cstdint>
#include <memory>
#include <new>
#include <string>
#include <utility>
#include <vector>

#include "../../include/dpdlp.h"

namespace dpdlp {

// Tile descriptor: 8 int32 (see dpdlp_build_tiles; on the device width_log2
// also holds what choose_sum_lanes adds, and npieces < 0 marks the tiles that
// merge_short_splits makes).
struct Tile {
    int32_t seg_begin, seg_end, nnz_begin, nnz_end;
    int32_t width_log2, piece, npieces, slice;   // slice: gather slice (sliced sets)
};

// Host arrays of matrix size: resize() leaves the elements uninitialised,
// so that the threads that fill them also take their first-touch page
// faults (a zero-filling resize of 40M elements costs about a second).
template <class T>
struct NoInitAlloc : std::allocator<T> {
    template <class U> struct rebind { using other = NoInitAlloc<U>; };
    NoInitAlloc() = default;
    template <class U> NoInitAlloc(const NoInitAlloc<U> &) {}
    template <class U, class... A> void construct(U *p, A &&...a)
    {
        if constexpr (sizeof...(A) == 0) ::new ((void *)p) U;
        else ::new ((void *)p) U(std::forward<A>(a)...);
    }
};
template <class T> using hvec = std::vector<T, NoInitAlloc<T>>;

// The XCD-sliced form of one format (gathered dimension cut into S slices
// of `size` indices) in compact layout: slice s keeps only the segments
// with a nonzero in its index range, numbered globally in slice-major order
// ("compact segments", seg_base[s] .. seg_base[s+1]); ptr has one entry per
// compact segment (+1) into idx/src, and src[q] is the position in the
// unsliced format that sliced nonzero q comes from.  mask holds, per
// original segment, one bit per slice in S/8 byte planes (plane-major);
// cbase[q * S + s] is the compact index of the first segment of slice s at
// or after original segment q * kBlock.  Tiles carry their slice.
struct SlicedHost {
    int32_t S = 0;
    std::vector<int32_t> bounds;     // slice s gathers indices [bounds[s], bounds[s+1])
    int64_t G = 0;
    hvec<int32_t> ptr, idx, src;
    std::vector<int32_t> seg_base, cbase;
    std::vector<uint8_t> mask;
    std::vector<Tile> tiles;
};
// Distinct 128-byte lines of the gathered vector (line_elems indices per
// line) that the tiles' wave instructions touch: each tile's nonzeros in
// groups of 64 consecutive positions (one wave's load of a tile kernel),
// counted in storage order, or (sorted = true) after ordering every tile's
// nonzeros by gathered index.
int64_t tile_gather_lines(const std::vector<Tile> &tiles, const hvec<int32_t> &idx,
                          int32_t line_elems, bool sorted);
// Orders every tile's nonzeros by gathered index (stable), permuting idx
// and src alike; pos[q] receives, for the nonzero now at q, its position
// inside its tile before the sort (the tile kernel stores its product
// there, so the segment sums keep their order).
void sort_tiles_by_gather(const std::vector<Tile> &tiles, hvec<int32_t> &idx,
                          hvec<int32_t> &src, hvec<uint16_t> &pos);

// Unsliced tile sets: the pieces of a segment split into few become one tile
// (npieces = -pieces, piece = nonzeros per piece) that one workgroup walks, so
// that no launch has to add them up; such tiles come first in each XCD's
// contiguous run of tiles, so that none of them starts last.  Other splits
// stay consecutive tiles.
// The walk is a serial chain.  Up to kMergeAlways pieces take no longer than
// the launch that adds them up; more have to hide behind other tiles: up to
// kMergeBeside where such segments and four times the whole tiles make
// kMergeWhole, up to kMergeMany where kMergeSegs segments of more than
// kMergeBeside are among kMergeFull whole tiles.  Us per iteration, separate /
// merged, R rows of P pieces among S rows of 5 nonzeros, FP64 where not said:
//   P 4: R 40, S 0 8.3 / 8.2; R 400, S 0 11.2 / 10.7; R 8, S 2e4 9.5 / 8.7;
//        R 80, S 4e5 28.8 / 25.3; FP32 R 8, S 1e6 43.6 / 43.9
//   P 5: R 8, S 0 8.3 / 9.0; R 80, S 0 8.9 / 9.3; R 400, S 0 12.7 / 12.3;
//        R 1, S 5000 9.0 / 8.6; R 1, S 2e4 9.5 / 8.7; R 8, S 4e5 26.8 / 25.2
//   P 6: R 80, S 0 9.0 / 10.0; R 260, S 0 11.6 / 12.1; R 400, S 0 14.8 / 14.5;
//        R 8, S 2500 9.0 / 9.4; R 8, S 5000 9.9 / 9.6; R 8, S 4e5 27.2 / 25.8;
//        R 1, S 1.4e6 84.0 / 83.2; FP32 R 8, S 1e6 44.5 / 45.3
//   P 7: R 8, S 1.4e6 86.3 / 88.0; R 80, S 2e5 22.4 / 20.1, 1.4e6 100.1 / 92.1
//   P 8: R 40, S 0 8.0 / 10.6; R 8, S 2e4 9.4 / 10.8; R 80, S 2e4 11.2 / 11.5;
//        R 8, S 1.4e6 85.4 / 90.6; R 80, S 4e5 29.2 / 28.5, 1.4e6 100.3 / 94.3
constexpr int kMergeAlways = 4, kMergeBeside = 6, kMergeMany = 8;
constexpr int64_t kMergeWhole = 384, kMergeSegs = 64, kMergeFull = 1536;
void merge_short_splits(std::vector<Tile> &tiles);

// Lanes of the segment sums of every whole tile: width_log2 holds, beside the
// W of the order of additions (bits 0-7), the h of 2^(W - h) lanes per segment
// (bits 8-11) and, where the FP64 sums take another order with w lanes, w + 1
// (bits 12-15).
void choose_sum_lanes(std::vector<Tile> &tiles, const int32_t *ptr);

// Tiles of one unsliced format, as the device gets them: build_tiles,
// merge_short_splits, choose_sum_lanes.
void plan_tiles(const int32_t *ptr, int32_t nseg, int32_t tile_nnz, std::vector<Tile> &tiles);

// Slices are S contiguous ranges of the gathered index that hold about
// nnz / S nonzeros each; gptr[nidx + 1] is the gathered dimension's own
// pointer array (its nonzero counts as prefix sums).
void slice_bounds(const hvec<int32_t> &gptr, int32_t nidx, int32_t S,
                  std::vector<int32_t> &bounds);
void slice_format(const hvec<int32_t> &ptr, const hvec<int32_t> &idx, const hvec<int32_t> &gptr,
                  int32_t nseg, int32_t nidx, int32_t S, int32_t tile_nnz, SlicedHost &out);
// Number of compact segments (segment, slice) with a nonzero, for S slices.
int64_t count_compact(const hvec<int32_t> &ptr, const hvec<int32_t> &idx,
                      const hvec<int32_t> &gptr, int32_t nseg, int32_t nidx, int32_t S);
// Bytes of the gathered vector (distinct 128-byte lines of line_elems
// indices) touched by `window` consecutive nonzeros in storage order: the
// median over nsample windows spread over the matrix.
double gather_window_bytes(const hvec<int32_t> &idx, int64_t nnz, int32_t nidx, int64_t window,
                           int32_t line_elems, int nsample);

constexpr int kBlock = 256;          // threads per workgroup (4 wave64)
#ifndef DPDLP_TILE_NNZ_MAX
#define DPDLP_TILE_NNZ_MAX 2048
#endif
#ifndef DPDLP_TILE_SEGS_MAX
#define DPDLP_TILE_SEGS_MAX 1024
#endif
constexpr int kTileNnzMax = DPDLP_TILE_NNZ_MAX;   // products staged in LDS per tile
constexpr int kMaxSegs = DPDLP_TILE_SEGS_MAX;     // segments per tile
// positions inside a tile are 16 bits (gather-sorted tiles)
static_assert(kTileNnzMax >= 1 && kTileNnzMax <= 65536 && kMaxSegs >= 1, "tile limits");

// Nonzeros per thread of the tile kernel for tiles of at most tile_nnz: the
// instantiation (1, 2, 4, 8, or what the largest tile needs) with the fewest.
constexpr int kTileLoadsMax = (kTileNnzMax + kBlock - 1) / kBlock > 8 ? (kTileNnzMax + kBlock - 1) / kBlock : 8;
constexpr int tile_loads(int tile_nnz)
{
    const int per = (tile_nnz + kBlock - 1) / kBlock;
    return per <= 1 ? 1 : per <= 2 ? 2 : per <= 4 ? 4 : per <= 8 ? 8 : kTileLoadsMax;
}

// LDS that the kernels of the largest tiles take without using it, so that
// fewer of their workgroups share a CU: where many do, their gathers displace
// each other's lines.  Not for the two-sided check pass on the tiles.  Us per
// launch, with / without it (40M and 10M nonzeros with skewed columns, 9.4M
// uniform, a LASSO of 6.9M, transportation LPs of 18M):
//   FP64, one right-hand side (5 workgroups per CU / 7): dual step 40M 283 /
//     290, 10M 69 / 74, uniform 68 / 69, transportation 73 / 76; primal step of
//     the LASSO 46 / 48; check of the columns 50 / 53
//   FP64 partial sums of two right-hand sides (3 / 4): 10M 100 / 113, 40M 631 /
//     620, uniform 118 / 116, transportation 97 / 96
//   FP32 (7 / 8): 10M dual 47.6 / 48.2, the others within 0.5%
//   two-sided check pass on the tiles (3 / 4): LASSO 68.6 / 66.3, of 9.9M 108 /
//     104, uniform 3.1M 49.0 / 48.4
constexpr unsigned tile_pad(int tile_nnz, bool two_sided_check)
{
    return tile_nnz > 4 * kBlock && !two_sided_check ? 8192 : 0;
}

void set_error(const std::string &msg);

// The nonzeros begin + first, begin + first + s, ... < end of a segment, s per
// step.  Unsigned: the last step passes the end by up to s - 1, and positions
// reach 2^31 - 1, where an int would wrap to a negative position below the end.
struct Walk {
    uint32_t p, end;
    constexpr Walk(int32_t begin_, int32_t end_, uint32_t first)
        : p((uint32_t)begin_ + first), end((uint32_t)end_)
    {
    }
    constexpr bool has(uint32_t ahead = 0) const { return p + ahead < end; }
    constexpr int32_t left() const { return (int32_t)(end - p); }   // where has()
    constexpr void step(uint32_t s) { p += s; }
};

// The two memory kinds of the C ABI.  Any other value is rejected before a
// pointer is touched (a host pointer read as device memory would fault).
inline bool mem_kind_ok(int32_t k) { return k == DPDLP_MEM_HOST || k == DPDLP_MEM_DEVICE; }
int bad_mem_kind();     // sets the message, returns DPDLP_E_INVALID_ARG

// Host copy of an LP after the block permutation, with both formats.
struct HostMatrix {
    int32_t m = 0, n = 0;
    int64_t nnz = 0;
    hvec<int32_t> rp, ci;             // CSR (permuted)
    hvec<double> v;
    hvec<int32_t> cp, ri;             // CSC (permuted), row order kept
    hvec<double> vt;
    std::vector<int32_t> perm_row, perm_col;   // perm[new] = old
};

// Read-only view of a prepared problem's device data (permuted order), for
// the warm-start network, which runs on the same bipartite graph.
struct ProblemView {
    int32_t m = 0, n = 0;
    int64_t nnz = 0;
    const int32_t *rp = nullptr, *ci = nullptr, *cp = nullptr, *ri = nullptr;
    const double *v = nullptr, *vt = nullptr;        // scaled A~ (CSR, CSC)
    const int32_t *perm_row = nullptr, *perm_col = nullptr;
    const double *dr = nullptr, *dc = nullptr;
    const double *vlo0 = nullptr, *vhi0 = nullptr;   // original variable bounds (permuted)
};
int problem_view(dpdlp_problem *P, ProblemView *out);

int validate_host(const dpdlp_csr_lp *lp);
// Start vector of the Golub-Kahan-Lanczos process: w[j] in [-1, 1) from a
// splitmix64 stream; returns ||w||_2.
double lanczos_start(int32_t n, uint64_t seed, double *w);
// Largest singular value of the k x k upper bidiagonal matrix with diagonal
// alpha[0..k-1] and superdiagonal beta[1..k-1] (beta[0] unused), from the
// largest eigenvalue of B^T B by Sturm-sequence bisection.
double bidiag_sigma_max(const double *alpha, const double *beta, int k);
void block_permutation(int32_t count, int32_t block, uint64_t seed, int32_t *perm);
void build_tiles(const int32_t *seg_ptr, int32_t nseg, int32_t tile_nnz,
                 std::vector<Tile> &out);
// Permute rows/columns of a host CSR LP and build the CSC copy.
void permute_and_transpose(const dpdlp_csr_lp *lp, int32_t block, uint64_t seed,
                           int32_t order, HostMatrix &H);

}  // namespace dpdlp
