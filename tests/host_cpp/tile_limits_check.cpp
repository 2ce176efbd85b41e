// Host check of the tile kernel's instantiation choice: for every tile size up
// to the largest this build allows, the threads of a workgroup must be able to
// load and stage a whole tile, and the tiles must respect the build's limits;
// and of the workgroups per CU that their LDS allows.
// Built by tests/test_host_checks_cpu.py with the default limits and with
// other ones (DPDLP_TILE_NNZ_MAX, DPDLP_TILE_SEGS_MAX).
#include "dpdlp_internal.h"

#include <algorithm>
#include <cstdio>
#include <random>

using namespace dpdlp;

int main()
{
    int bad = 0;
    for (int t = 1; t <= kTileNnzMax; ++t) {
        const int per = tile_loads(t);
        bad += per * kBlock < t;                        // a tile that does not fit
        bad += per > 1 && per <= 8 && per / 2 * kBlock >= t;    // a smaller one would do
    }
    // workgroups per CU of the largest tiles that 160 KB of LDS allow (products,
    // segment pointers, at most 320 bytes of reductions, the pad)
    if (kTileNnzMax == 2048 && kMaxSegs == 1024) {
        auto wgs = [](int value_bytes, int sides, int sums, bool check) {
            const int fixed = sides * 2048 * value_bytes + 1025 * 4 + sums * 32 + sides * 4 * value_bytes;
            return 160 * 1024 / (fixed + (int)tile_pad(2048, check));
        };
        bad += wgs(8, 1, 1, false) != 5 || wgs(8, 1, 5, false) != 5;    // steps, column check
        bad += wgs(8, 2, 1, false) != 3 || wgs(8, 2, 5, true) != 4;     // partials, row check
        bad += wgs(4, 1, 1, false) != 7;
        bad += tile_pad(1024, false) != 0 || tile_pad(1024, true) != 0;
    }
    // tiles, summing lanes and merged splits at the largest tile size
    std::mt19937 rng(3);
    for (int trial = 0; trial < 20; ++trial) {
        std::vector<int32_t> ptr(1, 0);
        for (int s = 0; s < 4000; ++s) {
            const int len = rng() % 50 ? (int)(rng() % 9) : (int)(rng() % (3 * kTileNnzMax));
            ptr.push_back(ptr.back() + (trial % 4 == 0 ? (int)(rng() % 2) : len));
        }
        std::vector<Tile> tiles;
        build_tiles(ptr.data(), 4000, 0, tiles);
        merge_short_splits(tiles);
        choose_sum_lanes(tiles, ptr.data());
        int64_t nnz = 0;
        for (const Tile &t : tiles) {
            const int cnt = t.npieces < 0 ? t.piece : t.nnz_end - t.nnz_begin;
            bad += cnt > kTileNnzMax || t.seg_end - t.seg_begin > kMaxSegs;
            bad += (t.width_log2 & 15) > 6 || (t.width_log2 >> 8 & 15) > 2 || (t.width_log2 >> 12) > 7;
            nnz += t.nnz_end - t.nnz_begin;
        }
        bad += nnz != ptr.back();
    }
    std::printf("%s\n", bad ? "FAILED" : "ok");
    return bad != 0;
}
