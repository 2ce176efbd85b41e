// Host check of merge_short_splits on random segmented matrices:
//   * every nonzero is in exactly one tile, every whole tile is kept;
//   * the pieces of a split that stays are consecutive tiles in piece order
//     (the carries are addressed from the first one's position);
//   * a merged tile covers its whole segment, in pieces of equal size, and
//     comes first in its XCD's run of tiles (after the rest of a split that
//     began in the run before);
// and of the rule that decides which splits are merged: a serial walk of many
// pieces must not be left alone on the chip.
// Built by tests/test_host_checks_cpu.py.
#include "dpdlp_internal.h"

#include <algorithm>
#include <cstdio>
#include <random>

using namespace dpdlp;

static int check(const std::vector<int32_t> &ptr, int tile_nnz)
{
    int bad = 0;
    const int nseg = (int)ptr.size() - 1;
    std::vector<Tile> before, t;
    build_tiles(ptr.data(), nseg, tile_nnz, before);
    t = before;
    merge_short_splits(t);
    std::vector<std::pair<int32_t, int32_t>> cover;
    size_t whole = 0, whole_before = 0;
    for (const Tile &d : before) whole_before += d.npieces == 0;
    const size_t per = (t.size() + 7) / 8;
    for (size_t i = 0; i < t.size(); ++i) {
        const Tile &d = t[i];
        cover.push_back({d.nnz_begin, d.nnz_end});
        whole += d.npieces == 0;
        if (d.npieces > 0 && d.piece == 0)
            for (int p = 0; p < d.npieces; ++p) {
                if (i + (size_t)p >= t.size()) { ++bad; break; }
                const Tile &q = t[i + (size_t)p];
                bad += q.seg_begin != d.seg_begin || q.piece != p || q.npieces != d.npieces;
                bad += q.nnz_begin != ptr[(size_t)d.seg_begin] + p * tile_nnz;
            }
        if (d.npieces < 0) {
            bad += d.seg_end != d.seg_begin + 1 || d.piece != tile_nnz;
            bad += d.nnz_begin != ptr[(size_t)d.seg_begin] || d.nnz_end != ptr[(size_t)d.seg_end];
            bad += (d.nnz_end - d.nnz_begin + tile_nnz - 1) / tile_nnz != -d.npieces;
            // in front of it in its run: merged tiles, or the run's leading rest of a split
            for (size_t j = i; j-- > i / per * per;)
                if (t[j].npieces >= 0) {
                    for (size_t r = i / per * per; r <= j; ++r) bad += t[r].npieces <= 0 || t[r].piece == 0;
                    break;
                }
        }
    }
    bad += whole != whole_before;
    std::sort(cover.begin(), cover.end());
    int32_t at = 0;
    for (auto &c : cover) {
        if (c.first == c.second) continue;          // a tile of empty segments
        bad += c.first != at;
        at = c.second;
    }
    bad += at != ptr.back();
    return bad;
}

// The tiles that R rows of P pieces among S rows of 5 nonzeros merge to.
static int merged(int R, int P, int S, int tile_nnz)
{
    std::vector<int32_t> ptr(1, 0);
    for (int s = 0, r = 0; s < R + S; ++s) {
        const bool lng = r < R && (int64_t)s * R >= (int64_t)r * (R + S);
        ptr.push_back(ptr.back() + (lng ? P * tile_nnz - 5 : 5));
        r += lng;
    }
    std::vector<Tile> t;
    build_tiles(ptr.data(), R + S, tile_nnz, t);
    merge_short_splits(t);
    return (int)std::count_if(t.begin(), t.end(), [](const Tile &d) { return d.npieces < 0; });
}

int main()
{
    int bad = 0;
    std::mt19937 rng(5);
    for (int trial = 0; trial < 600; ++trial) {
        const int tile = trial % 3 == 0 ? 96 : trial % 3 == 1 ? 256 : 512;
        const int one_in = 1 + (int)(rng() % 40), most = 1 + (int)(rng() % 20);
        std::vector<int32_t> ptr(1, 0);
        for (int s = 0, n = 1 + (int)(rng() % 3000); s < n; ++s)
            ptr.push_back(ptr.back() + (int)(rng() % (uint32_t)one_in ? rng() % 9
                                             : rng() % (uint32_t)(most * tile)));
        bad += check(ptr, tile);
    }
    // few long rows alone: their pieces go to as many workgroups
    for (int R : {1, 20, 40, 80, 260}) {
        for (int P : {5, 6, 7, 8}) bad += merged(R, P, 0, 512) != 0;
        for (int P : {2, 4}) bad += merged(R, P, 0, 512) != R;
    }
    bad += merged(400, 5, 0, 512) != 400;           // enough of them for every CU
    // a few pieces behind other tiles, many pieces never for a few rows
    for (int R : {1, 8, 80})
        for (int P : {5, 6}) {
            bad += merged(R, P, 20000, 512) != R;
            if (R < 80) bad += merged(R, P, 2500, 512) != 0;
        }
    for (int R : {1, 8})
        for (int S : {0, 20000, 400000})
            for (int P : {7, 8}) bad += merged(R, P, S, 512) != 0;
    bad += merged(80, 8, 400000, 512) != 80;
    bad += merged(80, 8, 20000, 512) != 0;
    bad += merged(80, 9, 400000, 512) != 0;
    std::printf("%s\n", bad ? "FAILED" : "ok");
    return bad != 0;
}
