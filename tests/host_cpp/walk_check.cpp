// Host check of the walks over a segment's nonzeros (Walk) where positions
// reach the largest a nonzero count of 2^31 - 1 allows: every lane's walk must
// end, and together they must visit each position of the segment once.  The
// strides are those of the kernels: 64 to 256 lanes over one segment, 8 or 64
// lanes with four reads ahead, 16 at a time, and the pieces of a merged tile.
// Built with g++ (AddressSanitizer, UBSan) by tests/test_host_checks_cpu.py.
#include "dpdlp_internal.h"

#include <algorithm>
#include <climits>
#include <cstdio>

using namespace dpdlp;

int main()
{
    int bad = 0;
    const int32_t ends[] = {INT_MAX, INT_MAX - 1, INT_MAX - 255, INT_MAX - 256, INT_MAX - 2047, 5000};
    const int32_t lens[] = {0, 1, 2, 63, 64, 65, 255, 256, 257, 511, 2047, 2048, 2049, 4099};
    for (int32_t e : ends)
        for (int32_t len : lens) {
            const int32_t b = e - len;
            // one position per lane and step
            for (uint32_t lanes : {1u, 2u, 16u, 64u, 256u}) {
                std::vector<int> seen((size_t)len, 0);
                for (uint32_t l = 0; l < lanes; ++l) {
                    int trips = 0;
                    for (Walk w(b, e, l); w.has(); w.step(lanes)) {
                        if (++trips > len || w.left() < 1 || w.left() > len) { ++bad; break; }
                        seen[(size_t)(len - w.left())]++;
                    }
                }
                for (int s : seen) bad += s != 1;
            }
            // four positions ahead per step
            for (uint32_t lanes : {8u, 64u}) {
                std::vector<int> seen((size_t)len, 0);
                for (uint32_t l = 0; l < lanes; ++l) {
                    int trips = 0;
                    for (Walk w(b, e, l); w.has(); w.step(4 * lanes)) {
                        if (++trips > len) { ++bad; break; }
                        for (uint32_t u = 0; u < 4; ++u)
                            if (w.has(u * lanes)) seen[(size_t)(w.p + u * lanes - (uint32_t)b)]++;
                    }
                }
                for (int s : seen) bad += s != 1;
            }
            // pieces of a merged tile after the first
            for (int32_t piece : {1, 96, 256, 2048}) {
                if (len <= piece) continue;
                int64_t sum = piece;
                int trips = 0;
                for (Walk w(b, e, (uint32_t)piece); w.has(); w.step((uint32_t)piece)) {
                    if (++trips > len) { ++bad; break; }
                    sum += std::min(piece, w.left());
                }
                bad += sum != len;
            }
        }
    std::printf("%s\n", bad ? "FAILED" : "ok");
    return bad != 0;
}
