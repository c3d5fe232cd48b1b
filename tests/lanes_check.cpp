// The lanes of every rank, factor type and number of gathered factors (csrc/lanes.h):
// each launch's lanes cover its columns, stay inside the row, and load from addresses on
// 4 bytes.  Prints the failures and their number.
#include <algorithm>
#include <cstdio>
#include <vector>

#include "lanes.h"

using namespace amped;
using namespace amped::dev;

int main()
{
    int failures = 0, wide = 0;
    auto fail = [&](const char* what, int rank, int ft, int nin) {
        if (++failures <= 20) std::printf("%s: rank %d, type %d, %d factors\n", what, rank, ft, nin);
    };
    for (int rank = 1; rank <= 4096; ++rank)
        for (int ft = 0; ft < 2; ++ft)
            for (int nin = 1; nin <= kMaxOrder - 1; ++nin) {
                const int64_t size = ft == 0 ? 4 : 2;
                const Columns c = split_columns(rank, static_cast<FactorType>(ft), nin);
                const Lanes v = c.lanes;
                if (v.lpr == 0) continue;
                ++wide;
                if (c.tile < 1 || c.tile > kMaxVecCols || v.lpr * v.rpl < c.tile || v.lpr > 64) {
                    fail("lanes do not hold the columns", rank, ft, nin);
                    continue;
                }
                for (int col0 = 0; col0 < rank; col0 += c.tile) {
                    const int ncols = std::min(c.tile, rank - col0);
                    if (ncols < v.rpl) {
                        fail("fewer columns than a lane reads", rank, ft, nin);
                        break;
                    }
                    std::vector<bool> held(ncols, false);
                    bool inside = true, aligned = true;
                    for (int s = 0; s < v.lpr; ++s) {
                        const int at = std::min(s * v.rpl, ncols - v.rpl);
                        for (int i = 0; i < v.rpl; ++i)
                            if (at + i < 0 || at + i >= ncols) inside = false;
                            else held[at + i] = true;
                        for (int64_t row = 0; row < 4; ++row)
                            if ((row * rank + col0 + at) * size % 4 != 0) aligned = false;
                    }
                    if (!inside) fail("a lane outside the row", rank, ft, nin);
                    if (!aligned) fail("a load that is not on 4 bytes", rank, ft, nin);
                    if (std::count(held.begin(), held.end(), false)) fail("a column in no lane", rank, ft, nin);
                    if (v.exact && (ncols != v.lpr * v.rpl || c.tile != rank)) fail("not exact", rank, ft, nin);
                }
            }
    std::printf("%d launches on the vector path, %d failures\n", wide, failures);
    return failures ? 1 : 0;
}
