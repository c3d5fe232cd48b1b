#pragma once
// How a launch spreads the columns of a factor row over lanes (host code, no device
// types: the rules are checked on the CPU over all ranks).
#include "internal.h"

namespace amped {
namespace dev {

// lpr lanes of rpl columns (lpr = 0: the column-tile path), exactly or with overlap.
struct Lanes {
    int lpr = 0, rpl = 1;
    bool exact = true;
};

// How a launch spreads `cols` columns over a lane group.  One load per lane
// covers the row, so the loads of a nonzero take cols * size / 16 lanes of the
// address unit's time instead of a whole wave's (the column-tile path walks one
// nonzero per wave step: 597 us for all modes of 3M nonzeros at rank 20, against
// 167 us here; their gradients 1513 and 186 us).  fp32 rows: 4 columns (16 bytes) per lane.
//  bfloat16 rows of up to 32 columns: 4 columns (8 bytes), so that a wave still
// covers 8 rows per gather at rank 32, except above 16 columns with three or more
// gathered factors, where 16-byte lanes (16 rows per gather instruction) measured
// faster, in every mode of the order-4 tensors, and slower on the order-3 ones;
// wider ones 8 columns.  Fewer columns than a lane reads take the column-tile path.
inline Lanes choose_lanes(int cols, FactorType ft, int nin)
{
    Lanes v;
    const bool f32 = ft == FactorType::F32;
    v.rpl = f32 || cols <= 16 || (cols <= 32 && nin <= 2) ? 4 : 8;
    if (cols < v.rpl) return Lanes{};
    const int need = (cols + v.rpl - 1) / v.rpl;
    v.lpr = v.rpl == 4 ? 2 : 4;
    while (v.lpr < need) v.lpr *= 2;
    v.exact = cols == v.lpr * v.rpl && v.lpr >= 4 && v.lpr <= (f32 ? 32 : 16);
    return v;
}

// Most columns of one launch on the vector path.
constexpr int kMaxVecCols = 256;

// The launches of an MTTKRP: `tile` columns each, the last what is left.  Ranks above
// one launch's columns take equal launches, of whole 16-byte pieces.
//  The row stride decides whether lanes may load several columns at once: the rows of
// an odd bfloat16 rank start on 2 bytes, and loads of 8 and 16 bytes are only made
// from addresses on 4, so these ranks take the column-tile path whatever the tile.
struct Columns {
    int tile = 0;
    Lanes lanes;
};
inline Columns split_columns(int rank, FactorType ft, int nin)
{
    Columns c;
    const int parts = (rank + kMaxVecCols - 1) / kMaxVecCols;
    c.tile = parts == 1 ? rank : ((rank + parts - 1) / parts + 3) & ~3;
    if (ft == FactorType::BF16 && rank % 2) return c;
    c.lanes = choose_lanes(c.tile, ft, nin);
    if (c.tile != rank) c.lanes.exact = false;
    return c;
}

}  // namespace dev
}  // namespace amped
