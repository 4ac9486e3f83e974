// shapes.hpp -- the tile shapes compiled for the fused sweep, per precision, and what they cost.
//
// An entry X(NWI, NWH, HPT, COLS, PER_CU, COST, STEP, STEP_FULL): NWI interior waves (one output
// site per lane, NWI x 64 / COLS rows of COLS columns), NWH halo waves whose lanes hold HPT halo
// positions each, PER_CU blocks resident on one CU (LDS and registers), and its prices:
//   COST       the relative time of one output site and plane in a full round of the chip, measured
//              at 256^3, by which the default tile is chosen (the one that is reported and that saved
//              settings name: a rule that stays as it is);
//   STEP       microseconds of one step of the march in a launch of one round of one block a CU,
//   STEP_FULL  and in one that fills the chip further (PER_CU blocks on a CU; several rounds, for which
//              a factor comes on top), by which launches are chosen: those of a lattice on its default
//              tile and the slabs of batches.
// COST prices the 16 x 16 and the 8 x 32 double tile alike; STEP was measured on the sweep as it is, over
// cubes of 40 .. 256 sites.  STEP_FULL is fitted to the times of all shapes and up to twelve slab
// lengths on 90 lattices of 1 .. 25 million sites and checked on 130 others.  Double: the choice is 0.4%
// off the fastest in the mean, 6% at worst; with STEP in its place it was 1.7% and 21% (5 x 2000 x 300
// sites, 8 x 32 tiles taken at 146 us where 12 x 32 take 121).  Float: 1.2% and 13%; it was 1.8% and 25%.
// Two blocks on a CU wait for memory together: the second float shape's price is for whole tiles, and
// less for those of which the lattice uses a part (launch_cost).  A build may define its own lists (one
// shape per precision for a quick build, say) before this header.
#pragma once

#ifndef SKYR_SHAPES_F64
#define SKYR_SHAPES_F64(X) \
    X(4, 4, 1, 16, 1, 1.0, 1.6, 1.8) X(4, 4, 1, 32, 1, 1.02, 1.51, 1.58) X(6, 2, 2, 32, 1, 0.95, 2.17, 2.2)
#endif
#ifndef SKYR_SHAPES_F32
#define SKYR_SHAPES_F32(X) \
    X(8, 4, 1, 32, 1, 1.0, 1.5, 1.7) X(6, 2, 2, 32, 2, 2.0, 1.3, 2.9) X(12, 4, 1, 32, 1, 0.9, 2.0, 2.0)
#endif

namespace skyr {

struct Shape {
    int nwi, nwh, hpt, cols;
    int per_cu;
    double cost, step, step_full;
    constexpr int threads() const { return (nwi + nwh) * 64; }
    constexpr int oy() const { return nwi * 64 / cols; }
    constexpr int oz() const { return cols; }
};

#define SKYR_SHAPE_ENTRY(...) Shape{__VA_ARGS__},
constexpr Shape kShapesF64[] = {SKYR_SHAPES_F64(SKYR_SHAPE_ENTRY)};
constexpr Shape kShapesF32[] = {SKYR_SHAPES_F32(SKYR_SHAPE_ENTRY)};
#undef SKYR_SHAPE_ENTRY

}  // namespace skyr
