// cut.hpp -- how a batch cuts a field's interior planes along x: units, whose sums are kept apart,
// and slabs of whole units, one block per slab and tile.  Plain functions of whole numbers, the same
// on the host, which lays the blocks out, and on the device, where a block finds its planes.
#pragma once

#include <algorithm>

namespace skyr {

// records of a block: the most units that one slab may hold
constexpr int MAX_UNITS = 16;

// First plane of unit k of a field's nx planes in `units` units: of `len` planes (the last one of
// those that are left), or all of the same length (but one), floor(k nx / units), where len is 0.
// k nx passes 2^31 from 185,352 planes on.  In double it is exact (k < 2^21, nx < 2^25, len < 2^31),
// and so is the floor of the rounded quotient: one that is not whole lies at least 1 / units > 2^-21
// off the next whole number, which is less than 2^25 and so rounds 2^-28 at most.  (With 64-bit whole
// numbers the division filled a sixth of the batched kernels' code: 0.3% of 64 fields' time.)
constexpr int unit_start(int k, int nx, int units, int len)
{
    const double product = (double)k * (len > 0 ? len : nx);
    return (int)(len > 0 ? std::min((double)nx, product) : product / units);
}

// planes of slab `slab`, of per_block units
constexpr int slab_planes(int slab, int per_block, int nx, int units, int len)
{
    const int first = slab * per_block, end = std::min(units, first + per_block);
    return unit_start(end, nx, units, len) - unit_start(first, nx, units, len);
}

// units of a field on its default batch tile: an even number, of at most `planes` planes each
constexpr int default_units(int nx, int planes) { return std::min(nx, 2 * ((nx + 2 * planes - 1) / (2 * planes))); }

// units of a slab when slabs of whole units hold at most `cap` planes (one unit at least) and are as
// even as the units allow
constexpr int slab_units(int nx, int units, int cap)
{
    const int most = std::max(1, std::min(MAX_UNITS, (int)((long long)cap * units / nx)));
    const int slabs = (units + most - 1) / most;
    return (units + slabs - 1) / slabs;
}

}  // namespace skyr
