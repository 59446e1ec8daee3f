// Workgroups of a launch over (unit, block of its rows) with other work behind them, one a unit (plain C++).
#pragma once

namespace uoe {

// In one dimension: the entry points bound the units, b * k, by 65535, what y and z are certain to take, and work behind the units' rows
// does not fit that bound (units of one block of rows have twice as many workgroups).  x has room for the lot: the attention off the
// 32-grid takes units * rows^2 up to 2^31, which is 2^21 workgroups.
struct UnitGrid {
    int rows, units, behind;   // blocks of rows a unit, units, other workgroups
    constexpr unsigned own() const { return (unsigned)rows * (unsigned)units; }
    constexpr unsigned workgroups() const { return own() + (unsigned)behind; }
    // workgroup `id`: a unit's block of rows, or, from own() on, the other work's id - own()
    constexpr int unit(unsigned id) const { return (int)(id / (unsigned)rows); }
    constexpr int block(unsigned id) const { return (int)(id % (unsigned)rows); }
};

}  // namespace uoe
