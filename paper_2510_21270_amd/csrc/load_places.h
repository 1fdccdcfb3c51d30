// Where the loads of listed key blocks start.  Plain C++17, so that the host can go through all places.
#pragma once

namespace pbs {

// First key slot of piece `part` (of `step` keys) of listed block j, or -1 where there is nothing to load: an entry that the
// causal structure does not admit (it admits blocks 0 .. ni - 1), or a piece of the last block that lies behind the n-th key whole.
constexpr int listed_slot(int j, int part, int step, int block, int ni, int n)
{
    return j >= 0 && j < ni && j * block + part * step < n ? j * block + part * step : -1;
}

// Scalar offset of a raw buffer load that would start at `at` of a descriptor of `size` bytes (or rows): it stops at the end,
// where every lane is out of range and reads zeros.  The hardware compares a lane's own offset with the size less the
// scalar offset, a difference that must not fall below zero.
constexpr int scalar_offset(int at, int size) { return at < size ? at : size; }

}  // namespace pbs
