// Index arithmetic of the row kernels that read column codes.  Plain constexpr
// functions: the kernels call them, and a host test walks every load of every
// wave with them.
#pragma once

namespace amg {

constexpr int kWave = 64;
constexpr int kNumXcd = 8;  // MI355X: 8 accelerator complex dies, 32 CUs each

// The blocks of RB rows that one workgroup takes: first, first + step, ... below
// end.  Each XCD has one contiguous part of the rows; the grid is one workgroup
// a block, or at least one for each XCD.
struct BlockRange {
    int first, end, step;
};
constexpr BlockRange xcd_range(int blocks, int block, int grid) {
    const int xcd = block % kNumXcd, per = blocks / kNumXcd, rem = blocks % kNumXcd;
    const int before = xcd < rem ? xcd : rem;                 // larger parts below this one
    const int more = xcd < grid % kNumXcd ? 1 : 0;            // workgroups on this XCD
    return BlockRange{xcd * per + before + block / kNumXcd, (xcd + 1) * per + (xcd + 1 < rem ? xcd + 1 : rem),
                      grid / kNumXcd + more};
}

// Slice (of 64 rows) of wave w of block b.  The last block's waves may lie past
// the matrix as a whole (wave_has_rows false): they have no slice of their own,
// and with another slice's distances they would read x past its end.
constexpr int wave_slice(int b, int rb, int w) { return b * (rb / kWave) + w; }
constexpr bool wave_has_rows(int slice, int n) { return slice <= (n - 1) / kWave; }

// The record a wave loads: in bounds also where the wave has no rows (it is not
// used then).
constexpr int slice_at(int slice, int n) { return wave_has_rows(slice, n) ? slice : (n - 1) / kWave; }

// The x a lane loads for one distance of its slice: its own row's where it has
// no such entry.  `on` is false for the lanes past n of a slice that has rows.
constexpr int coded_col(int row, int n, bool on, int off) { return (row < n ? row : n - 1) + (on ? off : 0); }

// The value a lane loads of its slice's entries, `at` counted from the first.
constexpr int coded_val(int at, int last) { return at < last ? at : last; }

}  // namespace amg
