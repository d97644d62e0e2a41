// Where the rows of a segment come from in one decode step.  Plain integer rules, apart from the kernels so that they can
// be compiled and enumerated on the host.
#pragma once

namespace pkv {

// Virtual row numbering of a segment under pruning: rows [0, perm) are the permanent slots, rows
// perm + j are ring slot j (the last d+1 slots of the segment).  r_new is the row of the token stored
// in this step, r_mask the row of a token pruned in this step (-1 if none).
struct RingMap {
    int shift;    // ring slot j is physical slot perm + j + shift
    int r_new;
    int r_mask;
};

struct RowSource {
    bool valid;      // the row takes part in this step
    bool from_new;   // read from k_new / v_new instead of `slot`
    int slot;        // slot of the segment
};

// Row r of the block that starts at row r0 < len.  len_old rows were stored before this step (under pruning: permanent
// ones); app: the step stores a token.  A row that does not take part is read like the block's first one and ignored, so
// that a load needs no branch: no load of the step reads the slot that the step writes.
template <bool EV>
__device__ __forceinline__ RowSource row_source(int r, int r0, int len, int len_old, bool app, const RingMap& ring) {
    RowSource s;
    s.valid = r < len && (!EV || r != ring.r_mask);
    const int x = s.valid ? r : r0;
    s.from_new = EV ? x == ring.r_new : app && x == len_old;
    s.slot = EV && x >= len_old ? x + ring.shift : x;
    return s;
}

}  // namespace pkv
