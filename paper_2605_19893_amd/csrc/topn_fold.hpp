// Indices of the in-launch selection's fold in the standard geometry (l' / d = 4, l / d = 2: block j takes compressed columns
// 4 j - 1 .. 4 j + 3), plain functions so that the host can run them over every position.
#pragma once

namespace ssv {

// The last block that takes a score: J is the block of the query's own slot, the n_local blocks up to it are forced.  -1 where
// they are all there is (a position in the first n_local blocks), not less: the counts below are shifts and divisions of it.
constexpr int fold_last_scored(int J, int n_local) {
    const int last = J - (n_local > 0 ? n_local : 0);
    return last > -1 ? last : -1;
}
// Groups of 64 scored blocks all of whose columns are visible; ncv: visible compressed columns.
constexpr int fold_full_groups(int last_scored, int ncv) {
    const int whole = ncv >> 2;
    return (last_scored + 1 < whole ? last_scored + 1 : whole) >> 6;
}
// First of block j's own four columns, column 0 where it takes no score or has no visible column; j >= 0.  (A row holds a
// multiple of 64 columns: the three behind a visible one exist.)
constexpr int fold_column(int j, int last_scored, int ncv) {
    const int c0 = j <= last_scored ? 4 * j : 0;
    return c0 < ncv ? c0 : 0;
}
// The column before them, column 0 where there is none.
constexpr int fold_left_column(int j, int last_scored, int ncv) {
    const int c0 = j <= last_scored ? 4 * j : 0;
    return c0 >= 1 && c0 - 1 < ncv ? c0 - 1 : 0;
}

}  // namespace ssv
