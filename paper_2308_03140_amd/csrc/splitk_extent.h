// How far the K-split tile product may read (plain C++, shared with its test on the host).
#pragma once

// Bytes of a descriptor over kn columns of a matrix of leading dimension ld that
// begins at row `row` of the first: up to the end of the last column, not row
// elements past it.  The last tile of rows may reach past ld (its height need
// not divide it), which in the last column is past the matrix.
constexpr unsigned splitk_bytes(int kn, int ld, int row) {
    return kn > 0 ? ((unsigned)kn * (unsigned)ld - (unsigned)row) * 8u : 0u;
}
