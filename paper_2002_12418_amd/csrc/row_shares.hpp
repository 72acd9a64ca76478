// A rows dealt to Q shares of wavefronts: consecutive rows, the first A % Q shares have one more.
#pragma once

namespace mnnconv {

struct RowShare { int first, rows; };

constexpr RowShare row_share(int A, int Q, int share)
{
    return RowShare{share * (A / Q) + (share < A % Q ? share : A % Q), A / Q + (share < A % Q ? 1 : 0)};
}

// The row, counted from the share's first, whose operands are loaded for step q of the largest share's steps: a share that has no such row takes
// its last one again (behind it lie the rows of the next share, or the end of the block).
constexpr int row_of_step(int A, int Q, int share, int q)
{
    return q < row_share(A, Q, share).rows ? q : row_share(A, Q, share).rows - 1;
}

}  // namespace mnnconv
