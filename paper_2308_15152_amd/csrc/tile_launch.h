// Host side of the tile kernel (tile_gemm.hpp): which products it takes, with
// which workgroup tile, and its launch.
#pragma once

#include <stdint.h>

#include <hip/hip_runtime.h>

namespace sgemm_emu {
namespace tile {

// D_t = op(A_t) op(B_t) + C_t, t < batch, D row-major.  a_kc: op(A)'s rows are
// contiguous along k (A stored m x k), otherwise along m (stored k x m);
// b_kc: op(B)'s columns are contiguous along k (B stored n x k), otherwise
// its rows along n (stored k x n).  C null: nothing is added.
struct Problem {
    int m, n, k;
    const float* A;
    int64_t lda, sa;
    bool a_kc;
    const float* B;
    int64_t ldb, sb;
    bool b_kc;
    const float* C;
    int64_t ldc, sc;
    float* D;
    int64_t ldd, sd;
    int batch;
    bool acc;  // accumulate form: its instances, also where C is null
};

// Workgroup tile and number of wave groups that share its k chunks.
enum Shape { T64, T64_K2, T64_K4, T128x64, T128x64_K2, T128, T128_K2, T128x256, NONE, T128x256_FAR };

// The shape expected to be the fastest for this product, NONE if no shape
// takes it (sizes or leading dimensions out of range, more tiles in an item
// than one launch holds, or fewer than four values along an operand's
// contiguous m or n).
Shape choose(const Problem& p);

// T128x256_FAR for a product whose D rows are too far apart for the 32-bit
// offsets of T128x256 and that takes that shape otherwise, else NONE.
Shape far_rows(const Problem& p);

hipError_t launch(const Problem& p, Shape shape, hipStream_t stream);

// Rows and columns of a shape's workgroup tile and its wave groups.
struct Form {
    int rows, cols, groups;
};
Form form(Shape shape);

}  // namespace tile
}  // namespace sgemm_emu
