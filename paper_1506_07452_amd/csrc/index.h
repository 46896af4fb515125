// Index arithmetic of the kernels without integer division.
#pragma once

namespace plstm {

// floor(i / w) for 0 <= i < 2^22 and w >= 1, from a float reciprocal: the
// fraction of (i + 0.5) / w is at least 0.5 / w away from an integer, while the
// reciprocal's and the product's rounding make an error below (i / w) 2^-23 <=
// 0.5 / w, so the truncation is exact.  (Above it is not: 4397273 / 63 comes out one
// too large.  Positions inside a staged block are far below; coordinates of a
// plane are not.)
__host__ __device__ inline int fdiv_floor(int i, float inv_w)
{
    return (int)(((float)i + 0.5f) * inv_w);
}

// The blocks of an axis cut into `count` blocks of `size` that block b widened
// by r on both sides touches.  (From the block's number: its coordinates may be
// too large for fdiv_floor.)
struct Span {
    int lo, hi;
};
__host__ __device__ inline Span blocks_touched(int b, int size, int count, int r)
{
    const int reach = fdiv_floor(r + size - 1, 1.0f / (float)size);
    return {b > reach ? b - reach : 0, b + reach < count ? b + reach : count - 1};
}

}  // namespace plstm
