// fp32 products on the 16-bit matrix unit: operands split into two halves.
//
// A value v is scaled by a power of two s that puts the largest magnitude of
// its tensor into [2^14, 2^15) and split into two fp16 numbers,
//   v s = hi + 2^-11 lo + e,   hi = fp16(v s),  lo = fp16(2^11 (v s - hi)),
// |e| <= 2^-22 |v s| while |v s| is at least 2^-14, that is |v| 2^-28 of the
// largest, and <= 2^-36 absolutely (2^-50 of the largest) below that.  The
// residual of an fp16 number is below 2^-11 of it, so it is kept 2^11 times
// larger, in the range of hi itself; at its own size it would sink into the
// subnormals from 2^-17 of the largest on and a value 2^-40 of it would be lost.
// A product of two such numbers is 2^-11 (lo hi' + hi lo') + hi hi' (lo lo' is
// below 2^-22 of it): three
// v_mfma_f32_16x16x32_f16, which multiply exactly and accumulate in fp32,
// where v_mfma_f32_16x16x4_f32 needs eight instructions of twice the cycles
// for the same K: 48 against 256 cycles.  The sum of 32 products is rounded
// once instead of 32 times, so the result is closer to the exact one than the
// fp32 instruction's: over 576 products of N(0,1) x U(-0.1,0.1) the relative
// error (2-norm) is 1.7e-7 against 4.3e-7.  The scales are exact and are undone on
// the sums.
//
// The cross products lo hi' + hi lo' have an accumulator of their own, added
// last (join): the instruction drops the bits of a product below the accumulator's
// last ones towards -inf, which on one accumulator leaves every sum low by
// 1.1e-8 of the mean magnitude (288 products; error 2.0e-7).  That is nothing for
// one sum, but the bias gradients add millions of them with cancelling signs
// (db off by 9e-6 instead of 3e-6 on 25 x 240 x 240).  Apart it is 1.2e-9.
//
// A split pair takes 4 bytes like the fp32 value: 8 channels are 16 bytes of
// hi followed by 16 bytes of lo, in LDS and in the weight fragments.
//
// Where the scale comes from:
//   h        |h| <= 1 (o tanh c): s = 2^15;
//   weights  the largest magnitude of a gate row (per-row scale);
//   x        the largest magnitude of the tensor.
// The forward's x and h products of a gate row share an accumulator and so one
// scale 2^s = (scale of x) (scale of its W_x) = 2^15 (scale of its W_h), the
// smaller of the two (row_scale): the other weights lie lower in fp16's range.
// Every operand is then off by at most 2^-22 of itself or by what changes the
// pre-activation by 2^-(21 + s).  A call where that exceeds 2^-29 for some row
// (max |x| max |W_x| above 2^20, or max |W_h| so) or that holds a value that is
// not finite keeps the fp32 instruction: the step kernels then read the same 32
// bytes as eight fp32 channels (ctl[0] = 1).  2^-29 a product is below what
// the gate functions are off by (2^-23 in tanh as 1 - 2 / (e^2a + 1)).
// The weight gradients are sums whose size is not known beforehand: they keep the
// fp32 instruction for an x that one scale does not serve (a value that is not
// finite, or more than 1 in 1024 of its non-zero values below 2^-28 of the
// largest, where the split starts to lose bits).  dA has a scale per gate row there,
// lowered as larger values come (split_wgrad.hip).
// The reverse steps scale dA by the largest magnitude of the pixels they stage.  Where
// the loudest gate-unit of some pixel is below 2^-28 of it (da_wide; away from the
// labelled voxels of a masked loss dA falls off exponentially) each pixel has a
// scale of its own instead: a tap's products then start from zero and its sums,
// times 1 / its pixel's scale, are added up in fp32.  A pixel's products are so off by
// at most 2^-22 of its own largest.  The fp32 instruction is kept where a value is
// not finite, and for a unit's weights (a row of W_h^T, W_x^T) of which more than 1 in
// 64 are below 2^-28 of the largest.
#pragma once

#include "common.h"

#include <type_traits>

namespace plstm {

typedef _Float16 h8 __attribute__((ext_vector_type(8)));
typedef _Float16 h4 __attribute__((ext_vector_type(4)));
typedef _Float16 h2 __attribute__((ext_vector_type(2)));
typedef float v4 __attribute__((ext_vector_type(4)));
typedef float v2 __attribute__((ext_vector_type(2)));

constexpr float kHScale = 32768.0f;     // 2^15
constexpr int kStatBlocks = 256;
constexpr unsigned kStatRange = 28u << 23;   // 2^-28 of the largest, in exponent bits
constexpr float kLo = 2048.0f, kLoInv = 1.0f / 2048.0f;   // scale of lo

// One value, already scaled.
__device__ inline void split1(float v, _Float16 &hi, _Float16 &lo)
{
    hi = (_Float16)v;
    lo = (_Float16)__builtin_fmaf((float)hi, -kLo, v * kLo);
}
// Four values, already scaled.  (Two at a time, and hi hidden from the compiler, which
// would fold the scaling into the conversion and convert every value twice: 30 instead
// of 36 instructions per eight values.)
struct Split4 {
    h4 hi, lo;
};
__device__ inline Split4 split4(v4 v)
{
    Split4 s;
#pragma unroll
    for (int i = 0; i < 4; i += 2) {
        h2 h = __builtin_convertvector(v2{v[i], v[i + 1]}, h2);
        asm("" : "+v"(h));
#pragma unroll
        for (int k = 0; k < 2; ++k) {
            s.hi[i + k] = h[k];
            s.lo[i + k] = (_Float16)__builtin_fmaf((float)h[k], -kLo, v[i + k] * kLo);
        }
    }
    return s;
}
struct Split8 {
    h8 hi, lo;
};
// Two f4 (channels 0..3, 4..7), already scaled.
__device__ inline Split8 split8(v4 a, v4 b)
{
    const Split4 x = split4(a), y = split4(b);
    Split8 s;
    s.hi = __builtin_shufflevector(x.hi, y.hi, 0, 1, 2, 3, 4, 5, 6, 7);
    s.lo = __builtin_shufflevector(x.lo, y.lo, 0, 1, 2, 3, 4, 5, 6, 7);
    return s;
}
// The sums of hi hi' and of the cross products.
__device__ inline v4 join(v4 sum, v4 cross)
{
#pragma unroll
    for (int i = 0; i < 4; ++i) sum[i] = __builtin_fmaf(cross[i], kLoInv, sum[i]);
    return sum;
}

__device__ inline v4 mfma_h(h8 a, h8 b, v4 c)
{
    return __builtin_amdgcn_mfma_f32_16x16x32_f16(a, b, c, 0, 0, 0);
}

// Exponent that brings magnitude bits `m` (a finite float's, sign cleared)
// into [2^14, 2^15); 0 for m = 0.
__device__ inline int scale_exp(unsigned m)
{
    if (m == 0) return 0;
    const int e = 14 - ((int)(m >> 23) - 127);
    return e > 110 ? 110 : e;           // (denormals count as 2^-127)
}
__device__ inline float exp2i(int e) { return __uint_as_float((unsigned)(e + 127) << 23); }

// Statistics of a tensor, two passes: per block the largest finite magnitude
// (bits) and whether a value is not finite; then, per block, how many values
// are not zero and how many of those lie below 2^-28 of the tensor's largest.
struct SplitStat {
    unsigned max_bits, bad, nonzero, small;
};
struct SplitStats {
    SplitStat first[kStatBlocks], second[kStatBlocks];
};
// (of fp32 values; clears *ctl too)
int split_stats(const float *x, long long n, SplitStats *part, unsigned *ctl, hipStream_t st);
// What the forward's scales follow from, in one launch: x's largest finite
// magnitude and whether it holds one that is not, and the largest |W_x| and |W_h| of
// every gate row (bits; an infinity or NaN counts).
struct SplitScan {
    SplitStat x[kStatBlocks];
    unsigned row[kDirs * 4 * 64][2];
};
// Clears nclear words of `clear` too.
int split_scan(int dtype, const void *x, long long n, int rows, int nx, int nh, const void *wx,
               const void *wh, SplitScan *scan, int *clear, int nclear, hipStream_t st);

__device__ inline SplitStat stat_combine(SplitStat a, SplitStat b)
{
    SplitStat r;
    r.max_bits = a.max_bits > b.max_bits ? a.max_bits : b.max_bits;
    r.bad = a.bad | b.bad;
    r.nonzero = a.nonzero + b.nonzero;      // (at most 2^31 values)
    r.small = a.small + b.small;
    return r;
}
__device__ inline SplitStat stat_wave(SplitStat s)
{
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) {
        SplitStat t;
        t.max_bits = __shfl_xor(s.max_bits, o);
        t.bad = __shfl_xor(s.bad, o);
        t.nonzero = __shfl_xor(s.nonzero, o);
        t.small = __shfl_xor(s.small, o);
        s = stat_combine(s, t);
    }
    return s;
}
// The kStatBlocks partials of one pass, reduced by a workgroup's first wave
// (`red`: one SplitStat of LDS); every thread returns the result.
__device__ inline SplitStat stat_reduce(const SplitStat *part, SplitStat *red)
{
    if (threadIdx.x < 64) {
        SplitStat s = part[threadIdx.x];
#pragma unroll
        for (int k = 1; k < kStatBlocks / 64; ++k)
            s = stat_combine(s, part[threadIdx.x + 64 * k]);
        s = stat_wave(s);
        if (threadIdx.x == 0) *red = s;
    }
    __syncthreads();
    return *red;
}
// Scale exponent of a gate row's sums, and whether split products serve it; `ex`: scale
// exponent of x.  A row without weights takes any.
constexpr int kMinRowExp = 8;
struct RowScale {
    int s;
    bool fits;
};
__device__ inline RowScale row_scale(int ex, unsigned mx, unsigned mh)
{
    int s = 100;
    if (mx) s = min(s, ex + scale_exp(mx));
    if (mh) s = min(s, 15 + scale_exp(mh));
    if (!mx && !mh) s = kMinRowExp;
    return {s, s >= kMinRowExp && mx < 0x7f800000u && mh < 0x7f800000u};
}
// The scale exponent of x (an x of zeros bounds no row's) and, the same in every
// workgroup, whether split products serve the call's `rows` gate rows.
struct CallScale {
    int ex;
    bool split;
};
__device__ inline CallScale call_scale(const SplitScan *scan, int rows, SplitStat *red)
{
    const SplitStat st = stat_reduce(scan->x, red);
    const int ex = st.max_bits ? scale_exp(st.max_bits) : 100;
    bool ok = !st.bad;
    for (int r = threadIdx.x; r < rows; r += blockDim.x)
        ok &= row_scale(ex, scan->row[r][0], scan->row[r][1]).fits;
    return {ex, __syncthreads_and(ok) != 0};
}
// Magnitudes of a stretch of dA, as biased exponents: x the largest (255: a value is
// not finite), y 255 minus the smallest of the pixels' largest (pixels of zeros apart;
// 0: none).  Stretches join by the maximum of each.
typedef unsigned short DaRange __attribute__((ext_vector_type(2)));
__device__ inline DaRange da_join(DaRange a, DaRange b) { return __builtin_elementwise_max(a, b); }
__device__ inline DaRange da_shuffle(DaRange r, int o)
{
    return __builtin_bit_cast(DaRange, __shfl_xor(__builtin_bit_cast(int, r), o));
}
// Scale exponent of a pixel's gate-units whose largest magnitude has these bits (zeros
// take any).
__device__ inline int pixel_exp(unsigned m) { return min(14 - ((int)(m >> 23) - 127), 110); }
// The maximum over aligned groups of eight lanes, all of them active.
__device__ inline float max8(float m)
{
    auto other = [](float v, auto ctrl) {
        return __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, v),
                                                                     decltype(ctrl)::value, 0xf, 0xf, false));
    };
    m = fmaxf(m, other(m, std::integral_constant<int, 0xB1>{}));     // lanes 1 0 3 2
    m = fmaxf(m, other(m, std::integral_constant<int, 0x4E>{}));     // lanes 2 3 0 1
    return fmaxf(m, other(m, std::integral_constant<int, 0x141>{})); // lanes 7 .. 0
}
__device__ inline float top8(v4 a, v4 b)
{
    float m = 0.0f;
#pragma unroll
    for (int i = 0; i < 4; ++i) m = fmaxf(m, fmaxf(fabsf(a[i]), fabsf(b[i])));
    return m;
}
// Of one pixel whose largest is `m` (bits).
__device__ inline DaRange da_of(unsigned m)
{
    return {(unsigned short)(m >> 23), (unsigned short)(m ? 255u - (m >> 23) : 0u)};
}
// Over a wave whose lanes l, l + 16, l + 32, l + 48 hold one pixel's largest (bits).
__device__ inline DaRange da_wave(unsigned m)
{
#pragma unroll
    for (int o = 32; o > 8; o >>= 1) {
        const unsigned t = __shfl_xor(m, o);
        m = t > m ? t : m;
    }
    DaRange r = da_of(m);
#pragma unroll
    for (int o = 8; o > 0; o >>= 1) r = da_join(r, da_shuffle(r, o));
    return r;
}
// One scale does not serve it.
__device__ inline bool da_wide(DaRange r)
{
    return r.x == 255 || (int)r.x + (int)r.y - 255 > (int)(kStatRange >> 23);
}
// Exponent of its scale (a range of zeros takes any).
__device__ inline int da_exp(DaRange r) { return min(14 - ((int)r.x - 127), 110); }
// Eight weights as fp32 values, from their fragment's two halves: split pairs (the
// value to 22 bits, still scaled), or, `raw`, the values themselves.
struct Wide8 {
    v4 a, b;
};
__device__ inline Wide8 widen8(h8 hi, h8 lo, bool raw)
{
    if (raw) return {__builtin_bit_cast(v4, hi), __builtin_bit_cast(v4, lo)};
    Wide8 w;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        w.a[i] = __builtin_fmaf((float)lo[i], kLoInv, (float)hi[i]);
        w.b[i] = __builtin_fmaf((float)lo[4 + i], kLoInv, (float)hi[4 + i]);
    }
    return w;
}
// One scale serves the tensor.
__device__ inline bool stat_fits(const SplitStat &max, const SplitStat &count)
{
    return !max.bad && count.small <= count.nonzero / 1024u;
}

}  // namespace plstm
