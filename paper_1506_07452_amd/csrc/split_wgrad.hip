// Parameter gradients on the 16-bit matrix unit (split.h): per direction
//   dW[g][k] = sum over voxels of dA[v][g] col[v][k],
// col = the K x K taps of h_{t-1} and of x_t, K of the MFMA running over voxels.
#include "split.h"
#include "strip_plan.h"
#include "sweep.h"

namespace plstm {
namespace {

typedef v4 f4;
typedef __fp16 g4 __attribute__((ext_vector_type(4)));
typedef __attribute__((address_space(3))) g4 lds_g4;
typedef __attribute__((address_space(3))) char lds_char;

constexpr int kWaves = 8, kThreads = 64 * kWaves;
constexpr int kRowA = 288;               // bytes of a staged dA pixel: 64 gates as split tiles, 32 pad
constexpr int kStatic = 2048;            // LDS of k_wgrad_h2 beside its stage buffers, at most
constexpr int kXB = 2;                   // staged 8-channel slots of [h | x] per thread

// Transposed LDS read: within a group of 16 lanes lane l names 8 bytes (four
// columns) of row l / 4 and receives rows 0 .. 3 of column l.
__device__ inline h4 tr4(lds_char *base, int off)
{
    return __builtin_bit_cast(h4, __builtin_amdgcn_ds_read_tr16_b64_v4f16((lds_g4 *)(base + off)));
}
__device__ inline h8 tr8(lds_char *base, int o0, int o1)
{
    const h4 a = tr4(base, o0), b = tr4(base, o1);
    h8 r;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        r[i] = a[i];
        r[4 + i] = b[i];
    }
    return r;
}

struct WgH2Args {
    Geom g;
    int C8;                   // channels of x in memory
    int CT, PC, TG;           // column tiles (U of h, then x's), tiles and tap groups of a part
    int nct;                  // parts along the column tiles
    int kch, NTt;             // voxel chunks per part, N-tiles of a row of partial
    const float *x, *hd, *dA;
    const SplitStats *part;   // x's statistics
    unsigned *ctl;            // 1: left to the fp32 kernel (cleared before)
    float *partial;           // [nd][kch][4O][16 NTt]
    int rowB;                 // bytes of a staged [h | x] pixel
    int bufb;                 // bytes of one stage buffer
    int bp[kDirs], bq[kDirs], nbq[kDirs], nblk[kDirs];
};

// One workgroup of eight waves per (direction, 64 gates, PC column tiles, chunk of
// the direction's pixel blocks); it owns the whole [64 gates x PC 16 K K] partial
// sum.  Wave items are (column tile, group of NT taps) with the 64 gates: 4 NT
// accumulator tiles; KS = 8 / items waves share an item, each taking every KS-th
// 32-pixel piece of a block.
// - A block of 64 DB pixels of dA and the [h_{t-1} | x_t] pixels its taps reach are
//   staged as split pairs in their own order (channels contiguous); the operands,
//   which need eight consecutive voxels of one channel per lane, are read with the
//   transposing LDS read, so a tap is an address offset and nothing is staged per
//   tap.  Pixels are 32 bytes past a multiple of 64 apart: the 16 rows of a read
//   fall on distinct banks.  Two buffers; the next block's loads are in
//   flight beside this block's products.
// - The three products of a piece start from zero and are added to the
//   accumulators in fp32 (round to nearest): over the millions of voxels of a
//   direction the instruction's own rounding towards -inf would add up.
// - dA has a scale per gate row, which is undone on the sums: rows of a shut gate or
//   an idle unit lie far below the others.  A row's scale starts from its largest value in
//   the workgroup's first block, brought to 2^10; a value that reaches 2^15 under it has
//   the block's row maxima found, the scales of such rows lowered, their
//   sums with them, and the block split again (a few times a workgroup).  What lies
//   2^-24 or more below a row's largest loses bits only beside sums that size.
// Bound by the waves' own instruction stream: of 9.5 kilocycles a block (32 -> 32
// units, 3 x 3) the products are 3.8, each wave's loads, splits and LDS stores 3
// and the transposed reads' latency most of the rest.  Measured against the fp32
// GEMM it replaces (im2col columns staged per tap, or operands streamed from
// memory), with the reduction: 32 -> 32 units on 48 x 240 x 240 24.1 -> 9.8 ms, on
// 25 x 240 x 240 12.6 -> 5.7; 64 -> 64 on 20 x 64 x 64 3.2 -> 1.2; 7 x 7, 25 -> 32 on
// 15 x 128 x 128 10.7 -> 4.5; 16 -> 16, 5 x 5 on 2 x 61 x 132 x 144 19.0 -> 5.1; error
// against 64 bits 4.6e-6 -> 9e-7.  After the persistent reverse sweep (16 units, 3
// channels on 48 x 240 x 240, training step of two layers) 49.9 -> 47.9 ms and after
// the 2D line blocks (30 x 512 x 512 x 1, forward and backward) 17.7 -> 16.6, where
// a wave streamed operands from memory for fp32 products.  Generic pointers into LDS and values hoisted out
// of the block loop cost 120 spilled registers (15.1 ms on the second).
template <int NT, int DB>
__global__ void __launch_bounds__(kThreads, 1) __attribute__((amdgpu_waves_per_eu(2, 2)))
k_wgrad_h2(WgH2Args a)
{
    extern __shared__ h8 wl_smem[];
    __shared__ SplitStat red[2];
    __shared__ float rscale[64], rlower[64];    // of each gate row: scale, and factor of its sums
    __shared__ int rexp[64];                    // exponent of the scale
    __shared__ unsigned rmax[64];               // largest |dA| of the block (bits)
    __shared__ int raised[2];                   // a row's scale is too large for the block, by parity
    const SplitStat xs = stat_reduce(a.part->first, &red[0]);
    if (!stat_fits(xs, stat_reduce(a.part->second, &red[1]))) {
        if (blockIdx.x == 0 && threadIdx.x == 0) *a.ctl = 1u;
        return;
    }
    constexpr int TP = 64 * DB;
    const int tid = threadIdx.x, lane = tid & 63, q4 = lane >> 4, col = lane & 15;
    const int wv = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int O = a.g.O, U = O >> 4, G = 4 * O;
    // (integer division leaves uniform values in vector registers: an index into
    // the arguments made of them would be a memory round trip a use)
    auto uni = [](int v) { return __builtin_amdgcn_readfirstlane(v); };
    int r = blockIdx.x;
    const int kc = uni(r % a.kch);
    r = uni(r / a.kch);
    const int cp = uni(r % a.nct);
    r = uni(r / a.nct);
    const int mg = uni(r % U), d = uni(r / U);
    const int PC = a.PC, NI = PC * a.TG, KS = uni(min(kWaves / NI, TP / 32));
    const int item = uni(wv % NI), ks = uni(wv / NI), ic = uni(item % PC);
    const int ct = cp * PC + ic, tg = uni(item / PC);
    const bool busy = ks < KS && ct < a.CT;
    const DirGeom dg = a.g.dir[d];
    const int ss = (int)dg.ss, sp = (int)dg.sp, sq = (int)dg.sq, P = dg.P, Q = dg.Q;
    const long long V = a.g.V;
    const int KQ = a.g.KQ, KK = a.g.KP * KQ, radp = a.g.KP >> 1, radq = KQ >> 1;
    const int BP = a.bp[d], BQ = a.bq[d], NBQ = a.nbq[d], NBLK = a.nblk[d], SW = BQ + 2 * radq, SH = BP + 2 * radp;
    const int C8 = a.C8, rowB = a.rowB, NSL = PC * 2;
    char *const smem = (char *)wl_smem;

    const int exx = scale_exp(xs.max_bits);
    const float sx = exp2i(exx);
    if (tid < 64) {
        rexp[tid] = 110;
        rscale[tid] = exp2i(110);
    }
    if (tid < 2) raised[tid] = 0;
    __syncthreads();

    // this wave's taps and its lane's rows of a piece (voxel 16 j + 4 q + i of the
    // piece for k = 8 q + 4 j + i)
    const int per = (KK + a.TG - 1) / a.TG;
    const int tap0 = min(tg * per, KK), ntap = min(KK - tap0, per);
    int toff[NT];
#pragma unroll
    for (int j = 0; j < NT; ++j) {
        const int tap = min(tap0 + j, KK - 1);
        const int ka = tap / KQ, kb = tap - ka * KQ;
        toff[j] = uni(((ka - radp) * SW + kb - radq) * rowB);
    }
    const int lrow = 4 * q4 + (col >> 2);
    // staged center pixel of row e (rows past the block read its first pixel: their dA is zero)
    auto b_row = [&](int e) {
        const int ey = fdiv_floor(e, 1.0f / (float)BQ), ex = e - ey * BQ;
        const int px = ey < BP ? (ey + radp) * SW + ex + radq : radp * SW + radq;
        return TP * kRowA + px * rowB + ic * 64 + (lane & 3) * 8;
    };

    // staging: one dA slot (8 gates) of pixel (tid >> 3) + 64 u, and kXB slots of
    // [h | x], per thread
    f4 ra[DB][2], rb[kXB][2];
    bool oka[DB], okb[kXB];
    f4 dbs[2] = {{0.0f, 0.0f, 0.0f, 0.0f}, {0.0f, 0.0f, 0.0f, 0.0f}};   // bias sums of this thread's slot
    const int nstb = SH * SW * NSL;
    const float inv_nsl = 1.0f / (float)NSL, inv_sw = 1.0f / (float)SW, inv_bq = 1.0f / (float)BQ;
    // `fresh` hides where a value comes from, so that what is computed of it is
    // computed again for each block instead of being kept in registers that the
    // accumulators need (a hundred of them, spilled)
    auto fresh = [](int v) {
        asm volatile("" : "+v"(v));
        return v;
    };
    auto fetch = [&](int n, int t, int blk) {
        const int ti = fresh(tid);
        const int bi = uni(blk / NBQ), p0 = bi * BP, q0 = (blk - bi * NBQ) * BQ;
        const int s = dg.sign > 0 ? t : dg.T - 1 - t;
        const long long sb = ((long long)d * a.g.N + n) * V;
        const float *const dA_n = a.dA + sb * G + mg * 64, *const h_n = a.hd + sb * O;
        const float *const x_n = a.x + (long long)n * V * C8;
#pragma unroll
        for (int u = 0; u < DB; ++u) {
            const int e = (ti >> 3) + 64 * u;
            const int ey = fdiv_floor(e, inv_bq), ex = e - ey * BQ;
            oka[u] = ey < BP && p0 + ey < P && q0 + ex < Q;
            const int v = s * ss + (p0 + ey) * sp + (q0 + ex) * sq;
            const float *src = dA_n + (oka[u] ? (long long)v * G + 8 * (ti & 7) : 0);
            ra[u][0] = *(const f4 *)src;
            ra[u][1] = *(const f4 *)(src + 4);
        }
#pragma unroll
        for (int u = 0; u < kXB; ++u) {
            const int e = ti + kThreads * u;
            const int spx = fdiv_floor(e, inv_nsl), c = e - spx * NSL;
            const int sy = fdiv_floor(spx, inv_sw), sxx = spx - sy * SW;
            const int pp = p0 - radp + sy, qq = q0 - radq + sxx;
            const int tile = cp * PC + (c >> 1);
            const bool is_h = tile < U;
            const int ch = (is_h ? tile : tile - U) * 16 + (c & 1) * 8;
            okb[u] = e < nstb && (unsigned)pp < (unsigned)P && (unsigned)qq < (unsigned)Q &&
                     (is_h ? t > 0 : ch < C8);
            const int v = s * ss + pp * sp + qq * sq;
            const float *src = is_h ? h_n : x_n;
            const int off = is_h ? (v - dg.sign * ss) * O + ch : v * C8 + ch;
            src = okb[u] ? src + off : x_n;
            rb[u][0] = *(const f4 *)src;
            rb[u][1] = *(const f4 *)(src + 4);
        }
    };
    const f4 zero = {0.0f, 0.0f, 0.0f, 0.0f};
    auto add_bias = [&]() {
#pragma unroll
        for (int u = 0; u < DB; ++u) {
            dbs[0] += oka[u] ? ra[u][0] : zero;
            dbs[1] += oka[u] ? ra[u][1] : zero;
        }
    };
    auto commit = [&](char *buf, int *flag) {
        const int ti = fresh(tid);
        const int c = ti & 7;
        const f4 s0 = *(const f4 *)&rscale[8 * c], s1 = *(const f4 *)&rscale[8 * c + 4];
        float top = 0.0f;
#pragma unroll
        for (int u = 0; u < DB; ++u) {
            const f4 v0 = (oka[u] ? ra[u][0] : zero) * s0, v1 = (oka[u] ? ra[u][1] : zero) * s1;
#pragma unroll
            for (int k = 0; k < 4; ++k) top = fmaxf(top, fmaxf(fabsf(v0[k]), fabsf(v1[k])));
            const Split8 w = split8(v0, v1);
            char *p = buf + ((ti >> 3) + 64 * u) * kRowA + (c >> 1) * 64 + (c & 1) * 16;
            *(h8 *)p = w.hi;
            *(h8 *)(p + 32) = w.lo;
        }
        if (top >= kHScale) *flag = 1;
#pragma unroll
        for (int u = 0; u < kXB; ++u) {
            const int e = ti + kThreads * u;
            if (e >= nstb) continue;
            const int spx = fdiv_floor(e, inv_nsl), c = e - spx * NSL;
            const float sc = cp * PC + (c >> 1) < U ? kHScale : sx;
            const Split8 w = split8(okb[u] ? rb[u][0] * sc : zero, okb[u] ? rb[u][1] * sc : zero);
            char *p = buf + TP * kRowA + spx * rowB + (c >> 1) * 64 + (c & 1) * 16;
            *(h8 *)p = w.hi;
            *(h8 *)(p + 32) = w.lo;
        }
    };

    f4 acc[4][NT];
#pragma unroll
    for (int m = 0; m < 4; ++m)
#pragma unroll
        for (int j = 0; j < NT; ++j) acc[m][j] = zero;

    lds_char *const lds = (lds_char *)smem;
    auto piece = [&](int buf, int pc) {
        h8 av[4][2];
        const int lr = fresh(lrow);
        const int pa = buf + (pc * 32 + lr) * kRowA + (lane & 3) * 8;
#pragma unroll
        for (int m = 0; m < 4; ++m)
#pragma unroll
            for (int hl = 0; hl < 2; ++hl)
                av[m][hl] = tr8(lds, pa + m * 64 + hl * 32, pa + 16 * kRowA + m * 64 + hl * 32);
        const int b0 = buf + b_row(pc * 32 + lr), b1 = buf + b_row(pc * 32 + 16 + lr);
        h8 bh = tr8(lds, b0 + toff[0], b1 + toff[0]);
        h8 bl = tr8(lds, b0 + toff[0] + 32, b1 + toff[0] + 32);
#pragma unroll
        for (int j = 0; j < NT; ++j) {
            h8 nh = bh, nl = bl;
            if (j + 1 < NT) {
                nh = tr8(lds, b0 + toff[j + 1], b1 + toff[j + 1]);
                nl = tr8(lds, b0 + toff[j + 1] + 32, b1 + toff[j + 1] + 32);
            }
#pragma unroll
            for (int m = 0; m < 4; m += 2) {
                f4 x0 = mfma_h(av[m][1], bh, zero), x1 = mfma_h(av[m + 1][1], bh, zero);
                f4 y0 = mfma_h(av[m][0], bh, zero), y1 = mfma_h(av[m + 1][0], bh, zero);
                x0 = mfma_h(av[m][0], bl, x0);
                x1 = mfma_h(av[m + 1][0], bl, x1);
                acc[m][j] += join(y0, x0);
                acc[m + 1][j] += join(y1, x1);
            }
            bh = nh;
            bl = nl;
            __builtin_amdgcn_sched_barrier(0);
        }
    };

    // after a commit and its barrier, where that found a scale too large: row maxima of
    // the block in flight, the scales and sums that follow; false where it is not finite
    auto lower_scales = [&](int *flag) {
        if (tid < 64) rmax[tid] = 0u;
        __syncthreads();
        if (tid == 0) *flag = 0;
#pragma unroll
        for (int u = 0; u < DB; ++u)
#pragma unroll
            for (int k = 0; k < 8; ++k) {
                const unsigned m = __float_as_uint(ra[u][k >> 2][k & 3]) & 0x7fffffffu;
                if (oka[u]) atomicMax(&rmax[8 * (tid & 7) + k], m);
            }
        __syncthreads();
        bool finite = true;
        if (tid < 64) {
            const int e = (int)(rmax[tid] >> 23) - 127, old = rexp[tid];
            finite = e < 128;
            const int now = e + old >= 15 ? 10 - e : old;
            rexp[tid] = now;
            rscale[tid] = exp2i(now);
            rlower[tid] = now - old < -126 ? 0.0f : exp2i(now - old);
        }
        finite = __syncthreads_and(finite) != 0;
#pragma unroll
        for (int m = 0; m < 4; ++m) {
            const f4 f = *(const f4 *)&rlower[m * 16 + 4 * q4];
#pragma unroll
            for (int j = 0; j < NT; ++j) acc[m][j] *= f;
        }
        return finite;
    };
    // this workgroup's blocks: (n, t, blk), blk fastest
    const long long tot = (long long)a.g.N * dg.T * NBLK;
    // (fewer than 2^31 blocks)
    const int u0 = uni((int)(tot * kc / a.kch)), u1 = uni((int)(tot * (kc + 1) / a.kch));
    if (u0 < u1) {
        int blk = uni((int)(u0 % NBLK));
        const int rest = uni((int)(u0 / NBLK));
        int t = uni(rest % dg.T), n = uni(rest / dg.T);
        bool finite = true;
        // block u's products beside block u + 1's loads (one pass of the loop before the first)
        for (int u = u0 - 1; finite && u < u1; ++u) {
            const int buf = ((u - u0) & 1) * a.bufb;
            const bool more = u + 1 < u1;
            if (more) {
                fetch(n, t, blk);
                if (++blk == NBLK) {
                    blk = 0;
                    if (++t == dg.T) {
                        t = 0;
                        ++n;
                    }
                }
            }
            __builtin_amdgcn_sched_barrier(0);
            if (busy && u >= u0)
#pragma unroll 1
                for (int pc = ks; pc < TP / 32; pc += KS) piece(buf, pc);
            __builtin_amdgcn_sched_barrier(0);
            if (more) add_bias();
            // (two flags: a wave may set the next block's before another has read this one's)
            int *const flag = &raised[(u - u0) & 1];
            for (bool again = true; again;) {
                if (more) commit(smem + (((u - u0) & 1) ^ 1) * a.bufb, flag);
                __syncthreads();
                again = more && *(volatile int *)flag != 0;
                if (__builtin_expect(again, 0)) {
                    finite = lower_scales(flag);
                    again = finite;
                }
            }
        }
        if (!finite) {
            if (tid == 0) *a.ctl = 1u;
            return;
        }
    }

    // the KS waves of an item, summed in order through LDS, one row tile at a time
    f4 *const xch = (f4 *)smem;
    if (KS > 1) {
#pragma unroll
        for (int m = 0; m < 4; ++m) {
            if (busy && ks > 0) {
#pragma unroll
                for (int j = 0; j < NT; ++j) xch[((ks * NI + item) * NT + j) * 64 + lane] = acc[m][j];
            }
            __syncthreads();
            if (busy && ks == 0)
                for (int k = 1; k < KS; ++k) {
#pragma unroll
                    for (int j = 0; j < NT; ++j) acc[m][j] += xch[((k * NI + item) * NT + j) * 64 + lane];
                }
            __syncthreads();
        }
    }
    const int KCp = a.NTt * 16, KO = KK * O, C = a.g.C;
    float *const out = a.partial + (((long long)d * a.kch + kc) * G + mg * 64) * KCp;
    if (busy && ks == 0) {
        const bool is_h = ct < U;
        const float inv2 = is_h ? 1.0f / kHScale : exp2i(-exx);
        const int c = (is_h ? ct : ct - U) * 16 + col;
#pragma unroll
        for (int j = 0; j < NT; ++j) {
            if (j >= ntap || (!is_h && c >= C)) continue;
            const int tap = tap0 + j;
            const int column = is_h ? tap * O + c : KO + tap * C + c;
#pragma unroll
            for (int m = 0; m < 4; ++m)
#pragma unroll
                for (int i = 0; i < 4; ++i)
                    out[(long long)(m * 16 + 4 * q4 + i) * KCp + column] =
                        acc[m][j][i] * inv2 * exp2i(-rexp[m * 16 + 4 * q4 + i]);
        }
    }
    // bias sums: 64 threads hold slot s (gates 8 s .. 8 s + 7)
    if (cp == 0) {
        __syncthreads();
        xch[tid * 2] = dbs[0];
        xch[tid * 2 + 1] = dbs[1];
        __syncthreads();
        if (tid < 64) {
            const float *f = (const float *)smem;
            float v = 0.0f;
            for (int k = 0; k < 64; ++k) v += f[(k * 8 + (tid >> 3)) * 8 + (tid & 7)];
            out[(long long)tid * KCp + KO + KK * C] = v;
        }
    }
}

// ---- host side --------------------------------------------------------------

inline int pad8(int c) { return (c + 7) / 8 * 8; }

struct WgPlan {
    int NT, TG, CT, PC, nct, KS, TP, kch, NTt, rowB, bufb;
    int bp[kDirs], bq[kDirs], nbq[kDirs], nblk[kDirs];
    size_t lds;
};
WgPlan wg_plan(const Geom &g)
{
    WgPlan w{};
    const int KK = g.KP * g.KQ, U = g.O / 16;
    // taps of an item: at most five of 3 x 3 filters (4 NT accumulator tiles; all nine
    // with the operands need more than the 256 registers of two waves per SIMD),
    // seven of larger ones, whose workgroups stage no second 64 pixels
    w.TG = KK == 9 ? 2 : KK == 25 ? 4 : KK == 49 ? 7 : 1;
    w.NT = KK == 9 ? 5 : KK < 9 ? KK : 7;
    w.CT = U + (g.C + 15) / 16;
    w.NTt = KK * U + (KK * g.C + 16) / 16;
    // column tiles of a part: the fullest use of eight waves, then the larger part
    double best = 0.0;
    for (int pc = 1; pc <= 4 && pc * w.TG <= kWaves; pc *= 2) {
        const int ks0 = kWaves / (pc * w.TG), ks = ks0 >= 4 ? 4 : ks0 >= 2 ? 2 : 1;
        const int parts = (w.CT + pc - 1) / pc;
        const double use = (double)w.CT * w.TG * ks / (parts * kWaves);
        if (use >= best) {
            best = use;
            w.PC = pc;
            w.nct = parts;
            w.KS = ks;
        }
    }
    w.TP = w.KS == 4 ? 128 : 64;
    w.rowB = w.PC * 64 + 32;
    const DevInfo di = device_info();
    const int lim = di.max_lds > 0 ? di.max_lds : 65536;
    int max_px = ((lim - kStatic) / 2 - w.TP * kRowA) / w.rowB;
    if (max_px > kXB * kThreads / (2 * w.PC)) max_px = kXB * kThreads / (2 * w.PC);
    int staged = 0;
    for (int d = 0; d < g.nd; ++d) {
        // blocks of at most TP pixels whose halo fits: fewest blocks, then pixels staged
        const DirGeom &dg = g.dir[d];
        double bc = 1e300;
        int bst = 0;
        for (int bq0 = 1; bq0 <= w.TP && bq0 <= dg.Q; ++bq0) {
            const int nbq = (dg.Q + bq0 - 1) / bq0, bq = (dg.Q + nbq - 1) / nbq;
            if (bq != bq0) continue;
            int h0 = w.TP / bq < dg.P ? w.TP / bq : dg.P;
            while (h0 > 1 && (h0 + g.KP - 1) * (bq + g.KQ - 1) > max_px) --h0;
            const int nbp = (dg.P + h0 - 1) / h0, bp = (dg.P + nbp - 1) / nbp;
            const int st = (bp + g.KP - 1) * (bq + g.KQ - 1);
            if (st > max_px) continue;
            const double c = (double)nbp * nbq * (w.TP + 0.25 * st);
            if (c < bc * (1 - 1e-9)) {
                bc = c;
                bst = st;
                w.bp[d] = bp; w.bq[d] = bq; w.nbq[d] = nbq; w.nblk[d] = nbp * nbq;
            }
        }
        if (bst > staged) staged = bst;
    }
    w.bufb = (w.TP * kRowA + staged * w.rowB + 15) / 16 * 16;
    w.lds = 2 * (size_t)w.bufb;
    const size_t xch = (size_t)kWaves * w.NT * 1024;
    if (w.lds < xch) w.lds = xch;
    if (w.lds < kThreads * 32) w.lds = kThreads * 32;
    const int cus = di.cus > 0 ? di.cus : 256, per = g.nd * U * w.nct;
    w.kch = cus / per > 1 ? cus / per : 1;
    return w;
}

template <int NT>
int launch_nt(const WgPlan &w, const WgH2Args &a, int grid, hipStream_t st)
{
    const void *fn = w.TP == 128 ? (const void *)k_wgrad_h2<NT, 2> : (const void *)k_wgrad_h2<NT, 1>;
    if (hipFuncSetAttribute(fn, hipFuncAttributeMaxDynamicSharedMemorySize, (int)w.lds) != hipSuccess)
        return PLSTM_EHIP;
    if (w.TP == 128)
        k_wgrad_h2<NT, 2><<<grid, kThreads, w.lds, st>>>(a);
    else
        k_wgrad_h2<NT, 1><<<grid, kThreads, w.lds, st>>>(a);
    PLSTM_LAUNCH_CHECK();
    return PLSTM_OK;
}

struct WgWs {
    float *xp;
    SplitStats *part;
    unsigned *ctl;
};
WgWs carve_wg(Carve &cv, const Geom &g, bool room)
{
    WgWs w;
    w.xp = pad8(g.C) != g.C && !room ? cv.take<float>((size_t)g.N * g.V * pad8(g.C)) : nullptr;
    w.part = cv.take<SplitStats>(1);
    w.ctl = cv.take<unsigned>(1);
    return w;
}

}  // namespace

WgradSplit split_wgrad_shape(const Geom &g)
{
    const WgPlan w = wg_plan(g);
    return {w.kch, (size_t)g.nd * w.kch * 4 * g.O * w.NTt * 16};
}

size_t split_wgrad_ws(const Geom &g, bool room)
{
    Carve cv(nullptr);
    carve_wg(cv, g, room);
    return cv.off;
}

int split_wgrad(const Geom &g, const float *x, const float *hd, const float *dA,
                float *partial, float *room, void *ws, const unsigned **ctl,
                hipStream_t st)
{
    Carve cv(ws);
    WgWs s = carve_wg(cv, g, room != nullptr);
    if (pad8(g.C) != g.C && room) s.xp = room;
    const WgPlan w = wg_plan(g);
    const long long nvox = (long long)g.N * g.V;
    int rc = split_stats(x, nvox * g.C, s.part, s.ctl, st);
    if (rc != PLSTM_OK) return rc;
    if (s.xp) {
        rc = split_pad_x(nvox, g.C, x, s.xp, st);
        if (rc != PLSTM_OK) return rc;
    }
    *ctl = s.ctl;
    WgH2Args a;
    a.g = g;
    a.C8 = pad8(g.C);
    a.CT = w.CT; a.PC = w.PC; a.TG = w.TG; a.nct = w.nct;
    a.kch = w.kch; a.NTt = w.NTt;
    a.x = s.xp ? s.xp : x; a.hd = hd; a.dA = dA;
    a.part = s.part; a.ctl = s.ctl;
    a.partial = partial;
    a.rowB = w.rowB; a.bufb = w.bufb;
    for (int d = 0; d < kDirs; ++d) {
        a.bp[d] = w.bp[d]; a.bq[d] = w.bq[d]; a.nbq[d] = w.nbq[d]; a.nblk[d] = w.nblk[d];
    }
    const int grid = g.nd * (g.O / 16) * w.nct * w.kch;
    switch (w.NT) {
    case 1: return launch_nt<1>(w, a, grid, st);
    case 3: return launch_nt<3>(w, a, grid, st);
    case 5: return launch_nt<5>(w, a, grid, st);
    case 7: return launch_nt<7>(w, a, grid, st);
    default: return PLSTM_EUNSUPPORTED;
    }
}

}  // namespace plstm
