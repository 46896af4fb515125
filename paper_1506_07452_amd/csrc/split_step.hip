// Plane steps of fp32 layers on the 16-bit matrix unit (split.h), O = 16, 32
// or 64 units, up to 64 input channels, any K x K filter: the same launches
// (one per plane step, all directions) and the same mathematics as the fp32
// plane steps, with every contraction on v_mfma_f32_16x16x32_f16.
//
// K layout.  The contraction runs over slots of eight channels: slot
// s < NSX is input tap s / CS, channels 8 (s % CS) .. + 7 (CS = C8 / 8, C
// zero-padded to C8 = a multiple of 8); the rest are h taps, O / 8 slots
// each.  A K-group is four consecutive slots, one per lane group q of the
// instruction (lane l supplies A[m = l%16][k = 8 (l/16) + j] and
// B[k][n = l%16], j = 0..7), whatever taps they belong to, so no filter and
// no channel count pads a tap to 32 channels.
#include "split.h"
#include "strip_plan.h"
#include "sweep.h"
#include "timing.h"

namespace plstm {
namespace {

typedef v4 f4;

constexpr int kXcds = 8;                 // XCDs: workgroup b runs on XCD b % 8
constexpr int kRsrcWord3 = 0x00020000;   // raw buffer, 32-bit data
constexpr int kWaitAllLds = 0x0070;      // s_waitcnt vmcnt(0) lgkmcnt(0)

typedef __attribute__((address_space(3))) void lds_void;

__device__ inline float frcp(float v) { return __builtin_amdgcn_rcpf(v); }
__device__ inline float fsig(float a) { return frcp(1.0f + __expf(-a)); }
__device__ inline float ftanh(float a) { return 1.0f - 2.0f * frcp(__expf(2.0f * a) + 1.0f); }

__device__ inline __amdgpu_buffer_rsrc_t rsrc_of(const void *p, long long bytes)
{
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<void *>(p), (short)0, (int)bytes,
                                             kRsrcWord3);
}
__device__ inline int item_dir(const int *base, int item)
{
    int d = 0;
#pragma unroll
    for (int k = 1; k < kDirs; ++k) d += item >= base[k] ? 1 : 0;
    return d;
}
__device__ inline bool on_plane(int p, int q, int P, int Q)
{
    return ((unsigned)p < (unsigned)P) & ((unsigned)q < (unsigned)Q);
}

// ---- statistics and packing -------------------------------------------------

// One workgroup's share (of kStatBlocks) of a tensor's statistics: the largest
// magnitude, or with COUNT the non-zero values and those below `low`.  Thread 0
// returns it.
template <typename TS, bool COUNT>
__device__ SplitStat scan_values(long long n, const TS *__restrict__ x, unsigned low, SplitStat *red)
{
    SplitStat s = {0u, 0u, 0u, 0u};
    auto add = [&](float v) {
        const unsigned m = __float_as_uint(v) & 0x7fffffffu;
        if constexpr (COUNT) {
            s.nonzero += m != 0 ? 1u : 0u;
            s.small += m != 0 && m < low ? 1u : 0u;
        } else {
            const bool fin = m < 0x7f800000u;
            s.max_bits = fin && m > s.max_bits ? m : s.max_bits;
            s.bad |= fin ? 0u : 1u;
        }
    };
    const long long stride = (long long)kStatBlocks * 256;
    const long long id = (long long)blockIdx.x * 256 + threadIdx.x;
    if constexpr (sizeof(TS) == 4) {
        const long long n4 = n / 4;
        const f4 *x4 = (const f4 *)x;
        for (long long i = id; i < n4; i += 4 * stride) {
            f4 v[4];
#pragma unroll
            for (int u = 0; u < 4; ++u) v[u] = x4[i + u * stride < n4 ? i + u * stride : i];
#pragma unroll
            for (int u = 0; u < 4; ++u)
#pragma unroll
                for (int k = 0; k < 4; ++k) add(i + u * stride < n4 ? v[u][k] : 0.0f);
        }
        for (long long i = n4 * 4 + id; i < n; i += stride) add(Store<TS>::load(x, i));
    } else {
        for (long long i = id; i < n; i += stride) add(Store<TS>::load(x, i));
    }
    s = stat_wave(s);
    if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = s;
    __syncthreads();
    return stat_combine(stat_combine(red[0], red[1]), stat_combine(red[2], red[3]));
}
template <bool COUNT>
__global__ void __launch_bounds__(256)
k_split_stats(long long n, const float *__restrict__ x, SplitStats *__restrict__ part,
              unsigned *__restrict__ ctl)
{
    __shared__ SplitStat red[5];
    unsigned low = 0;                       // magnitudes below this are small
    if constexpr (COUNT) {
        const unsigned m = stat_reduce(part->first, &red[4]).max_bits;
        low = m > kStatRange ? m - kStatRange : 0u;
    }
    const SplitStat s = scan_values<float, COUNT>(n, x, low, red);
    if (!COUNT && blockIdx.x == 0 && threadIdx.x == 0) *ctl = 0u;
    if (threadIdx.x == 0) (COUNT ? part->second : part->first)[blockIdx.x] = s;
}
// x's statistics (the first kStatBlocks workgroups) and the weights' row maxima, a row a
// wave.
template <typename TS>
__global__ void __launch_bounds__(256)
k_split_scan(long long n, int nx, int nh, const TS *__restrict__ x, const TS *__restrict__ wx,
             const TS *__restrict__ wh, SplitScan *__restrict__ scan, int *__restrict__ clear, int nclear)
{
    for (int i = blockIdx.x * 256 + threadIdx.x; i < nclear; i += gridDim.x * 256) clear[i] = 0;
    if (blockIdx.x < kStatBlocks) {
        __shared__ SplitStat red[4];
        const SplitStat s = scan_values<TS, false>(n, x, 0u, red);
        if (threadIdx.x == 0) scan->x[blockIdx.x] = s;
        return;
    }
    const int l = threadIdx.x & 63;
    const long long row = (long long)(blockIdx.x - kStatBlocks) * 4 + (threadIdx.x >> 6);
    auto row_max = [&](const TS *w, int cnt) {
        unsigned m = 0;
#pragma unroll 4
        for (int i = l; i < cnt; i += 64) {
            const unsigned v = __float_as_uint(Store<TS>::load(w, row * cnt + i)) & 0x7fffffffu;
            m = v > m ? v : m;
        }
#pragma unroll
        for (int o = 32; o > 0; o >>= 1) {
            const unsigned t = __shfl_xor(m, o);
            m = t > m ? t : m;
        }
        return m;
    };
    const unsigned mx = row_max(wx, nx), mh = row_max(wh, nh);
    if (l == 0) {
        scan->row[row][0] = mx;
        scan->row[row][1] = mh;
    }
}

// x [N][V][C] -> fp32 [N][V][C8], channels >= C zero.
template <typename TS>
__global__ void __launch_bounds__(256)
k_pad_x8(long long nvox, int C, int C8, const TS *__restrict__ x, float *__restrict__ xp)
{
    const long long i = (long long)blockIdx.x * 256 + threadIdx.x;
    if (i >= nvox * C8) return;
    const long long v = i / C8;
    const int c = (int)(i - v * C8);
    xp[i] = c < C ? Store<TS>::load(x, v * C + c) : 0.0f;
}

struct PackArgs {
    int O, C, CS, KK, NSX, NS, KG, rows;
    const SplitScan *scan;
    unsigned *ctl;            // [0] 1: fp32 channels instead of split pairs, [1] scale of x (bits)
    h8 *frag;                 // [nd][U][KG][4 gates][2][64]
    float *bias, *rinv;       // [nd][4O]: bias, 1 / scale of each gate row's sums
};

// One workgroup per (direction, unit group, gate): the 16 rows' scales (row_scale) and
// fragments.
constexpr int kPackThreads = 512;
template <typename TS>
__global__ void __launch_bounds__(kPackThreads)
k_pack_fwd_h2(PackArgs a, const TS *__restrict__ wx, const TS *__restrict__ wh,
              const TS *__restrict__ b)
{
    __shared__ SplitStat red;
    __shared__ float fx[16], fh[16];
    const int O = a.O, U = O / 16, C = a.C, KK = a.KK;
    const int gate = blockIdx.x & 3, ug = (blockIdx.x >> 2) % U, d = (blockIdx.x >> 2) / U;
    const int tid = threadIdx.x;
    const CallScale cs = call_scale(a.scan, a.rows, &red);
    const bool split = cs.split;
    const int ex = cs.ex;
    const long long gu0 = (long long)d * 4 * O + gate * O + ug * 16;
    if (tid < 16) {
        const unsigned *const m = a.scan->row[gu0 + tid];
        const int s = row_scale(ex, m[0], m[1]).s;
        fx[tid] = !split ? 1.0f : m[0] ? ldexpf(1.0f, s - ex) : 0.0f;   // (2^(s - ex) may overflow)
        fh[tid] = split ? ldexpf(1.0f, s - 15) : 1.0f;
        a.rinv[gu0 + tid] = split ? ldexpf(1.0f, -s) : 1.0f;
        a.bias[gu0 + tid] = Store<TS>::load(b, gu0 + tid);
    }
    if (blockIdx.x == 0 && tid == 0) {
        a.ctl[0] = split ? 0u : 1u;
        a.ctl[1] = __float_as_uint(split ? exp2i(ex) : 1.0f);
    }
    __syncthreads();
    const int HS = O / 8;
    for (int e = tid; e < a.KG * 64; e += kPackThreads) {
        const int lane = e & 63, kg = e >> 6, q = lane >> 4, col = lane & 15;
        const int slot = 4 * kg + q;
        const long long gu = gu0 + col;
        f4 w[2];
#pragma unroll
        for (int j = 0; j < 8; ++j) {
            float v = 0.0f;
            if (slot < a.NSX) {
                const int tap = slot / a.CS, c = (slot - tap * a.CS) * 8 + j;
                if (c < C) v = Store<TS>::load(wx, (gu * C + c) * KK + tap) * fx[col];
            } else if (slot < a.NS) {
                const int sh = slot - a.NSX, tap = sh / HS, u = (sh - tap * HS) * 8 + j;
                v = Store<TS>::load(wh, (gu * O + u) * KK + tap) * fh[col];
            }
            w[j >> 2][j & 3] = v;
        }
        h8 *out = a.frag + ((((long long)d * U + ug) * a.KG + kg) * 4 + gate) * 128 + lane;
        if (split) {
            const Split8 sp = split8(w[0], w[1]);
            out[0] = sp.hi;
            out[64] = sp.lo;
        } else {
            out[0] = __builtin_bit_cast(h8, w[0]);
            out[64] = __builtin_bit_cast(h8, w[1]);
        }
    }
}

// ---- forward step -----------------------------------------------------------

struct FwdH2Args {
    Geom g;
    int t;
    int C8, CS, NSX, NS, KG, KGX;   // slots and K-groups (KGX: those with input slots)
    int NUB;                        // workgroups per pixel block: U / UB
    int nchp;                       // 16-byte chunks per staged pixel
    int tab_off;                    // chunks of the staged block: the slot table follows
    int k_mul;                      // ceil(2^16 / KQ)
    const float *x;                 // [N][V][C8]
    const h8 *frag;
    const float *bias, *rinv;
    const unsigned *ctl;
    float *hd;                      // [nd][N][V][O]
    float *cell;                    // [nd][N][V][O] (training) or null:
    float *cpp;                     // c^d of the last two planes, [N][min(T,2)][P Q][O] at coff
    float *gates;                   // [nd][N][V][4O] or null
    long long coff[kDirs];
    int bp[kDirs], bq[kDirs], nbq[kDirs], nblk[kDirs];
    int base[kDirs + 1];
};

// Workgroup: 4 UB waves take a BP x BQ block of at most 64 NT pixels of one
// plane and the gates of UB unit groups; wave (wm, wn) computes unit group
// wm of them (four 16-row gate tiles) for NT 16-pixel tiles.
// - [x_t | h_{t-1}] of the block and its filter halo is staged once as split
//   pairs (fp32 loads, split in registers); a staged pixel has 2 mod 4 chunks
//   of 16 bytes, a stride of 8 mod 16 floats, on which 64 lanes reading 16
//   bytes each run without bank conflicts.
//   The loads are branch-free and wait together: with a branch per source the
//   compiler waited for each in turn (staging 12 -> 8 kilocycles).
// - The A fragments of a K-group (UB x 8 KB) stream through three LDS arrays
//   with direct-to-LDS loads two K-groups ahead; step kg reads K-group kg + 1
//   into registers beside kg's products and refills the array that held kg.
//   Its barrier publishes kg + 2 (each wave has waited for its own share) and
//   frees kg + 1's array.  The arrays are distinct objects named statically
//   (the loop is unrolled by six), so no wait for a load in flight is inserted
//   before a read.
// Bound by each launch's latency on small planes (staging 8, cell update 2.5 of
// 15-28 kilocycles) and by LDS reads and barriers on large ones (a K-group takes
// 1.0 kilocycles for 0.77 of products).  Measured against the fp32 instruction on
// 64-pixel blocks: 32 -> 32 units on 48 x 240 x 240, training, 24.1 -> 11.0 ms (223
// TFLOP/s of fp32 products); 64 -> 64 on 20 x 64 x 64 6.0 -> 1.8; 7 x 7, 25 -> 32 on
// 15 x 128 x 128 18.2 -> 5.5; 6 -> 16 on 19 x 101 x 75 1.35 -> 0.84.  Not kept: a ring
// of two arrays with operands read in the step that uses them (8.0 against 7.4 ms
// on 25 x 240 x 240, 32 -> 32); 256-pixel blocks (8.5).
template <int UB, int NT>
__global__ void __launch_bounds__(256 * UB)
k_step_fwd_h2(FwdH2Args a)
{
    constexpr int NW = 4 * UB, THREADS = 64 * NW, AT = 4 * 2 * UB;   // 1 KB fragments per K-group
    constexpr int NDMA = AT / NW;                                     // 2
    constexpr int kWaitRingLds = 0x0070 | NDMA;
    __shared__ h8 ring0[AT * 64], ring1[AT * 64], ring2[AT * 64];
    extern __shared__ h8 stg[];
    const int tid = threadIdx.x, lane = tid & 63, q4 = lane >> 4, col = lane & 15;
    const int wv = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wm = wv % UB, wn = wv / UB;
    const int per_xcd = gridDim.x / kXcds;
    const int blk = (blockIdx.x % kXcds) * per_xcd + blockIdx.x / kXcds;
    if (blk >= a.base[kDirs]) return;
    const int d = item_dir(a.base, blk);
    const DirGeom dg = a.g.dir[d];
    int r = blk - a.base[d];
    const int n = r / (a.nblk[d] * a.NUB);
    r -= n * a.nblk[d] * a.NUB;
    const int ub = r / a.nblk[d];
    r -= ub * a.nblk[d];
    const int BP = a.bp[d], BQ = a.bq[d];
    const int bi = r / a.nbq[d], bj = r - bi * a.nbq[d];
    const int p0 = bi * BP, q0 = bj * BQ;
    const int t = a.t, O = a.g.O, G = 4 * O, U = O >> 4;
    const int s = dg.sign > 0 ? t : dg.T - 1 - t;
    const int ss = (int)dg.ss, sp = (int)dg.sp, sq = (int)dg.sq;
    const int P = dg.P, Q = dg.Q;
    const long long V = a.g.V;
    const int C8 = a.C8, CS = a.CS, NSP = CS + (O >> 3), nchp = a.nchp;
    const int hoff = -dg.sign * ss;
    const int KQ = a.g.KQ, radp = a.g.KP >> 1, radq = KQ >> 1;
    const int SW = BQ + 2 * radq, SH = BP + 2 * radp;
    const long long sbase = ((long long)d * a.g.N + n) * V;
    const bool f32 = a.ctl[0] != 0;
    const float xs = __uint_as_float(a.ctl[1]);
    int *const tab = (int *)(stg + a.tab_off);
    float *const rowp = (float *)(tab + 4 * a.KG + 4);   // bias, then 1 / scale, of the block's rows
    const int ug0 = ub * UB, ug = ug0 + wm;
    const int uo = ug * 16 + 4 * q4;
    const float *const x_n = a.x + (long long)n * V * C8, *const h_n = a.hd + sbase * O;
    const auto rs_a = rsrc_of(a.frag + (long long)d * U * a.KG * 512, (long long)U * a.KG * 8192);

    auto issue_a = [&](int kg, h8 *slot) {
#pragma unroll
        for (int j0 = 0; j0 < AT; j0 += NW) {
            const int j = j0 + wv;
            __builtin_amdgcn_raw_ptr_buffer_load_lds(
                rs_a, (lds_void *)&slot[j * 64], 16,
                (int)((unsigned)(((ug0 + (j >> 3)) * a.KG + kg) * 512 + (j & 7) * 64 + lane) * 16u),
                0, 0, 0);
        }
    };

    // chunk offset of each slot from a pixel's first chunk (slots past the
    // last, whose weights are zero, read the pixel's own h, which is finite
    // where x may not be)
    auto slot_table = [&]() {
        for (int e = tid; e < 4 * a.KG + 4; e += THREADS) {
            const bool is_x = e < a.NSX;
            const int sl = is_x ? e : e - a.NSX, per = is_x ? CS : O >> 3;
            const int tap = fdiv_floor(sl, 1.0f / (float)per), c = sl - tap * per;
            const int ka = ((tap * a.k_mul) >> 16) - radp, kb = tap - (ka + radp) * KQ - radq;
            tab[e] = e < a.NS ? (ka * SW + kb) * nchp + 2 * (c + (is_x ? 0 : CS)) : 2 * CS;
        }
    };

    const int KG = t > 0 ? a.KG : a.KGX;
    issue_a(0, ring0);
    if (KG > 1) issue_a(1, ring1);
    if (KG > 2) issue_a(2, ring2);

    // this lane's pixel of each tile: first chunk in the staged block
    int spb[NT], evox[NT], epix[NT];
    bool elive[NT];
#pragma unroll
    for (int nt = 0; nt < NT; ++nt) {
        const int e = (wn * NT + nt) * 16 + col;
        const int ey = fdiv_floor(e, 1.0f / (float)BQ), ex = e - ey * BQ;
        const bool in = ey < BP;
        elive[nt] = in && on_plane(p0 + ey, q0 + ex, P, Q);
        spb[nt] = in ? ((ey + radp) * SW + ex + radq) * nchp : (radp * SW + radq) * nchp;
        epix[nt] = elive[nt] ? (p0 + ey) * Q + q0 + ex : 0;
        evox[nt] = s * ss + (elive[nt] ? (p0 + ey) * sp + (q0 + ex) * sq : 0);
    }

    // c_{t-1}, in flight beside the staging loads (any value where t = 0)
    const int PQ = P * Q;
    const float *cin;
    float *cout;
    if (a.cell) {
        cout = a.cell + sbase * O;
        cin = cout + (long long)hoff * O;
    } else {
        const int np = dg.T > 1 ? 2 : 1;
        float *c0 = a.cpp + a.coff[d] + (long long)n * np * PQ * O;
        cout = c0 + (long long)(t & 1) * PQ * O;
        cin = c0 + (long long)((t + 1) & 1) * PQ * O;
    }
    f4 cprev[NT];
#pragma unroll
    for (int nt = 0; nt < NT; ++nt) {
        const bool ok = t > 0 && elive[nt];
        cprev[nt] = *(const f4 *)((ok ? cin + (a.cell ? evox[nt] : epix[nt]) * O : cout) + uo);
    }

    // ---- stage [x_t | h_{t-1}] (zero off the plane and before the first one)
    {
        const int nst = SH * SW * NSP;
        const float inv_nsp = 1.0f / (float)NSP, inv_sw = 1.0f / (float)SW;
        constexpr int SB = 3;
        for (int e0 = tid; e0 - tid < nst; e0 += SB * THREADS) {
            // branch-free: lanes without a source read the first voxel of x
            // and take zero, so every load of the batch is in flight at once
            f4 va[SB], vb[SB];
            int dst[SB];
            float sc[SB];
            bool ok[SB];
#pragma unroll
            for (int u = 0; u < SB; ++u) {
                const int e = e0 + u * THREADS;
                const int spx = fdiv_floor(e, inv_nsp), c = e - spx * NSP;
                const int sy = fdiv_floor(spx, inv_sw), sx = spx - sy * SW;
                const int pp = p0 - radp + sy, qq = q0 - radq + sx;
                const int v = s * ss + pp * sp + qq * sq;
                const bool is_x = c < CS;
                dst[u] = e < nst ? spx * nchp + 2 * c : -1;
                sc[u] = is_x ? xs : kHScale;
                ok[u] = e < nst && on_plane(pp, qq, P, Q) && (is_x || t > 0);
                const float *src = is_x ? x_n : h_n;
                const int off = is_x ? v * C8 + 8 * c : (v + hoff) * O + 8 * (c - CS);
                src = ok[u] ? src + off : x_n;
                va[u] = *(const f4 *)src;
                vb[u] = *(const f4 *)(src + 4);
            }
            if (e0 == tid) {                       // beside the first batch's loads
                slot_table();
                for (int e = tid; e < UB * 128; e += THREADS) {
                    const int k = e & (UB * 64 - 1);       // unit group, gate, unit
                    const int row = d * G + ((k >> 4) & 3) * O + (ug0 + (k >> 6)) * 16 + (k & 15);
                    rowp[e] = e < UB * 64 ? a.bias[row] : a.rinv[row];
                }
            }
#pragma unroll
            for (int u = 0; u < SB; ++u) {
                if (dst[u] < 0) continue;
                const f4 zero = {0.0f, 0.0f, 0.0f, 0.0f};
                va[u] = ok[u] ? va[u] : zero;
                vb[u] = ok[u] ? vb[u] : zero;
                if (f32) {
                    stg[dst[u]] = __builtin_bit_cast(h8, va[u]);
                    stg[dst[u] + 1] = __builtin_bit_cast(h8, vb[u]);
                } else {
                    const Split8 w = split8(va[u] * sc[u], vb[u] * sc[u]);
                    stg[dst[u]] = w.hi;
                    stg[dst[u] + 1] = w.lo;
                }
            }
        }
    }
    struct Ops {
        h8 a[4][2];
        h8 b[NT][2];
    };
    f4 sum[2][4][NT];                // lo hi' + hi lo', hi hi'
    f4(&acc)[4][NT] = sum[1];
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int nt = 0; nt < NT; ++nt) sum[0][i][nt] = sum[1][i][nt] = f4{0.0f, 0.0f, 0.0f, 0.0f};

    __builtin_amdgcn_s_waitcnt(kWaitAllLds);
    __syncthreads();
    if (!f32) {
        Ops X, Y;
        int bo = tab[q4], bn = tab[4 + q4];    // slot offsets of K-groups kg, kg + 1
#pragma unroll
        for (int i = 0; i < 8; ++i) X.a[i >> 1][i & 1] = ring0[(wm * 8 + i) * 64 + lane];
#pragma unroll
        for (int i = 0; i < 2 * NT; ++i) X.b[i >> 1][i & 1] = stg[spb[i >> 1] + bo + (i & 1)];
        // products of `cur` (K-group kg) beside the reads of kg + 1 from `rd`
        auto step = [&](int kg, const Ops &cur, Ops &nxt, const h8 *rd, h8 *dm) {
            const bool more = kg + 3 < KG;
            const int bt = tab[min(4 * (kg + 2), 4 * a.KG) + q4];
#pragma unroll
            for (int p = 0; p < 3; ++p)
#pragma unroll
                for (int i = 0; i < 4; ++i) {
#pragma unroll
                    for (int nt = 0; nt < NT; ++nt)
                        sum[p == 2][i][nt] = mfma_h(cur.a[i][p == 0 ? 1 : 0],
                                                    cur.b[nt][p == 1 ? 1 : 0], sum[p == 2][i][nt]);
                    const int k = p * 4 + i;
                    if (k < 8) nxt.a[k >> 1][k & 1] = rd[(wm * 8 + k) * 64 + lane];
                    if (k < 2 * NT) nxt.b[k >> 1][k & 1] = stg[spb[k >> 1] + bn + (k & 1)];
                    if (k == 5 && more) issue_a(kg + 3, dm);
                    __builtin_amdgcn_sched_barrier(0);
                }
            bn = bt;
            if (more)
                __builtin_amdgcn_s_waitcnt(kWaitRingLds);
            else
                __builtin_amdgcn_s_waitcnt(kWaitAllLds);
            asm volatile("" ::: "memory");
            __builtin_amdgcn_s_barrier();
            asm volatile("" ::: "memory");
        };
        // step 0 refills ring0: every wave has read K-group 0 from it first
        __syncthreads();
        for (int kg = 0; kg + 1 < KG; kg += 6) {
            step(kg, X, Y, ring1, ring0);
            if (kg + 2 < KG) step(kg + 1, Y, X, ring2, ring1);
            if (kg + 3 < KG) step(kg + 2, X, Y, ring0, ring2);
            if (kg + 4 < KG) step(kg + 3, Y, X, ring1, ring0);
            if (kg + 5 < KG) step(kg + 4, X, Y, ring2, ring1);
            if (kg + 6 < KG) step(kg + 5, Y, X, ring0, ring2);
        }
        if ((KG - 1) & 1) X = Y;
#pragma unroll
        for (int p = 0; p < 3; ++p)
#pragma unroll
            for (int i = 0; i < 4; ++i)
#pragma unroll
                for (int nt = 0; nt < NT; ++nt)
                    sum[p == 2][i][nt] = mfma_h(X.a[i][p == 0 ? 1 : 0], X.b[nt][p == 1 ? 1 : 0],
                                                sum[p == 2][i][nt]);
#pragma unroll
        for (int i = 0; i < 4; ++i)
#pragma unroll
            for (int nt = 0; nt < NT; ++nt) sum[1][i][nt] = join(sum[1][i][nt], sum[0][i][nt]);
    } else {
        // fp32 channels: K-group kg is eight k-steps of the fp32 instruction,
        // lane group q supplying channel j of its slot
        auto products = [&](int kg, auto masked) {
            const int bo = tab[4 * kg + q4];
            // (h slots of the last group with input slots at t = 0: no product with an
            // infinite weight where there is no h)
            const bool real = !decltype(masked)::value || 4 * kg + q4 < a.NSX;
#pragma unroll
            for (int hl = 0; hl < 2; ++hl)
#pragma unroll
                for (int nt = 0; nt < NT; ++nt) {
                    const f4 bv = __builtin_bit_cast(f4, stg[spb[nt] + bo + hl]);
#pragma unroll
                    for (int i = 0; i < 4; ++i) {
                        f4 av = __builtin_bit_cast(f4, ring0[(wm * 8 + 2 * i + hl) * 64 + lane]);
                        if (!real) av = f4{0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
                        for (int j = 0; j < 4; ++j)
                            acc[i][nt] = __builtin_amdgcn_mfma_f32_16x16x4f32(av[j], bv[j],
                                                                              acc[i][nt], 0, 0, 0);
                    }
                }
        };
        for (int kg = 0; kg < KG; ++kg) {
            __syncthreads();
            issue_a(kg, ring0);
            __builtin_amdgcn_s_waitcnt(kWaitAllLds);
            __syncthreads();
            if (t == 0 && kg == KG - 1)
                products(kg, std::true_type{});
            else
                products(kg, std::false_type{});
        }
    }

    // ---- Eq. (7)-(12) of units uo .. uo + 3
    f4 bias[4], rinv[4];
#pragma unroll
    for (int gt = 0; gt < 4; ++gt) {
        bias[gt] = *(const f4 *)(rowp + wm * 64 + gt * 16 + 4 * q4);
        rinv[gt] = *(const f4 *)(rowp + (UB + wm) * 64 + gt * 16 + 4 * q4);
    }
#pragma unroll
    for (int nt = 0; nt < NT; ++nt) {
        if (!elive[nt]) continue;
        const long long vo = sbase + evox[nt];
        f4 gi, gf, gg, go, c, h;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            gi[i] = fsig(__builtin_fmaf(acc[0][nt][i], rinv[0][i], bias[0][i]));
            gf[i] = fsig(__builtin_fmaf(acc[1][nt][i], rinv[1][i], bias[1][i]));
            gg[i] = ftanh(__builtin_fmaf(acc[2][nt][i], rinv[2][i], bias[2][i]));
            go[i] = fsig(__builtin_fmaf(acc[3][nt][i], rinv[3][i], bias[3][i]));
            c[i] = gg[i] * gi[i] + (t > 0 ? cprev[nt][i] : 0.0f) * gf[i];
            h[i] = go[i] * ftanh(c[i]);
        }
        *(f4 *)(cout + (long long)(a.cell ? evox[nt] : epix[nt]) * O + uo) = c;
        *(f4 *)(a.hd + vo * O + uo) = h;
        if (a.gates) {
            float *gp = a.gates + vo * G + uo;
            *(f4 *)gp = gi;
            *(f4 *)(gp + O) = gf;
            *(f4 *)(gp + 2 * O) = gg;
            *(f4 *)(gp + 3 * O) = go;
        }
    }
}

// ---- reverse step -----------------------------------------------------------

// A fragments frag[d][kg][rt][2][64]: row tile rt < U holds units 16 rt .. + 15
// of W_h^T, the rest channels 16 (rt - U) .. + 15 of W_x^T (0 past C).  K-groups run
// over passes of 64 gate-units, then taps, then halves: kg = (pass KK + tap) 2 +
// half, lane group q taking gate-units 64 pass + 32 half + 8 q .. + 7.
// One workgroup per (direction, row tile): the 16 rows' largest magnitudes and
// their scale, then the fragments.  Rows that one scale does not serve leave fp32
// values instead (raw[d][rt] = 1).
struct PackBwdArgs {
    int O, C, KK, RT, rt0, nrt;   // packs row tiles rt0 .. rt0 + nrt - 1
    const float *wx, *wh;
    h8 *frag;
    float *rinv;              // [nd][16 RT]: 1 / scale of each row
    unsigned *raw;            // [nd][RT]
};
constexpr int kPackBwdThreads = 1024;
__global__ void __launch_bounds__(kPackBwdThreads)
k_pack_bwd_h2(PackBwdArgs a)
{
    __shared__ unsigned mx[16], mn[16], nonzero[16], small[16];
    __shared__ float fr[16];
    const int O = a.O, U = O / 16, G = 4 * O, KK = a.KK, C = a.C, tid = threadIdx.x;
    const int rt = a.rt0 + blockIdx.x % a.nrt, d = blockIdx.x / a.nrt;
    const bool is_h = rt < U;
    const float *w = (is_h ? a.wh : a.wx) + (long long)d * G * (is_h ? O : C) * KK;
    const int cols = is_h ? O : C, r0 = (is_h ? rt : rt - U) * 16;
    if (tid < 16) {
        mx[tid] = nonzero[tid] = small[tid] = 0u;
        mn[tid] = ~0u;
    }
    __syncthreads();
    constexpr int TR = kPackBwdThreads / 16;
    const int row = tid / TR;
    auto each = [&](auto use) {              // magnitudes of this thread's share of its row
        if (r0 + row < cols)
            for (int i = tid % TR; i < G * KK; i += TR) {
                const int g = i / KK, tap = i - g * KK;
                use(__float_as_uint(w[((long long)g * cols + r0 + row) * KK + tap]) & 0x7fffffffu);
            }
    };
    {
        unsigned m0 = 0, m1 = ~0u;
        each([&](unsigned m) {
            m0 = m > m0 ? m : m0;
            m1 = m - 1u < m1 ? m - 1u : m1;      // (zeros apart)
        });
        atomicMax(&mx[row], m0);
        atomicMin(&mn[row], m1);
    }
    __syncthreads();
    const unsigned low = mx[row] > kStatRange ? mx[row] - kStatRange : 0u;
    if (__syncthreads_or(mn[row] != ~0u && mn[row] + 1u < low)) {   // (seldom: counted then only)
        unsigned nz = 0, sm = 0;
        each([&](unsigned m) {
            nz += m != 0 ? 1u : 0u;
            sm += m != 0 && m < low ? 1u : 0u;
        });
        atomicAdd(&nonzero[row], nz);
        atomicAdd(&small[row], sm);
    }
    __syncthreads();
    const int r16 = tid & 15;
    const bool raw = __syncthreads_or(mx[r16] >= 0x7f800000u || small[r16] > nonzero[r16] / 64u) != 0;
    if (tid < 16) {
        const int s = raw ? 0 : scale_exp(mx[tid]);
        fr[tid] = exp2i(s);
        a.rinv[(d * a.RT + rt) * 16 + tid] = exp2i(-s);
    }
    if (tid == 0) a.raw[d * a.RT + rt] = raw ? 1u : 0u;
    __syncthreads();
    const int KG = KK * U * 2;
    for (int e = tid; e < KG * 64; e += kPackBwdThreads) {
        const int lane = e & 63, kg = e >> 6, q = lane >> 4, col = lane & 15;
        const int half = kg & 1, pt = kg >> 1, pass = pt / KK, tap = pt - pass * KK;
        const int g0 = pass * 64 + half * 32 + 8 * q;
        f4 v[2];
#pragma unroll
        for (int j = 0; j < 8; ++j)
            v[j >> 2][j & 3] =
                r0 + col < cols ? w[((long long)(g0 + j) * cols + r0 + col) * KK + tap] * fr[col]
                                : 0.0f;
        const Split8 sp = split8(v[0], v[1]);
        h8 *out = a.frag + (((long long)d * KG + kg) * a.RT + rt) * 128 + lane;
        out[0] = raw ? __builtin_bit_cast(h8, v[0]) : sp.hi;
        out[64] = raw ? __builtin_bit_cast(h8, v[1]) : sp.lo;
    }
}

struct BwdH2Args {
    Geom g;
    int t;                    // plane (-1: dL/dx of plane 0 only)
    int RT, KG;               // row tiles: U of units, then the channels'; K-groups of a pass
    int k_mul;
    int tab_off;
    const h8 *frag;
    const float *rinv;
    const unsigned *raw;
    DaRange *amax;            // range of each plane's waves, [N][T][nblk][waves] at aoff
    long long aoff[kDirs + 1];
    const float *gates, *cell, *dh;
    float *dA;                // [nd][N][V][4O]
    float *gcp;               // dL/dc f of the last two planes, [N][min(T,2)][P Q][O] at coff
    float *dxd;               // [nd][N][V][C] or null
    long long coff[kDirs];
    int bp[kDirs], bq[kDirs], nbp[kDirs], nbq[kDirs], nblk[kDirs];
    int base[kDirs + 1];
};

// 1 KB fragment loads of a K-group: the row tiles' halves, rounded up to a
// whole number per wave.
constexpr int bwd_frags(int RTW, int WM) { return (RTW * WM * 2 + 4 * WM - 1) / (4 * WM) * (4 * WM); }
// staged pixel: 64 gate-units as 8 split slots, 1 / their own scale, pad
constexpr int kBwdChunks = 18, kBwdScale = 16;

// Reverse plane step: dL/dh_t = dL/dh + sum_taps W_h^T dA_{t+1}[p - tap] and, with
// CT channel tiles, dL/dx_{t+1} = sum_taps W_x^T dA_{t+1}[p - tap] of the same
// staged dA_{t+1}; then the gate gradients dA_t.  4 WM waves take at most 64 NT
// pixels; wave (wm, wn) computes row tiles RTW wm .. + RTW - 1 for NT pixel tiles.
// dA_{t+1} of the block and its filter halo is staged 64 gate-units at a time
// (28 KB for 64 pixels, two to three workgroups share a CU), scaled by the
// largest magnitude of the blocks it touches, which the launch before left in
// amax (one range a wave: an atomic maximum per plane cost 0.4 us a launch); the
// fragments stream as in the forward step.  Blocks that one scale does not serve
// (da_wide) give each pixel its own; blocks with a value that is not finite, or
// rows of weights that one scale does not serve, stage dA as it is and take the fp32
// instruction.  Both run in a loop that reads a K-group's operands when it needs them.
// Bound by the launches on small planes (37 us for 400 workgroups: staging twice
// 4, K-groups 0.6 each, 36 of them, cell update 11 kilocycles) and by LDS reads and
// barriers on large ones.  Measured against the fp32 instruction on 64-pixel
// blocks, with dL/dx: 32 -> 32 units on 48 x 240 x 240 27.2 -> 14.3 ms, on 25 x 240 x
// 240 17.4 -> 9.3; 64 -> 64 on 20 x 64 x 64 6.3 -> 2.7 (steps and a dL/dx pass); 7 x 7,
// 25 -> 32 on 15 x 128 x 128 21.0 -> 8.5; 6 -> 16 on 19 x 101 x 75 1.39 -> 1.17.  Not
// kept: 128-pixel blocks (15.7 ms on the first); the cell update's operands loaded
// before the last pass (two instead of three workgroups a CU: 15.9).
// (Registers for the three workgroups that a CU's LDS holds: left alone, the compiler counts
// the rare loop's too and two of <4, 1> fit.  The same for <2, 1>, four, spills: 3 % slower on
// small planes.)
template <int RTW, int WM, int EU>
__global__ void __launch_bounds__(256 * WM, WM == 1 && RTW >= 3 ? 3 : 1)
k_step_bwd_h2(BwdH2Args a)
{
    constexpr int NT = 1;                // pixel tiles of a wave
    constexpr int NW = 4 * WM, THREADS = 64 * NW, AT = bwd_frags(RTW, WM), NDMA = AT / NW;
    constexpr int kWaitRingLds = 0x0070 | NDMA;
    __shared__ h8 ring0[AT * 64], ring1[AT * 64], ring2[AT * 64];
    extern __shared__ h8 stg[];
    const int tid = threadIdx.x, lane = tid & 63, q4 = lane >> 4, col = lane & 15;
    const int wv = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wm = wv % WM, wn = wv / WM;
    const int per_xcd = gridDim.x / kXcds;
    const int blk = (blockIdx.x % kXcds) * per_xcd + blockIdx.x / kXcds;
    if (blk >= a.base[kDirs]) return;
    const int d = item_dir(a.base, blk);
    const DirGeom dg = a.g.dir[d];
    int r = blk - a.base[d];
    const int n = r / a.nblk[d];
    r -= n * a.nblk[d];
    const int BP = a.bp[d], BQ = a.bq[d];
    const int bi = r / a.nbq[d], bj = r - bi * a.nbq[d];
    const int p0 = bi * BP, q0 = bj * BQ;
    const int t = a.t, O = a.g.O, G = 4 * O, U = O >> 4, RT = a.RT;
    const int s = dg.sign > 0 ? t : dg.T - 1 - t;
    const int ss = (int)dg.ss, sp = (int)dg.sp, sq = (int)dg.sq;
    const int P = dg.P, Q = dg.Q, PQ = P * Q;
    const long long V = a.g.V;
    const bool do_h = t >= 0, has_next = t + 1 < dg.T;
    const int noff = dg.sign * ss;       // voxel of plane t + 1 = voxel of plane t + noff
    const int KQ = a.g.KQ, radp = a.g.KP >> 1, radq = KQ >> 1, KK = a.g.KP * KQ;
    const int SW = BQ + 2 * radq, SH = BP + 2 * radp;
    const long long sbase = ((long long)d * a.g.N + n) * V;
    const int KG = a.KG;                 // of one pass
    int *const tab = (int *)(stg + a.tab_off);
    float *const rowp = (float *)(tab + (KK + 3) / 4 * 4);   // 1 / scale of the rows
    DaRange *const am = a.amax + a.aoff[d] + (long long)n * dg.T * a.nblk[d] * NW;

    // this lane's pixel of each tile
    int spb[NT], evox[NT], epix[NT];
    bool elive[NT];
#pragma unroll
    for (int nt = 0; nt < NT; ++nt) {
        const int e = (wn * NT + nt) * 16 + col;
        const int ey = fdiv_floor(e, 1.0f / (float)BQ), ex = e - ey * BQ;
        const bool in = ey < BP;
        elive[nt] = in && on_plane(p0 + ey, q0 + ex, P, Q);
        spb[nt] = (in ? (ey + radp) * SW + ex + radq : radp * SW + radq) * kBwdChunks + 2 * q4;
        epix[nt] = elive[nt] ? (p0 + ey) * Q + q0 + ex : 0;
        evox[nt] = s * ss + (elive[nt] ? (p0 + ey) * sp + (q0 + ex) * sq : 0);
    }
    f4 sum[2][RTW][NT];              // lo hi' + hi lo', hi hi'
    f4(&acc)[RTW][NT] = sum[1];
#pragma unroll
    for (int i = 0; i < RTW; ++i)
#pragma unroll
        for (int nt = 0; nt < NT; ++nt) sum[0][i][nt] = sum[1][i][nt] = f4{0.0f, 0.0f, 0.0f, 0.0f};
    // neighbouring blocks and planes take opposite signs: what the instruction's
    // rounding towards -inf leaves (1e-9 of the mean magnitude) then cancels in the
    // bias gradients, which add it up over all voxels
    const float flip = (bi + bj + t) & 1 ? -1.0f : 1.0f;
    float unscale = 1.0f;
    unsigned raw = 0;                // row tiles with fp32 weights
    bool f32 = false, own = false;   // dA as it is; a scale per pixel
    const f4 zero = {0.0f, 0.0f, 0.0f, 0.0f};

    if (has_next) {
        // range of dA_{t+1} of the blocks the staged one touches: this lane's
        // first wave now, the rest (wide halos) and the reduction beside the
        // staging loads
        const DaRange *const an = am + (long long)(t + 1) * a.nblk[d] * NW;
        const Span si = blocks_touched(bi, BP, a.nbp[d], radp), sj = blocks_touched(bj, BQ, a.nbq[d], radq);
        const int i0 = si.lo, j0 = sj.lo;
        const int nj = (sj.hi - j0 + 1) * NW, cnt = (si.hi - i0 + 1) * nj;
        auto top_word = [&](int e) {
            const int i = fdiv_floor(e, 1.0f / (float)nj);
            return an[((i0 + i) * a.nbq[d] + j0) * NW + e - i * nj];
        };
        DaRange range = top_word(min(lane, cnt - 1));
        const unsigned raw_tile = a.raw[d * RT + min(lane, RT - 1)];
        const auto rs_a =
            rsrc_of(a.frag + (long long)d * KG * U * RT * 128, (long long)KG * U * RT * 2048);
        const float *const dA_n = a.dA + sbase * G;
        const float inv_sw = 1.0f / (float)SW;
        const int nst = SH * SW * 8;
        struct Ops {
            h8 a[RTW][2];
            h8 b[NT][2];
        };
        for (int pass = 0; pass < U; ++pass) {
            // (rows past the last tile repeat it)
            auto issue_a = [&](int kg, h8 *slot) {
#pragma unroll
                for (int j0 = 0; j0 < AT; j0 += NW) {
                    const int j = j0 + wv;
                    const int rt = min(j >> 1, RT - 1);
                    __builtin_amdgcn_raw_ptr_buffer_load_lds(
                        rs_a, (lds_void *)&slot[j * 64], 16,
                        (int)((unsigned)((((pass * KG + kg) * RT + rt) * 2 + (j & 1)) * 64 + lane) *
                              16u),
                        0, 0, 0);
                }
            };
            if (pass > 0) __syncthreads();   // every wave is done with the staged pass
            issue_a(0, ring0);
            issue_a(1, ring1);
            if (KG > 2) issue_a(2, ring2);
            constexpr int SB = 4;
            for (int e0 = tid; e0 - tid < nst; e0 += SB * THREADS) {
                f4 va[SB], vb[SB];
                int dst[SB];
                bool ok[SB];
#pragma unroll
                for (int u = 0; u < SB; ++u) {
                    const int e = e0 + u * THREADS;
                    const int spx = e >> 3, c = e & 7;
                    const int sy = fdiv_floor(spx, inv_sw), sx = spx - sy * SW;
                    const int pp = p0 - radp + sy, qq = q0 - radq + sx;
                    dst[u] = e < nst ? spx * kBwdChunks + 2 * c : -1;
                    ok[u] = e < nst && on_plane(pp, qq, P, Q);
                    const int v = (s + dg.sign) * ss + pp * sp + qq * sq;
                    const float *src = dA_n + (ok[u] ? (long long)v * G + pass * 64 + 8 * c : 0);
                    va[u] = *(const f4 *)src;
                    vb[u] = *(const f4 *)(src + 4);
                }
                if (pass == 0 && e0 == tid) {
                    // the pixels that received this pixel's h (and x) through a tap
                    for (int e = tid; e < KK; e += THREADS) {
                        const int ka = ((e * a.k_mul) >> 16) - radp, kb = e - (ka + radp) * KQ - radq;
                        tab[e] = (-ka * SW - kb) * kBwdChunks;
                    }
                    if (tid < RT * 16) rowp[tid] = a.rinv[d * RT * 16 + tid];
                }
                if (pass == 0 && e0 == tid) {
                    for (int e = 64 + lane; e < cnt; e += 64) range = da_join(range, top_word(e));
#pragma unroll
                    for (int o = 32; o > 0; o >>= 1) range = da_join(range, da_shuffle(range, o));
                    range = __builtin_bit_cast(
                        DaRange, __builtin_amdgcn_readfirstlane(__builtin_bit_cast(int, range)));
                    raw = (unsigned)__ballot(raw_tile != 0 && lane < RT);
                    f32 = raw != 0 || range.x == 255;
                    own = !f32 && da_wide(range);
                }
                const float scale = flip * exp2i(da_exp(range));
#pragma unroll
                for (int u = 0; u < SB; ++u) {
                    float sc = scale;
                    if (f32 || own) {
                        if (own) {                   // (a pixel is eight lanes)
                            const float top = ok[u] ? top8(va[u], vb[u]) : 0.0f;
                            const int ex = pixel_exp(__float_as_uint(max8(top)));
                            sc = flip * exp2i(ex);
                            if (dst[u] >= 0 && (tid & 7) == 0)
                                *(float *)&stg[((e0 + u * THREADS) >> 3) * kBwdChunks + kBwdScale] = flip * exp2i(-ex);
                        } else if (dst[u] >= 0) {
                            stg[dst[u]] = __builtin_bit_cast(h8, ok[u] ? va[u] : zero);
                            stg[dst[u] + 1] = __builtin_bit_cast(h8, ok[u] ? vb[u] : zero);
                        }
                    }
                    if (dst[u] < 0 || f32) continue;
                    const Split8 w = split8(ok[u] ? va[u] * sc : zero, ok[u] ? vb[u] * sc : zero);
                    stg[dst[u]] = w.hi;
                    stg[dst[u] + 1] = w.lo;
                }
            }
            __builtin_amdgcn_s_waitcnt(kWaitAllLds);
            __syncthreads();

            if (__builtin_expect(f32 || own, 0)) {
                // K-groups kg + 1 and kg + 2 are in flight beside kg
                f4 tap[2][RTW][NT];          // sums of a tap, own scales
                auto barrier = []() {        // (that waits for no load in flight)
                    asm volatile("" ::: "memory");
                    __builtin_amdgcn_s_barrier();
                    asm volatile("" ::: "memory");
                };
                auto slow = [&](int kg, h8 *slot) {
                    if (kg + 2 < KG)
                        __builtin_amdgcn_s_waitcnt(0x0070 | 2 * NDMA);
                    else
                        __builtin_amdgcn_s_waitcnt(kWaitAllLds);
                    barrier();
                    const int odd = kg & 1, bo = tab[kg >> 1];
#pragma unroll
                    for (int nt = 0; nt < NT; ++nt) {
                        const h8 *bp = &stg[spb[nt] + bo + 8 * odd];
                        const h8 b0 = bp[0], b1 = bp[1];
                        const float inv = *(const float *)&stg[spb[nt] - 2 * q4 + bo + kBwdScale];
#pragma unroll
                        for (int i = 0; i < RTW; ++i) {
                            const h8 *ap = &slot[(i * WM * 2 + wm * 2) * 64 + lane];
                            const h8 a0 = ap[0], a1 = ap[64];
                            if (f32) {
                                // eight k-steps of the fp32 instruction
                                const f4 v0 = __builtin_bit_cast(f4, b0), v1 = __builtin_bit_cast(f4, b1);
                                const Wide8 w = widen8(a0, a1, raw >> min(i * WM + wm, RT - 1) & 1);
#pragma unroll
                                for (int j = 0; j < 4; ++j) {
                                    acc[i][nt] = __builtin_amdgcn_mfma_f32_16x16x4f32(w.a[j], v0[j],
                                                                                      acc[i][nt], 0, 0, 0);
                                    acc[i][nt] = __builtin_amdgcn_mfma_f32_16x16x4f32(w.b[j], v1[j],
                                                                                      acc[i][nt], 0, 0, 0);
                                }
                                continue;
                            }
                            f4 x = odd ? tap[0][i][nt] : zero, y = odd ? tap[1][i][nt] : zero;
                            x = mfma_h(a1, b0, x);
                            y = mfma_h(a0, b0, y);
                            x = mfma_h(a0, b1, x);
                            tap[0][i][nt] = x;
                            tap[1][i][nt] = y;
                            if (odd) acc[i][nt] += join(y, x) * inv;
                        }
                    }
                    barrier();
                    if (kg + 3 < KG) issue_a(kg + 3, slot);
                };
#pragma unroll
                for (int i = 0; i < RTW; ++i)
#pragma unroll
                    for (int nt = 0; nt < NT; ++nt) tap[0][i][nt] = tap[1][i][nt] = zero;
#pragma unroll 1
                for (int kg = 0; kg < KG; kg += 3) {
                    slow(kg, ring0);
                    if (kg + 1 < KG) slow(kg + 1, ring1);
                    if (kg + 2 < KG) slow(kg + 2, ring2);
                }
                continue;
            }
            Ops X, Y;
#pragma unroll
            for (int i = 0; i < 2 * RTW; ++i) X.a[i >> 1][i & 1] = ring0[((i >> 1) * WM * 2 + wm * 2 + (i & 1)) * 64 + lane];
            {
                const int bo = tab[0];
#pragma unroll
                for (int i = 0; i < 2 * NT; ++i) X.b[i >> 1][i & 1] = stg[spb[i >> 1] + bo + (i & 1)];
            }
            int bn = tab[0] + 8;             // offset of K-group kg + 1
            auto step = [&](int kg, const Ops &cur, Ops &nxt, const h8 *rd, h8 *dm) {
                const bool more = kg + 3 < KG;
                const int bt = tab[min((kg + 2) >> 1, KK - 1)] + 8 * (kg & 1);
#pragma unroll
                for (int p = 0; p < 3; ++p)
#pragma unroll
                    for (int i = 0; i < RTW; ++i) {
#pragma unroll
                        for (int nt = 0; nt < NT; ++nt)
                            sum[p == 2][i][nt] =
                                mfma_h(cur.a[i][p == 0 ? 1 : 0], cur.b[nt][p == 1 ? 1 : 0],
                                       sum[p == 2][i][nt]);
                        const int k = p * RTW + i;
                        if (k < 2 * RTW) nxt.a[k >> 1][k & 1] = rd[((k >> 1) * WM * 2 + wm * 2 + (k & 1)) * 64 + lane];
                        if (k < 2 * NT) nxt.b[k >> 1][k & 1] = stg[spb[k >> 1] + bn + (k & 1)];
                        if (RTW * 3 < 2 * NT && k == RTW * 3 - 1) {
#pragma unroll
                            for (int m = RTW * 3; m < 2 * NT; ++m)
                                nxt.b[m >> 1][m & 1] = stg[spb[m >> 1] + bn + (m & 1)];
                        }
                        if (k == RTW && more) issue_a(kg + 3, dm);
                        __builtin_amdgcn_sched_barrier(0);
                    }
                bn = bt;
                if (more)
                    __builtin_amdgcn_s_waitcnt(kWaitRingLds);
                else
                    __builtin_amdgcn_s_waitcnt(kWaitAllLds);
                asm volatile("" ::: "memory");
                __builtin_amdgcn_s_barrier();
                asm volatile("" ::: "memory");
            };
            __syncthreads();
            for (int kg = 0; kg + 1 < KG; kg += 6) {
                step(kg, X, Y, ring1, ring0);
                if (kg + 2 < KG) step(kg + 1, Y, X, ring2, ring1);
                if (kg + 3 < KG) step(kg + 2, X, Y, ring0, ring2);
                if (kg + 4 < KG) step(kg + 3, Y, X, ring1, ring0);
                if (kg + 5 < KG) step(kg + 4, X, Y, ring2, ring1);
                if (kg + 6 < KG) step(kg + 5, Y, X, ring0, ring2);
            }
            // KG is even: the last K-group's operands are in Y
#pragma unroll
            for (int p = 0; p < 3; ++p)
#pragma unroll
                for (int i = 0; i < RTW; ++i)
#pragma unroll
                    for (int nt = 0; nt < NT; ++nt)
                        sum[p == 2][i][nt] = mfma_h(Y.a[i][p == 0 ? 1 : 0], Y.b[nt][p == 1 ? 1 : 0],
                                                    sum[p == 2][i][nt]);
        }
#pragma unroll
        for (int i = 0; i < RTW; ++i)
#pragma unroll
            for (int nt = 0; nt < NT; ++nt) sum[1][i][nt] = join(sum[1][i][nt], sum[0][i][nt]);
        unscale = f32 || own ? 1.0f : flip * exp2i(-da_exp(range));
    }

    const int np = dg.T > 1 ? 2 : 1;
    float *const gc0 = a.gcp + a.coff[d] + (long long)n * np * PQ * O;
    const float *const gcin = gc0 + (long long)((t + 1) & 1) * PQ * O;
    float *const gcout = gc0 + (long long)(t & 1) * PQ * O;
    // the cell update's operands of the wave's unit tiles (rt = wm, wm + WM,
    // .. < U), all in flight at once
    f4 e_g[EU][4], e_c[EU], e_cp[EU], e_gn[EU], e_dh[EU];
    const long long vo = sbase + evox[0];
#pragma unroll
    for (int i = 0; i < EU; ++i) {
        const int uo = min(i * WM + wm, U - 1) * 16 + 4 * q4;
        const float *gp = a.gates + (do_h ? vo : sbase) * G + uo;
#pragma unroll
        for (int k = 0; k < 4; ++k) e_g[i][k] = *(const f4 *)(gp + k * O);
        e_c[i] = *(const f4 *)(a.cell + (do_h ? vo : sbase) * O + uo);
        e_cp[i] = *(const f4 *)(a.cell + (t > 0 ? vo - noff : sbase) * O + uo);
        e_gn[i] = *(const f4 *)((has_next ? gcin : gcout) + (long long)epix[0] * O + uo);
        e_dh[i] = *(const f4 *)(a.dh + ((long long)n * V + (do_h ? evox[0] : 0)) * O + uo);
    }
    __builtin_amdgcn_sched_barrier(0);   // (the scheduler would sink each load to its use)
    unsigned top = 0;
    if (elive[0]) {
#pragma unroll
        for (int i = 0; i < RTW; ++i) {
            const int rt = i * WM + wm;
            if (rt >= RT) continue;
            if (rt >= U) {
                // dL/dx of plane t + 1, this direction's share
                if (!has_next) continue;
                const f4 rinv = *(const f4 *)(rowp + rt * 16 + 4 * q4) * unscale;
                const int C = a.g.C, c0 = (rt - U) * 16 + 4 * q4;
                float *out = a.dxd + (vo + noff) * C;
                const f4 v = acc[i][0] * rinv;
                if ((C & 3) == 0 && c0 + 3 < C) {
                    *(f4 *)(out + c0) = v;
                } else {
#pragma unroll
                    for (int k = 0; k < 4; ++k)
                        if (c0 + k < C) out[c0 + k] = v[k];
                }
            }
        }
#pragma unroll
        for (int i = 0; i < EU; ++i) {
            const int rt = i * WM + wm, uo = rt * 16 + 4 * q4;
            if (!do_h || rt >= U) continue;
            f4 rinv = {0.0f, 0.0f, 0.0f, 0.0f};
            if (has_next) rinv = *(const f4 *)(rowp + uo) * unscale;
            const f4 gi = e_g[i][0], gf = e_g[i][1], gg = e_g[i][2], go = e_g[i][3], c = e_c[i];
            f4 di, df, dgv, dov, gco;
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                const float gh = __builtin_fmaf(acc[i][0][k], rinv[k], e_dh[i][k]);
                const float tc = ftanh(c[k]);
                const float gcv = gh * go[k] * (1.0f - tc * tc) + (has_next ? e_gn[i][k] : 0.0f);
                di[k] = gcv * gg[k] * gi[k] * (1.0f - gi[k]);
                df[k] = gcv * (t > 0 ? e_cp[i][k] : 0.0f) * gf[k] * (1.0f - gf[k]);
                dgv[k] = gcv * gi[k] * (1.0f - gg[k] * gg[k]);
                dov[k] = gh * tc * go[k] * (1.0f - go[k]);
                gco[k] = gcv * gf[k];
            }
            float *dp = a.dA + vo * G + uo;
            *(f4 *)dp = di;
            *(f4 *)(dp + O) = df;
            *(f4 *)(dp + 2 * O) = dgv;
            *(f4 *)(dp + 3 * O) = dov;
            *(f4 *)(gcout + (long long)epix[0] * O + uo) = gco;
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                const float v4[4] = {di[k], df[k], dgv[k], dov[k]};
#pragma unroll
                for (int m = 0; m < 4; ++m) {
                    const unsigned bits = __float_as_uint(v4[m]) & 0x7fffffffu;
                    top = bits > top ? bits : top;
                }
            }
        }
    }
    if (do_h) {
        const DaRange range = da_wave(top);
        if (lane == 0) am[((long long)t * a.nblk[d] + bi * a.nbq[d] + bj) * NW + wv] = range;
    }
}

// ---- host side --------------------------------------------------------------

inline int pad8(int c) { return (c + 7) / 8 * 8; }
inline unsigned blocks_for(long long n, int per) { return (unsigned)((n + per - 1) / per); }
inline int max_T(const Geom &g)
{
    int m = 0;
    for (int d = 0; d < g.nd; ++d) m = g.dir[d].T > m ? g.dir[d].T : m;
    return m;
}
inline int staged_chunks(int slots) { return 2 * slots + (slots & 1 ? 0 : 2); }

struct PixBlocks {
    int bp[kDirs], bq[kDirs], nbq[kDirs], nblk[kDirs];
    int max_staged;           // pixels of the largest staged block (with halo)
};
// Blocks of at most `cap` pixels: per direction the shape whose count times
// the work of a block (its pixels at full capacity, plus `halo` per staged
// pixel) is smallest; rows and columns are spread evenly over the blocks.
// Shapes whose staged pixels exceed max_staged are left out (1 x 1 always fits).
PixBlocks pixel_blocks(const Geom &g, int cap, double halo, int max_staged)
{
    PixBlocks b{};
    for (int d = 0; d < g.nd; ++d) {
        const DirGeom &dg = g.dir[d];
        double best = 1e300;
        for (int w0 = 1; w0 <= cap && w0 <= dg.Q; ++w0) {
            const int nbq = (dg.Q + w0 - 1) / w0, bq = (dg.Q + nbq - 1) / nbq;
            if (bq != w0) continue;
            int h0 = cap / bq < dg.P ? cap / bq : dg.P;
            while (h0 > 1 && (h0 + 2 * (g.KP / 2)) * (bq + 2 * (g.KQ / 2)) > max_staged) --h0;
            const int nbp = (dg.P + h0 - 1) / h0, bp = (dg.P + nbp - 1) / nbp;
            const int st = (bp + 2 * (g.KP / 2)) * (bq + 2 * (g.KQ / 2));
            if (st > max_staged && bp * bq > 1) continue;
            const double c = (double)nbp * nbq * (cap + halo * st);
            if (c < best * (1 - 1e-9)) {
                best = c;
                b.bp[d] = bp;
                b.bq[d] = bq;
                b.nbq[d] = nbq;
                b.nblk[d] = nbp * nbq;
            }
        }
        const int st = (b.bp[d] + 2 * (g.KP / 2)) * (b.bq[d] + 2 * (g.KQ / 2));
        if (st > b.max_staged) b.max_staged = st;
    }
    return b;
}

// slot table, bias and scales of the block's rows
inline size_t fwd_h2_table(int KG, int UB) { return (size_t)(KG + 1) * 16 + UB * 512; }
constexpr size_t fwd_h2_ring(int UB) { return (size_t)3 * UB * 8192; }

template <int UB, int NT>
int launch_fwd_h2(const Geom &g, FwdH2Args &a, const PixBlocks &b, hipStream_t st)
{
    a.tab_off = b.max_staged * a.nchp;
    const size_t lds = (size_t)a.tab_off * 16 + fwd_h2_table(a.KG, UB);
    if (hipFuncSetAttribute((const void *)k_step_fwd_h2<UB, NT>,
                            hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds) != hipSuccess)
        return PLSTM_EHIP;
    for (int d = 0; d < kDirs; ++d) {
        a.bp[d] = b.bp[d]; a.bq[d] = b.bq[d]; a.nbq[d] = b.nbq[d]; a.nblk[d] = b.nblk[d];
    }
    const int T = max_T(g);
    for (int t = 0; t < T; ++t) {
        a.t = t;
        int nb = 0;
        for (int d = 0; d < kDirs; ++d) {
            a.base[d] = nb;
            if (t < g.dir[d].T) nb += g.N * a.nblk[d] * a.NUB;
        }
        a.base[kDirs] = nb;
        const int grid = (nb + kXcds - 1) / kXcds * kXcds;
        k_step_fwd_h2<UB, NT><<<grid, 256 * UB, lds, st>>>(a);
        PLSTM_LAUNCH_CHECK();
    }
    return PLSTM_OK;
}

struct FwdK {
    int C8, CS, NSX, NS, KG, KGX;
};
FwdK fwd_k(const Geom &g)
{
    FwdK k;
    const int KK = g.KP * g.KQ;
    k.C8 = pad8(g.C);
    k.CS = k.C8 / 8;
    k.NSX = KK * k.CS;
    k.NS = k.NSX + KK * (g.O / 8);
    k.KG = (k.NS + 3) / 4;
    k.KGX = (k.NSX + 3) / 4;
    return k;
}

// Launch shape of the forward steps: unit groups per workgroup (UB) and 16-pixel
// tiles per wave (NT), by modelled time.  A launch takes its workgroups over (CUs
// x the workgroups that share a CU's LDS and registers) rounds of a workgroup's
// time, in kilocycles from timestamps inside the kernel (25 x 240 x 240, 32 -> 32
// units; 20 x 64 x 64, 64 -> 64; 15 x 128 x 128, 25 -> 32, 7 x 7): staging 5.5 +
// 1.4 per batch of three loads a thread, 2.5 NT for the cell update, and per
// K-group the table below.  A K-group is 12 UB NT products per SIMD (0.19 UB NT);
// one workgroup a CU leaves them waiting on its barriers, more share them, and
// NT = 1 is bound by its LDS reads (ten per 12 products).  No one shape serves the
// range, ms for (UB, NT) = (1,1) / (1,2) / (2,1) / (2,2): 48 x 240 x 240, 32 -> 32
// 14.1 / 12.4 / 11.8 / 13.0; 12 x 60 x 60, 32 -> 32 0.66 / 0.84 / 0.79 / 1.10;
// 15 x 128 x 128, 25 -> 32, 7 x 7 5.5 / 6.0 / 6.4 / 8.5.
struct FwdPlan {
    int UB, NT;
    PixBlocks blocks;
};
FwdPlan plan_fwd(const Geom &g, const FwdK &k, int nchp)
{
    struct Shape {
        int UB, NT, max_res;
        double kg[4];       // kilocycles per K-group with 1 .. max_res workgroups on a CU
    };
    static const Shape shapes[] = {{1, 1, 4, {0.35, 0.55, 0.80, 1.05}},
                                   {1, 2, 3, {0.50, 0.86, 1.25, 0.0}},
                                   {2, 1, 2, {0.62, 1.00, 0.0, 0.0}},
                                   {2, 2, 1, {1.19, 0.0, 0.0, 0.0}}};
    const DevInfo di = device_info();
    const int cus = di.cus > 0 ? di.cus : 256, U = g.O / 16;
    const long long lim = di.max_lds > 0 ? di.max_lds : 65536;
    FwdPlan best{};
    double best_cost = 1e300;
    for (const Shape &s : shapes)
        for (int share = 1; share <= 2; ++share) {      // blocks sized for 1 or 2 a CU
            if (s.UB > U || share > s.max_res) continue;
            const long long fixed = (long long)(fwd_h2_ring(s.UB) + fwd_h2_table(k.KG, s.UB));
            const int max_px = (int)((lim / share - fixed) / (nchp * 16));
            if (max_px < g.KP * g.KQ) continue;
            const PixBlocks pb = pixel_blocks(g, 64 * s.NT, 0.35, max_px);
            const int fit = (int)(lim / (fixed + (long long)pb.max_staged * nchp * 16));
            const int slots = k.CS + g.O / 8, batch = 3 * 256 * s.UB;
            const double once = 5.5 + 1.4 * ((pb.max_staged * slots + batch - 1) / batch) +
                                2.5 * s.NT;
            double cost = 0.0;
            for (int t0 = 0;;) {         // stretches of planes with the same directions
                int t1 = 1 << 30;
                long long nb = 0;
                for (int d = 0; d < g.nd; ++d)
                    if (g.dir[d].T > t0) {
                        nb += (long long)g.N * pb.nblk[d] * (U / s.UB);
                        t1 = g.dir[d].T < t1 ? g.dir[d].T : t1;
                    }
                if (nb == 0) break;
                const long long want = (nb + cus - 1) / cus;
                int res = fit < s.max_res ? fit : s.max_res;
                if (want < res) res = (int)want;
                const double r = (double)nb / ((double)cus * res);
                cost += (t1 - t0) * (once + s.kg[res - 1] * k.KG) * (r <= 1.0 ? 1.0 : r + 0.3);
                t0 = t1;
            }
            if (cost < best_cost) {
                best_cost = cost;
                best.UB = s.UB;
                best.NT = s.NT;
                best.blocks = pb;
            }
        }
    return best;
}

// Reverse steps: U unit tiles and, with dL/dx, the channels' row tiles, spread
// over WM waves of RTW tiles.
struct BwdShape {
    int RT, RTW, WM;
};
BwdShape bwd_shape(const Geom &g, bool with_dx)
{
    BwdShape b;
    b.RT = g.O / 16 + (with_dx ? (g.C + 15) / 16 : 0);
    b.WM = b.RT > 4 || g.O == 64 ? 2 : 1;
    b.RTW = (b.RT + b.WM - 1) / b.WM;
    return b;
}

// tap table and row scales
inline size_t bwd_table(const Geom &g, int RT)
{
    return (size_t)(g.KP * g.KQ + 3) / 4 * 16 + (size_t)RT * 64;
}

template <int RTW, int WM, int EU>
int launch_bwd_h2(const Geom &g, BwdH2Args &a, const PixBlocks &b, bool with_dx, hipStream_t st)
{
    a.tab_off = b.max_staged * kBwdChunks;
    const size_t lds = (size_t)a.tab_off * 16 + bwd_table(g, a.RT);
    if (hipFuncSetAttribute((const void *)k_step_bwd_h2<RTW, WM, EU>,
                            hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds) != hipSuccess)
        return PLSTM_EHIP;
    for (int d = 0; d < kDirs; ++d) {
        a.bp[d] = b.bp[d]; a.bq[d] = b.bq[d]; a.nbq[d] = b.nbq[d]; a.nblk[d] = b.nblk[d];
        a.nbp[d] = b.nbq[d] ? b.nblk[d] / b.nbq[d] : 0;
    }
    // with dL/dx, a last launch (t = -1) gives plane 0's share
    for (int t = max_T(g) - 1; t >= (with_dx ? -1 : 0); --t) {
        a.t = t;
        int nb = 0;
        for (int d = 0; d < kDirs; ++d) {
            a.base[d] = nb;
            if (t < g.dir[d].T && g.dir[d].T > 0) nb += g.N * a.nblk[d];
        }
        a.base[kDirs] = nb;
        const int grid = (nb + kXcds - 1) / kXcds * kXcds;
        k_step_bwd_h2<RTW, WM, EU><<<grid, 256 * WM, lds, st>>>(a);
        PLSTM_LAUNCH_CHECK();
    }
    return PLSTM_OK;
}

int launch_bwd_shape(const Geom &g, BwdH2Args &a, const BwdShape &sh, const PixBlocks &b,
                     bool with_dx, hipStream_t st)
{
    const int U = g.O / 16, EU = (U + sh.WM - 1) / sh.WM;    // unit tiles per wave
    switch ((sh.WM * 8 + sh.RTW) * 4 + EU) {
    case 37: return launch_bwd_h2<1, 1, 1>(g, a, b, with_dx, st);
    case 41: return launch_bwd_h2<2, 1, 1>(g, a, b, with_dx, st);
    case 42: return launch_bwd_h2<2, 1, 2>(g, a, b, with_dx, st);
    case 45: return launch_bwd_h2<3, 1, 1>(g, a, b, with_dx, st);
    case 46: return launch_bwd_h2<3, 1, 2>(g, a, b, with_dx, st);
    case 49: return launch_bwd_h2<4, 1, 1>(g, a, b, with_dx, st);
    case 50: return launch_bwd_h2<4, 1, 2>(g, a, b, with_dx, st);
    case 74: return launch_bwd_h2<2, 2, 2>(g, a, b, with_dx, st);
    case 77: return launch_bwd_h2<3, 2, 1>(g, a, b, with_dx, st);
    case 78: return launch_bwd_h2<3, 2, 2>(g, a, b, with_dx, st);
    case 82: return launch_bwd_h2<4, 2, 2>(g, a, b, with_dx, st);
    default: return PLSTM_EUNSUPPORTED;
    }
}

struct BwdWs {
    float *dA, *gcp, *dxd, *rinv;
    h8 *frag;
    DaRange *amax;
    unsigned *raw;
    long long aoff[kDirs + 1];
    PixBlocks blocks;
};
BwdWs carve_bwd(Carve &cv, const Geom &g, bool with_dx)
{
    const BwdShape sh = bwd_shape(g, with_dx);
    BwdWs w;
    const long long lim = device_info().max_lds > 0 ? device_info().max_lds : 65536;
    const long long fixed =
        (long long)bwd_frags(sh.RTW, sh.WM) * 1024 * 3 + (long long)bwd_table(g, sh.RT);
    w.blocks = pixel_blocks(g, 64, 0.35, (int)((lim - fixed) / (kBwdChunks * 16)));
    w.dA = cv.take<float>((size_t)g.nd * g.N * g.V * 4 * g.O);
    size_t planes = 0;
    long long words = 0;
    for (int d = 0; d < kDirs; ++d) {
        w.aoff[d] = words;
        if (d >= g.nd) continue;
        planes += (size_t)(g.dir[d].T > 1 ? 2 : 1) * g.dir[d].P * g.dir[d].Q;
        words += (long long)g.N * g.dir[d].T * w.blocks.nblk[d] * 4 * sh.WM;
    }
    w.aoff[kDirs] = words;
    w.gcp = cv.take<float>(planes * g.N * g.O);
    w.frag = cv.take<h8>((size_t)g.nd * g.KP * g.KQ * (g.O / 8) * sh.RT * 128);
    w.rinv = cv.take<float>((size_t)g.nd * sh.RT * 16);
    w.raw = cv.take<unsigned>((size_t)g.nd * sh.RT);
    w.amax = cv.take<DaRange>((size_t)words);
    w.dxd = with_dx ? cv.take<float>((size_t)g.nd * g.N * g.V * g.C) : nullptr;
    return w;
}

}  // namespace

int split_stats(const float *x, long long n, SplitStats *part, unsigned *ctl, hipStream_t st)
{
    k_split_stats<false><<<kStatBlocks, 256, 0, st>>>(n, x, part, ctl);
    PLSTM_LAUNCH_CHECK();
    k_split_stats<true><<<kStatBlocks, 256, 0, st>>>(n, x, part, ctl);
    PLSTM_LAUNCH_CHECK();
    return PLSTM_OK;
}

int split_scan(int dtype, const void *x, long long n, int rows, int nx, int nh, const void *wx,
               const void *wh, SplitScan *scan, int *clear, int nclear, hipStream_t st)
{
    const unsigned grid = kStatBlocks + rows / 4;
    if (dtype == PLSTM_BF16)
        k_split_scan<uint16_t><<<grid, 256, 0, st>>>(n, nx, nh, (const uint16_t *)x,
                                                     (const uint16_t *)wx, (const uint16_t *)wh, scan,
                                                     clear, nclear);
    else
        k_split_scan<float><<<grid, 256, 0, st>>>(n, nx, nh, (const float *)x, (const float *)wx,
                                                  (const float *)wh, scan, clear, nclear);
    PLSTM_LAUNCH_CHECK();
    return PLSTM_OK;
}

int split_pad_x(long long nvox, int C, const float *x, float *xp, hipStream_t st)
{
    k_pad_x8<float><<<blocks_for(nvox * pad8(C), 256), 256, 0, st>>>(nvox, C, pad8(C), x, xp);
    PLSTM_LAUNCH_CHECK();
    return PLSTM_OK;
}

// Packed weights, their scales and x's statistics.
struct FwdPack {
    h8 *frag;
    float *bias, *rinv;
    SplitScan *scan;
    unsigned *ctl;
};
static FwdPack carve_pack(Carve &cv, const Geom &g, const FwdK &k)
{
    FwdPack p;
    p.frag = cv.take<h8>((size_t)g.nd * (g.O / 16) * k.KG * 512);
    p.bias = cv.take<float>((size_t)g.nd * 4 * g.O);
    p.rinv = cv.take<float>((size_t)g.nd * 4 * g.O);
    p.scan = cv.take<SplitScan>(1);
    p.ctl = cv.take<unsigned>(2);
    return p;
}
// Floats of the two-plane c^d buffer; the rest of the c^d array holds the packed weights
// where it is large enough, so that inference needs no more than x's copy beside it.
static size_t cell_planes(const Geom &g)
{
    size_t n = 0;
    for (int d = 0; d < g.nd; ++d)
        n += (size_t)g.N * (g.dir[d].T > 1 ? 2 : 1) * g.dir[d].P * g.dir[d].Q * g.O;
    return n;
}
static bool pack_in_cell(const Geom &g, const FwdK &k)
{
    Carve cv(nullptr);
    cv.take<float>(cell_planes(g));
    carve_pack(cv, g, k);
    return cv.off <= saved_state_count(g) * sizeof(float);
}
// fp32 input whose channels are a multiple of eight is read in place (bf16 input too
// wide for its own path is widened).
static bool fwd_in_place(const Geom &g, const FwdK &k, int dtype)
{
    return dtype == PLSTM_F32 && k.C8 == g.C;
}

size_t split_fwd_ws(const Geom &g, int dtype, bool cell_full)
{
    const FwdK k = fwd_k(g);
    Carve cv(nullptr);
    if (!fwd_in_place(g, k, dtype)) cv.take<float>((size_t)g.N * g.V * k.C8);
    if (cell_full || !pack_in_cell(g, k)) carve_pack(cv, g, k);
    return cv.off;
}

int split_fwd(const Geom &g, int dtype, const void *x, const void *wx, const void *wh,
              const void *b, float *hd, float *cell, bool cell_full, float *gates, void *ws,
              hipStream_t st, int *launches)
{
    const FwdK k = fwd_k(g);
    const int U = g.O / 16;
    Carve cv(ws);
    const bool in_place = fwd_in_place(g, k, dtype);
    float *xp = !in_place ? cv.take<float>((size_t)g.N * g.V * k.C8) : nullptr;
    Carve in_cell(cell);
    in_cell.take<float>(cell_planes(g));
    const FwdPack pk = carve_pack(cell_full || !pack_in_cell(g, k) ? cv : in_cell, g, k);
    h8 *const frag = pk.frag;
    float *const bias = pk.bias, *const rinv = pk.rinv;
    SplitScan *const scan = pk.scan;
    unsigned *const ctl = pk.ctl;
    const long long nvox = (long long)g.N * g.V;
    *launches = 2 + (in_place ? 0 : 1) + max_T(g);

    const int KK = g.KP * g.KQ, rows = g.nd * 4 * g.O;
    int rc = split_scan(dtype, x, nvox * g.C, rows, g.C * KK, g.O * KK, wx, wh, scan, nullptr, 0, st);
    if (rc != PLSTM_OK) return rc;
    if (!in_place) {
        const unsigned nb = blocks_for(nvox * k.C8, 256);
        if (dtype == PLSTM_BF16)
            k_pad_x8<uint16_t><<<nb, 256, 0, st>>>(nvox, g.C, k.C8, (const uint16_t *)x, xp);
        else
            k_pad_x8<float><<<nb, 256, 0, st>>>(nvox, g.C, k.C8, (const float *)x, xp);
        PLSTM_LAUNCH_CHECK();
    }
    PackArgs pa;
    pa.O = g.O; pa.C = g.C; pa.CS = k.CS; pa.KK = KK;
    pa.NSX = k.NSX; pa.NS = k.NS; pa.KG = k.KG;
    pa.rows = rows; pa.scan = scan; pa.ctl = ctl; pa.frag = frag; pa.bias = bias; pa.rinv = rinv;
    if (dtype == PLSTM_BF16)
        k_pack_fwd_h2<uint16_t><<<g.nd * U * 4, kPackThreads, 0, st>>>(
            pa, (const uint16_t *)wx, (const uint16_t *)wh, (const uint16_t *)b);
    else
        k_pack_fwd_h2<float><<<g.nd * U * 4, kPackThreads, 0, st>>>(
            pa, (const float *)wx, (const float *)wh, (const float *)b);
    PLSTM_LAUNCH_CHECK();

    FwdH2Args a;
    a.g = g;
    a.C8 = k.C8; a.CS = k.CS; a.NSX = k.NSX; a.NS = k.NS; a.KG = k.KG; a.KGX = k.KGX;
    a.k_mul = (65536 + g.KQ - 1) / g.KQ;
    a.nchp = staged_chunks(k.CS + g.O / 8);
    a.x = in_place ? (const float *)x : xp;
    a.frag = frag; a.bias = bias; a.rinv = rinv; a.ctl = ctl;
    a.hd = hd;
    a.cell = cell_full ? cell : nullptr;
    a.cpp = cell;
    a.gates = gates;
    long long off = 0;
    for (int d = 0; d < kDirs; ++d) {
        a.coff[d] = off;
        if (d < g.nd)
            off += (long long)g.N * (g.dir[d].T > 1 ? 2 : 1) * g.dir[d].P * g.dir[d].Q * g.O;
    }
    const FwdPlan pl = plan_fwd(g, k, a.nchp);
    a.NUB = U / pl.UB;
    switch (pl.UB * 8 + pl.NT) {
    case 9: return launch_fwd_h2<1, 1>(g, a, pl.blocks, st);
    case 10: return launch_fwd_h2<1, 2>(g, a, pl.blocks, st);
    case 17: return launch_fwd_h2<2, 1>(g, a, pl.blocks, st);
    default: return launch_fwd_h2<2, 2>(g, a, pl.blocks, st);
    }
}

size_t split_bwd_ws(const Geom &g)
{
    Carve cv(nullptr), cn(nullptr);
    carve_bwd(cv, g, true);
    carve_bwd(cn, g, false);
    return cv.off > cn.off ? cv.off : cn.off;
}

int split_bwd(const Geom &g, const float *wx, const float *wh, const Saved &sv, const float *dh,
              bool with_dx, void *ws, SplitBwd *out, hipStream_t st)
{
    Carve cv(ws);
    const BwdWs w = carve_bwd(cv, g, with_dx);
    const BwdShape sh = bwd_shape(g, with_dx);
    const int KK = g.KP * g.KQ, U = g.O / 16;
    PackBwdArgs pa;
    pa.O = g.O; pa.C = g.C; pa.KK = KK; pa.RT = sh.RT;
    pa.wx = wx; pa.wh = wh; pa.frag = w.frag; pa.rinv = w.rinv; pa.raw = w.raw;
    pa.rt0 = 0;
    pa.nrt = sh.RT;
    if (with_dx && sh.WM == 2) {
        // row tiles of two waves: the channels' fragments count as dL/dx
        timing_begin("dx_step", st);
        pa.rt0 = U;
        pa.nrt = sh.RT - U;
        k_pack_bwd_h2<<<g.nd * pa.nrt, kPackBwdThreads, 0, st>>>(pa);
        PLSTM_LAUNCH_CHECK();
        timing_end(1, st);
        pa.rt0 = 0;
        pa.nrt = U;
    }
    timing_begin("sweep_bwd_step", st);
    k_pack_bwd_h2<<<g.nd * pa.nrt, kPackBwdThreads, 0, st>>>(pa);
    PLSTM_LAUNCH_CHECK();

    BwdH2Args a;
    a.g = g;
    a.RT = sh.RT; a.KG = 2 * KK;
    a.k_mul = (65536 + g.KQ - 1) / g.KQ;
    a.frag = w.frag; a.rinv = w.rinv; a.raw = w.raw; a.amax = w.amax;
    a.gates = sv.gates; a.cell = sv.cell; a.dh = dh;
    a.dA = w.dA; a.gcp = w.gcp; a.dxd = w.dxd;
    long long off = 0;
    for (int d = 0; d < kDirs; ++d) {
        a.coff[d] = off;
        if (d < g.nd)
            off += (long long)g.N * (g.dir[d].T > 1 ? 2 : 1) * g.dir[d].P * g.dir[d].Q * g.O;
    }
    for (int d = 0; d <= kDirs; ++d) a.aoff[d] = w.aoff[d];
    const int rc = launch_bwd_shape(g, a, sh, w.blocks, with_dx, st);
    if (rc == PLSTM_OK) timing_end(1 + max_T(g) + (with_dx ? 1 : 0), st);
    out->dA = w.dA;
    out->dxd = w.dxd;
    out->used = cv.off;
    return rc;
}

}  // namespace plstm
