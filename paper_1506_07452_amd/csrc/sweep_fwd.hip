// Persistent MFMA forward sweep for O = 16 hidden units, C <= 4 input
// channels, fp32 (Section 2.3, Eq. (7)-(12); the sum of Eq. (13) follows in
// a separate pass).
//
// One cooperative launch runs all six directions (and all batch elements) at
// once.  The plane of each direction is cut into strips of whole rows x a few
// columns; one workgroup (16 waves, four per SIMD) owns one strip for the
// whole sweep.  A strip that fits LDS stays there for the whole sweep (h
// double-buffered, c in LDS, only the halo columns and x_t read per step);
// otherwise, per step:
//
//   for t in 0..T-1:
//     wait until the two neighbouring strips have published h_{t-1}
//     for each chunk of rows of the strip (sized to fit LDS):
//       stage h_{t-1} (chunk + 1-pixel halo) and the input plane x_t into LDS
//       each wave, per tile of 16 pixels:
//         A = bias + im2col(x_t) W_x + im2col(h_{t-1}) W_h   (split operands, split.h)
//         gates, c_t = g i + c_{t-1} f, h_t = o tanh(c_t)    (in registers)
//         write h_t, c_t (and the gates when training) to global memory
//     publish: flag = t + 1 once the stores have completed
//
// The weight fragments (48 KB of split pairs, packed once per call with their row
// scales), the bias and the scales live in LDS for the whole kernel; h of every
// plane stays in the per-direction volume in global memory, so a step only reads
// plane t-1 and writes plane t (no write-after-read hazard).  MFMA layout
// (16x16x32 f16): lane l supplies A[m = l%16][k = 8 (l/16) + j] and B[k][n = l%16],
// j = 0..7, and receives D[4(l/16) + i][l%16], i = 0..3.  Gate-units are on M
// (M-tile g = gate g of the 16 units, the weights are the A operand) and pixels
// on N (B = im2col in slots of eight channels).  Every lane ends with all four
// gates of units 4q..4q+3 of pixel l%16, so the cell update needs no data exchange
// and its loads and stores are 16-byte vectors.
//
// A tile is 72 products of 16 cycles (172 of 32 on the fp32 instruction), 60 LDS
// reads of 16 bytes a lane and the cell update of about a thousand cycles, which
// the four waves of a SIMD overlap.  Measured against the fp32 instruction, one
// launch: 48 x 240 x 240 x 3 inference 3.67 -> 1.87 ms, training (with the stores of
// the gates) 4.0 -> 2.7; 30 x 512 x 512 x 1 inference 8.9 -> 4.3; 2 x 8 x 64 x 64 x 1, bound by the
// hand-over between strips, 0.37 -> 0.32.
#include "common.h"
#include "coherent.h"
#include "sweep.h"
#include "split.h"
#include "strip_plan.h"
#include "timing.h"

namespace plstm {
namespace {

typedef float f4 __attribute__((ext_vector_type(4)));

constexpr int kO = 16;
constexpr int kG = 4 * kO;
constexpr int kWaves = 16;         // four waves per SIMD: gate math of some overlaps the MFMAs of others
constexpr int kKG = 6;             // K-groups: 18 slots of h (9 taps x 2), 6 of x (3 x 2 tap pairs)
constexpr int kAFloats = kKG * 4 * 2 * 256;   // A fragments in LDS: 48 KB
constexpr int kThreads = 64 * kWaves;
constexpr int kHS = 20;          // LDS floats per staged h pixel (16 + 4 pad)
constexpr int kWaitVmcnt0 = 0x0F70;   // s_waitcnt vmcnt(0), other counters unconstrained
constexpr int kBatch = 4;        // staging loads in flight per thread
constexpr int kCS = 20;          // LDS floats per cell state of a resident strip (16 + 4 pad)
constexpr int kResX = 4;         // x_t staging registers per thread (resident strips)

struct SweepArgs {
    Geom g;
    const float *x;
    const h8 *frag;     // [6][kKG][4 gates][2][64] A fragments (k_pack_sweep)
    const float *rows;  // [6][2][64] bias, 1 / scale of the gate rows
    const unsigned *ctl;    // [0] 1: fp32 channels instead of split pairs, [1] scale of x (bits)
    float *hd;          // [6][N][V][16] per-direction h^d
    float *cell;        // [6][N][V][16] c^d
    float *gates;       // [6][N][V][64] or null
    int *flags;         // [blocks] completed steps per strip
    int *err;           // set when a wait gives up
    int max_spin;       // polls before a wait gives up
    int wait_bias;      // added to the awaited step (0; failure-path test mode only)
    int nstrip[kDirs];  // strips per (direction, batch element)
    int first[kDirs];   // first block of direction d
    int chunk_rows[kDirs];  // rows staged per LDS chunk, per direction
    int max_w[kDirs];       // widest strip of each direction (LDS layout)
    int resident[kDirs];    // 1: strips of this direction stay in LDS
};

// Gate nonlinearities from exp and the hardware reciprocal (1 ulp each):
// sigma(a) = 1 / (1 + e^-a);  tanh(a) = 1 - 2 / (e^{2a} + 1), which saturates
// to +-1 at +-inf.
__device__ inline float frcp(float v) { return __builtin_amdgcn_rcpf(v); }
__device__ inline float fsig(float a) { return frcp(1.0f + __expf(-a)); }
__device__ inline float ftanh(float a) { return 1.0f - 2.0f * frcp(__expf(2.0f * a) + 1.0f); }

// Waits until the strip's neighbours have published `step` steps (bounded:
// a wait that never ends raises the error flag and gives up).  Their shared
// columns are then read at device coherence, so no cache invalidate is
// needed.
__device__ inline void wait_neighbours(const SweepArgs &a, int nb_lo, int nb_hi, int step)
{
    const int nb = threadIdx.x == 0 ? nb_lo : (threadIdx.x == 1 ? nb_hi : -1);
    if (nb >= 0) {
        int spins = 0;
        while (__hip_atomic_load(&a.flags[nb], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) <
               step + a.wait_bias) {
            __builtin_amdgcn_s_sleep(1);
            if (++spins > a.max_spin) {
                __hip_atomic_store(a.err, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                break;
            }
            if ((spins & 1023) == 0 &&
                __hip_atomic_load(a.err, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT))
                break;
        }
    }
}

// Publishes `step` completed steps of this strip.  The columns neighbours
// read are written at device coherence; callers make sure those stores have
// completed (every storing wave waited for vmcnt 0) before the flag goes up.
__device__ inline void publish(const SweepArgs &a, int step)
{
    __builtin_amdgcn_s_waitcnt(kWaitVmcnt0);
    __hip_atomic_store(&a.flags[blockIdx.x], step, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// Staged h of a pixel: 16 units as two split slots (8 hi, 8 lo fp16 each), or
// as 16 fp32 values in the same 64 bytes.  Units 4 qd .. 4 qd + 3:
__device__ inline void put_h(float *px, int qd, f4 v, bool f32)
{
    char *p = (char *)px + (qd >> 1) * 32;
    if (f32) {
        *(f4 *)(p + (qd & 1) * 16) = v;
        return;
    }
    const Split4 s = split4(v * kHScale);
    *(h4 *)(p + (qd & 1) * 8) = s.hi;
    *(h4 *)(p + 16 + (qd & 1) * 8) = s.lo;
}
// Staged x: 8 bytes of a pixel in each of two planes `xlo` bytes apart, four
// channels' hi and lo, or channels 0, 1 and 2, 3 in fp32.
__device__ inline void put_x(char *xs, int xlo, int px, int c, float v, float scale, bool f32)
{
    if (f32) {
        *(float *)(xs + (c >> 1) * xlo + px * 8 + (c & 1) * 4) = v;
        return;
    }
    _Float16 hi, lo;
    split1(v * scale, hi, lo);
    *(_Float16 *)(xs + px * 8 + c * 2) = hi;
    *(_Float16 *)(xs + xlo + px * 8 + c * 2) = lo;
}
// 16 bytes that are only 8-byte aligned (two neighbouring pixels of x).
__device__ inline h8 read_pair(const char *p)
{
    const h4 a = *(const h4 *)p, b = *(const h4 *)(p + 8);
    return __builtin_shufflevector(a, b, 0, 1, 2, 3, 4, 5, 6, 7);
}

// A tile's contraction, the sums of Eq. (7)-(9), (11) times their rows' scales.
// Lane group q of K-group kg takes slot 4 kg + q: slot 2 tap + half of h, or slot 18
// + 2 r + j of x, the pixels -1, 0 (j = 0) or 1, 2 (j = 1, the second with zero
// weights) along the axis that is contiguous in LDS, r - 1 across it.  `h` and
// `x` are this lane's pixel; off[kg] its slot's byte offset.
struct SlotOff {
    int h[5];      // K-groups 0 .. 3, and 4 for q < 2
    int x[2];      // K-groups 4 (q >= 2) and 5
    int xlo;       // plane distance of x
};
__device__ __forceinline__ void tile_preact(const float *afr, const char *h, const char *x,
                                            const SlotOff &o, int q4, int lane, f4 (&acc)[4])
{
    f4 cross[4];
#pragma unroll
    for (int g = 0; g < 4; ++g) acc[g] = cross[g] = f4{0.0f, 0.0f, 0.0f, 0.0f};
    const h8 *ap = (const h8 *)afr + lane;
#pragma unroll
    for (int kg = 0; kg < kKG; ++kg) {
        h8 bh, bl;
        if (kg < 4) {
            bh = *(const h8 *)(h + o.h[kg]);
            bl = *(const h8 *)(h + o.h[kg] + 16);
        } else {
            const bool is_h = kg == 4 && q4 < 2;
            const char *p = is_h ? h + o.h[4] : x + o.x[kg - 4];
            bh = read_pair(p);
            bl = read_pair(p + (is_h ? 16 : o.xlo));
        }
#pragma unroll
        for (int g = 0; g < 4; ++g) {
            const h8 ah = ap[(kg * 4 + g) * 128], al = ap[(kg * 4 + g) * 128 + 64];
            cross[g] = mfma_h(al, bh, cross[g]);
            acc[g] = mfma_h(ah, bh, acc[g]);
            cross[g] = mfma_h(ah, bl, cross[g]);
        }
    }
#pragma unroll
    for (int g = 0; g < 4; ++g) acc[g] = join(acc[g], cross[g]);
}
// The same of fp32 channels with the fp32 instruction, eight k-steps a K-group.  In a loop
// that works the slots out again: unrolled beside the other it cost the kernel, whose
// waves have 128 registers, up to 13 spilled.
__device__ __forceinline__ void tile_preact_f32(const float *afr, const char *h, const char *x, int xlo,
                                                int rs, int cs, bool resident, int q4, int lane,
                                                f4 (&acc)[4])
{
#pragma unroll
    for (int g = 0; g < 4; ++g) acc[g] = f4{0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll 1
    for (int kg = 0; kg < kKG; ++kg) {
        int q = q4;
        asm volatile("" : "+v"(q));          // (nothing of it kept over the steps)
        const int slot = 4 * kg + q, tap = slot >> 1, ta = (tap * 11) >> 5, xsl = slot - 18;
        const bool is_h = slot < 18;
        const char *p = is_h ? h + ((ta - 1) * rs + (tap - 3 * ta - 1) * cs) * kHS * 4 + (slot & 1) * 32
                             : x + (((xsl >> 1) - 1) * (resident ? cs : rs) + ((xsl & 1) ? 1 : -1)) * 8;
        f4 b0 = __builtin_bit_cast(f4, read_pair(p));
        f4 b1 = __builtin_bit_cast(f4, read_pair(p + (is_h ? 16 : xlo)));
        // (the pixel with zero weights may hold an infinity)
        const bool one = !is_h && (xsl & 1);
#pragma unroll
        for (int i = 2; i < 4; ++i) {
            b0[i] = one ? 0.0f : b0[i];
            b1[i] = one ? 0.0f : b1[i];
        }
        const h8 *ap = (const h8 *)afr + kg * 512 + lane;
#pragma unroll
        for (int g = 0; g < 4; ++g) {
            const f4 a0 = __builtin_bit_cast(f4, ap[g * 128]), a1 = __builtin_bit_cast(f4, ap[g * 128 + 64]);
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                acc[g] = __builtin_amdgcn_mfma_f32_16x16x4f32(a0[i], b0[i], acc[g], 0, 0, 0);
                acc[g] = __builtin_amdgcn_mfma_f32_16x16x4f32(a1[i], b1[i], acc[g], 0, 0, 0);
            }
        }
    }
}

// A fragments and row scales (split.h), one workgroup per (direction, gate); x
// slots pair the taps of the axis that is contiguous in the direction's strips.
struct PackSweepArgs {
    int C;
    const float *wx, *wh, *b;
    const SplitScan *scan;
    unsigned *ctl;
    h8 *frag;
    float *rows;
    int resident[kDirs];
};
__global__ void __launch_bounds__(256) k_pack_sweep(PackSweepArgs a)
{
    __shared__ SplitStat red;
    __shared__ float fx[16], fh[16];
    const int gate = blockIdx.x & 3, d = blockIdx.x >> 2, tid = threadIdx.x, C = a.C;
    const CallScale cs = call_scale(a.scan, kDirs * kG, &red);
    const bool split = cs.split;
    const int ex = cs.ex, gu0 = d * kG + gate * kO;
    if (tid < 16) {
        const unsigned *const m = a.scan->row[gu0 + tid];
        const int s = row_scale(ex, m[0], m[1]).s;
        fx[tid] = !split ? 1.0f : m[0] ? ldexpf(1.0f, s - ex) : 0.0f;   // (2^(s - ex) may overflow)
        fh[tid] = split ? ldexpf(1.0f, s - 15) : 1.0f;
        a.rows[d * 128 + gate * kO + tid] = a.b[gu0 + tid];
        a.rows[d * 128 + 64 + gate * kO + tid] = split ? ldexpf(1.0f, -s) : 1.0f;
    }
    if (blockIdx.x == 0 && tid == 0) {
        a.ctl[0] = split ? 0u : 1u;
        a.ctl[1] = __float_as_uint(split ? exp2i(ex) : 1.0f);
    }
    __syncthreads();
    for (int e = tid; e < kKG * 64; e += 256) {
        const int lane = e & 63, kg = e >> 6, q = lane >> 4, col = lane & 15, slot = 4 * kg + q;
        f4 w[2];
#pragma unroll
        for (int j = 0; j < 8; ++j) {
            float v = 0.0f;
            if (slot < 18) {
                v = a.wh[((gu0 + col) * kO + 8 * (slot & 1) + j) * 9 + (slot >> 1)] * fh[col];
            } else {
                // pixel and channel of element j: four channels of each pixel, or in
                // fp32 two of each pixel per plane
                const int r = (slot - 18) >> 1, jj = (slot - 18) & 1;
                const int px = split ? j >> 2 : (j >> 1) & 1;
                const int c = split ? j & 3 : (j >> 2) * 2 + (j & 1);
                const int k = 2 * jj + px;                 // tap along the contiguous axis
                if (k < 3 && c < C)
                    v = a.wx[((gu0 + col) * C + c) * 9 + (a.resident[d] ? k * 3 + r : r * 3 + k)] *
                        fx[col];
            }
            w[j >> 2][j & 3] = v;
        }
        h8 *out = a.frag + (((long long)d * kKG + kg) * 4 + gate) * 128 + lane;
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

// Gates, cell and hidden update of four units of one pixel (Eq. (7)-(12)).
// `bs`: biases of the gate rows, then 1 / their scales.
__device__ __forceinline__ void lstm_cell(const f4 (&acc)[4], const float *bs, int q4, f4 cprev,
                                          bool has_prev, f4 &gi, f4 &gf, f4 &gg, f4 &go, f4 &cn,
                                          f4 &hn)
{
    f4 pre[4];
#pragma unroll
    for (int g = 0; g < 4; ++g) {
        const f4 b = *(const f4 *)&bs[g * kO + 4 * q4], r = *(const f4 *)&bs[kG + g * kO + 4 * q4];
#pragma unroll
        for (int i = 0; i < 4; ++i) pre[g][i] = __builtin_fmaf(acc[g][i], r[i], b[i]);
    }
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        gi[i] = fsig(pre[0][i]);
        gf[i] = fsig(pre[1][i]);
        gg[i] = ftanh(pre[2][i]);
        go[i] = fsig(pre[3][i]);
        cn[i] = gg[i] * gi[i] + (has_prev ? cprev[i] : 0.0f) * gf[i];
        hn[i] = go[i] * ftanh(cn[i]);
    }
}

template <int C>
__global__ void __launch_bounds__(kThreads, 1) k_sweep_fwd(SweepArgs a)
{
    extern __shared__ float smem[];
    // ---- which strip this workgroup owns -------------------------------
    int d = 0;
#pragma unroll
    for (int k = 1; k < kDirs; ++k)
        if ((int)blockIdx.x >= a.first[k]) d = k;
    const int local = blockIdx.x - a.first[d];
    const int ns = a.nstrip[d];
    const int n = local / ns, strip = local % ns;
    const DirGeom dg = a.g.dir[d];
    const int q0 = (int)((long long)strip * dg.Q / ns);
    const int q1 = (int)((long long)(strip + 1) * dg.Q / ns);
    const int TQ = q1 - q0, W2 = TQ + 2;
    const int nb_lo = strip > 0 ? (int)blockIdx.x - 1 : -1;
    const int nb_hi = strip + 1 < ns ? (int)blockIdx.x + 1 : -1;

    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int q4 = lane >> 4, col = lane & 15;
    float *whs = smem;                       // [kKG][4 gates][2][64 lanes] A fragments
    float *bs = whs + kAFloats;              // [64] bias, [64] 1 / scale
    const bool f32 = a.ctl[0] != 0;
    const float xscale = __uint_as_float(a.ctl[1]);
    const bool resident = a.resident[d] != 0;
    const int P = dg.P;
    // LDS pixel strides of a staged tile: chunked strips are row-major,
    // resident strips column-major (a tile then covers one or two columns,
    // so the columns next to a neighbour strip form their own tiles).
    const int rs = resident ? 1 : W2, cs = resident ? P + 2 : 1;

    const long long V = a.g.V;
    for (int e = threadIdx.x; e < kAFloats / 4; e += kThreads)
        *(f4 *)&whs[e * 4] = ((const f4 *)(a.frag + (long long)d * kKG * 512))[e];
    if (threadIdx.x < 2 * kG) bs[threadIdx.x] = a.rows[d * 2 * kG + threadIdx.x];
    // byte offsets of this lane's slots from its pixel
    SlotOff so;
#pragma unroll
    for (int kg = 0; kg < 5; ++kg) {
        const int slot = min(4 * kg + q4, 17), tap = slot >> 1;
        so.h[kg] = ((tap / 3 - 1) * rs + (tap % 3 - 1) * cs) * kHS * 4 + (slot & 1) * 32;
    }
#pragma unroll
    for (int k = 0; k < 2; ++k) {
        const int xsl = k ? 2 + q4 : (q4 & 1), r = xsl >> 1;
        so.x[k] = ((r - 1) * (resident ? cs : rs) + ((xsl & 1) ? 1 : -1)) * 8;
    }

    // Base pointers of this (direction, batch element); element offsets inside
    // a slice fit in 32 bits (V * 64 < 2^31 is checked at the boundary).
    const long long dn = ((long long)d * a.g.N + n) * V;
    float *const hd_dn = a.hd + dn * kO;
    // h^d of the slice as a buffer resource for the device-coherent accesses
    // of the columns shared with neighbour strips (this strip's first and
    // last columns and the halo columns beside them)
    const __amdgpu_buffer_rsrc_t hd_rs = coherent_rsrc(hd_dn, V * kO);
    auto is_shared_col = [&](int pc) {
        return (pc == q0 - 1) | (pc == q1) | ((pc == q0) & (nb_lo >= 0)) |
               ((pc == q1 - 1) & (nb_hi >= 0));
    };
    float *const cell_dn = a.cell + dn * kO;
    float *const gates_dn = a.gates ? a.gates + dn * kG : nullptr;
    const float *const x_n = a.x + (long long)n * V * C;
    const int ss = (int)dg.ss, sp = (int)dg.sp, sq = (int)dg.sq;
    const float inv_w2 = 1.0f / (float)W2;

    if (resident) {
        // ================= resident strip: the whole strip in LDS ===========
        // h is double-buffered (h_{t-1} read, h_t written by the epilogue),
        // c stays in LDS, only the two halo columns come from global memory
        // each step and x_{t+1} is loaded while step t computes.  Pixels are
        // numbered column by column; the tiles touching a column next to a
        // neighbour strip run first and the step is published as soon as
        // they are stored, so neighbours seldom wait.
        const int P2 = P + 2;
        const int npl = P2 * W2;
        const int npx = P * TQ;
        const int nmt = (npx + 15) >> 4;
        float *hb0 = bs + 2 * kG;
        float *hb1 = hb0 + npl * kHS;
        char *xs = (char *)(hb1 + npl * kHS);      // two planes of 8 bytes a pixel (+ 2 pixels read past)
        so.xlo = (npl * 8 + 31) & ~15;
        float *cb = (float *)(xs + 2 * so.xlo);    // [npx][kCS] cell states
        int *order = (int *)(cb + npx * kCS);      // tile order, edge tiles first
        int *cnt = order + nmt;                    // edge tiles stored this step
        const float inv_p = 1.0f / (float)P;
        for (int e = threadIdx.x; e < 2 * npl * kHS; e += kThreads) hb0[e] = 0.0f;
        for (int e = threadIdx.x; e < so.xlo / 2; e += kThreads) ((float *)xs)[e] = 0.0f;
        if (threadIdx.x == 0) {
            int k = 0;
            for (int pass = 0; pass < 2; ++pass)
                for (int mt = 0; mt < nmt; ++mt) {
                    const int c0 = (mt * 16) / P, c1 = min(mt * 16 + 15, npx - 1) / P;
                    const bool edge = (c0 == 0 && nb_lo >= 0) || (c1 == TQ - 1 && nb_hi >= 0);
                    if (edge == (pass == 0)) order[k++] = mt;
                }
            int ne = 0;
            for (int mt = 0; mt < nmt; ++mt) {
                const int c0 = (mt * 16) / P, c1 = min(mt * 16 + 15, npx - 1) / P;
                ne += ((c0 == 0 && nb_lo >= 0) || (c1 == TQ - 1 && nb_hi >= 0)) ? 1 : 0;
            }
            cnt[0] = 0;
            cnt[1] = ne;
        }
        // x_t staging registers (loaded one step ahead).  Threads walk the
        // staged plane row by row (coalesced in global memory) and store
        // into the column-major LDS copy.
        float xr[kResX];
        auto issue_x = [&](int splane) {
#pragma unroll
            for (int u = 0; u < kResX; ++u) {
                const int e = threadIdx.x + u * kThreads;
                const int pix = e / C, c = e - (e / C) * C;
                const int rr = fdiv_floor(pix, inv_w2);
                const int pr = rr - 1, pc = pix - rr * W2 + q0 - 1;
                const bool ok = e < npl * C && pr >= 0 && pr < P && pc >= 0 && pc < dg.Q;
                const int off = ok ? (splane + pr * sp + pc * sq) * C + c : 0;
                const float v = x_n[off];
                xr[u] = ok ? v : 0.0f;
            }
        };
        auto commit_x = [&]() {
#pragma unroll
            for (int u = 0; u < kResX; ++u) {
                const int e = threadIdx.x + u * kThreads;
                const int pix = e / C, c = e - (e / C) * C;
                const int rr = fdiv_floor(pix, inv_w2);
                if (e < npl * C) put_x(xs, so.xlo, (pix - rr * W2) * P2 + rr, c, xr[u], xscale, f32);
            }
        };
        issue_x((dg.sign > 0 ? 0 : dg.T - 1) * ss);
        __syncthreads();
        const int n_edge = cnt[1];
        for (int t = 0; t < dg.T; ++t) {
            const int s = dg.sign > 0 ? t : dg.T - 1 - t;
            const int splane = s * ss;
            float *hprev = (t & 1) ? hb0 : hb1;      // h_{t-1}
            float *hcur = (t & 1) ? hb1 : hb0;       // h_t
            if (t > 0) {
                // halo columns of h_{t-1} from the neighbours
                wait_neighbours(a, nb_lo, nb_hi, t);
                __syncthreads();
                const int pplane = (s - dg.sign) * ss;
                for (int e = threadIdx.x; e < 2 * P * 4; e += kThreads) {
                    const int side = e / (P * 4), rem = e - side * P * 4;
                    const int r = rem >> 2, qd = rem & 3;
                    const int pc = side ? q1 : q0 - 1;
                    if (pc >= 0 && pc < dg.Q) {
                        const f4 v =
                            load_coherent(hd_rs, (pplane + r * sp + pc * sq) * kO + qd * 4);
                        put_h(&hprev[((side ? TQ + 1 : 0) * P2 + r + 1) * kHS], qd, v, f32);
                    }
                }
            }
            commit_x();
            __syncthreads();
            // One tile: contraction, cell update, stores (h_t to LDS for the
            // next step and to the volume for the neighbours and the sum).
            auto tile = [&](int mt) {
                const int pa = min(mt * 16 + col, npx - 1);     // this lane's pixel
                const int ca = fdiv_floor(pa, inv_p), ra = pa - ca * P;
                const int base = (ca + 1) * P2 + ra + 1;
                const int v = splane + ra * sp + (q0 + ca) * sq;
                const f4 cv = *(const f4 *)&cb[pa * kCS + 4 * q4];
                f4 acc[4];
                if (__builtin_expect(f32, 0))
                    tile_preact_f32(whs, (const char *)&hprev[base * kHS], xs + base * 8, so.xlo, rs, cs,
                                    true, q4, lane, acc);
                else
                    tile_preact(whs, (const char *)&hprev[base * kHS], xs + base * 8, so, q4, lane, acc);
                f4 gi, gf, gg, go, cn, hn;
                lstm_cell(acc, bs, q4, cv, t > 0, gi, gf, gg, go, cn, hn);
                if (mt * 16 + col < npx) {
                    *(f4 *)&cb[pa * kCS + 4 * q4] = cn;
                    put_h(&hcur[base * kHS], q4, hn, f32);
                    if (is_shared_col(q0 + ca))
                        store_coherent(hd_rs, v * kO + 4 * q4, hn);
                    else
                        *(f4 *)&hd_dn[v * kO + 4 * q4] = hn;
                    if (gates_dn) {
                        *(f4 *)&cell_dn[v * kO + 4 * q4] = cn;
                        float *gp = gates_dn + v * kG + 4 * q4;
                        *(f4 *)&gp[0] = gi;
                        *(f4 *)&gp[kO] = gf;
                        *(f4 *)&gp[2 * kO] = gg;
                        *(f4 *)&gp[3 * kO] = go;
                    }
                }
            };
            // Edge tiles first; once a wave's edge tile has reached L2 it
            // counts it, and the wave that stores the last one publishes.
            // The x_{t+1} prefetch goes out only after a wave's edge tiles,
            // so the store waits do not wait for it.
            int k = wave;
            for (; k < n_edge; k += kWaves) {
                tile(order[k]);
                __builtin_amdgcn_s_waitcnt(kWaitVmcnt0);
                if (lane == 0 && atomicAdd(cnt, 1) == n_edge - 1) publish(a, t + 1);
            }
            if (t + 1 < dg.T) issue_x((dg.sign > 0 ? t + 1 : dg.T - 2 - t) * ss);
            for (; k < nmt; k += kWaves) tile(order[k]);
            if (n_edge == 0) __builtin_amdgcn_s_waitcnt(kWaitVmcnt0);
            __syncthreads();
            if (threadIdx.x == 0) {
                if (n_edge == 0) publish(a, t + 1);
                cnt[0] = 0;
            }
        }
        return;
    }

    // ================= chunked strip: rows staged per step =================
    const int chunk_rows = a.chunk_rows[d];
    float *hs = bs + 2 * kG;
    const int max_px = (chunk_rows + 2) * (a.max_w[d] + 2);
    char *xs = (char *)(hs + max_px * kHS);
    so.xlo = (max_px * 8 + 31) & ~15;
    for (int e = threadIdx.x; e < so.xlo / 2; e += kThreads) ((float *)xs)[e] = 0.0f;
    const float inv_tq = 1.0f / (float)TQ;
    __syncthreads();
    for (int t = 0; t < dg.T; ++t) {
        const int s = dg.sign > 0 ? t : dg.T - 1 - t;
        const int sprev = s - dg.sign;
        if (t > 0) {
            wait_neighbours(a, nb_lo, nb_hi, t);
            __syncthreads();
        }
        const int splane = s * ss, sprev_plane = sprev * ss;
        const int cplane = t > 0 ? sprev_plane : splane;
        for (int r0 = 0; r0 < dg.P; r0 += chunk_rows) {
            const int CH = min(chunk_rows, dg.P - r0);
            const int npl = (CH + 2) * W2;            // staged pixels incl. halo
            // ---- stage h_{t-1} and x_t (zero outside the plane) ----------
            // Branch-free loads from clamped addresses, kBatch per thread in
            // flight before the LDS stores: one memory round trip per batch.
            const int nh = npl * 4, nx = npl * C;
            for (int e0 = threadIdx.x; e0 < max(nh, nx); e0 += kThreads * kBatch) {
                f4 hv[kBatch];
                float xv[kBatch];
#pragma unroll
                for (int u = 0; u < kBatch; ++u) {
                    const int e = e0 + u * kThreads;
                    {
                        const int pix = e >> 2, qd = e & 3;
                        const int rr = fdiv_floor(pix, inv_w2);
                        const int pr = rr + r0 - 1, pc = pix - rr * W2 + q0 - 1;
                        const bool ok = e < nh && t > 0 && pr >= 0 && pr < dg.P && pc >= 0 &&
                                        pc < dg.Q;
                        const int off = ok ? (sprev_plane + pr * sp + pc * sq) * kO + qd * 4 : 0;
                        f4 v;
                        if (is_shared_col(pc))
                            v = load_coherent(hd_rs, off);
                        else
                            v = *(const f4 *)&hd_dn[off];
                        hv[u] = ok ? v : f4{0.0f, 0.0f, 0.0f, 0.0f};
                    }
                    {
                        const int pix = e / C, c = e % C;
                        const int rr = fdiv_floor(pix, inv_w2);
                        const int pr = rr + r0 - 1, pc = pix - rr * W2 + q0 - 1;
                        const bool ok = e < nx && pr >= 0 && pr < dg.P && pc >= 0 && pc < dg.Q;
                        const int off = ok ? (splane + pr * sp + pc * sq) * C + c : 0;
                        const float v = x_n[off];
                        xv[u] = ok ? v : 0.0f;
                    }
                }
#pragma unroll
                for (int u = 0; u < kBatch; ++u) {
                    const int e = e0 + u * kThreads;
                    if (e < nh) put_h(&hs[(e >> 2) * kHS], e & 3, hv[u], f32);
                    if (e < nx) put_x(xs, so.xlo, e / C, e % C, xv[u], xscale, f32);
                }
            }
            __syncthreads();
            // ---- 16-pixel tiles -----------------------------------------
            const int npx = CH * TQ;
            const int nmt = (npx + 15) >> 4;
            for (int mt = wave; mt < nmt; mt += kWaves) {
                const int pa = min(mt * 16 + col, npx - 1);     // this lane's pixel
                const int ra = fdiv_floor(pa, inv_tq);
                const int base = (ra + 1) * W2 + (pa - ra * TQ) + 1;
                const int v = splane + (ra + r0) * sp + (pa - ra * TQ + q0) * sq;
                // c_{t-1} of this lane's units, loaded now so the load overlaps
                // the contraction below; at t = 0 there is no previous plane:
                // read (and discard) this plane's entry so the address stays
                // inside the slice.
                const f4 cv = *(const f4 *)&cell_dn[(v - splane + cplane) * kO + 4 * q4];
                // keep the load above the contraction (the scheduler would
                // otherwise sink it to its use and expose its latency)
                __builtin_amdgcn_sched_barrier(0);
                f4 acc[4];
                if (__builtin_expect(f32, 0))
                    tile_preact_f32(whs, (const char *)&hs[base * kHS], xs + base * 8, so.xlo, rs, cs,
                                    false, q4, lane, acc);
                else
                    tile_preact(whs, (const char *)&hs[base * kHS], xs + base * 8, so, q4, lane, acc);
                if (mt * 16 + col >= npx) continue;
                f4 gi, gf, gg, go, cn, hn;
                lstm_cell(acc, bs, q4, cv, t > 0, gi, gf, gg, go, cn, hn);
                *(f4 *)&cell_dn[v * kO + 4 * q4] = cn;
                if (is_shared_col(pa - ra * TQ + q0))
                    store_coherent(hd_rs, v * kO + 4 * q4, hn);
                else
                    *(f4 *)&hd_dn[v * kO + 4 * q4] = hn;
                if (gates_dn) {
                    float *gp = gates_dn + v * kG + 4 * q4;
                    *(f4 *)&gp[0] = gi;
                    *(f4 *)&gp[kO] = gf;
                    *(f4 *)&gp[2 * kO] = gg;
                    *(f4 *)&gp[3 * kO] = go;
                }
            }
            __syncthreads();
        }
        // ---- publish h_t -------------------------------------------------
        // Every wave waits until its own stores have completed, then one
        // thread raises the flag.
        __builtin_amdgcn_s_waitcnt(kWaitVmcnt0);
        __syncthreads();
        if (threadIdx.x == 0) publish(a, t + 1);
    }
}

// ---- launch planning ------------------------------------------------------
StripCostModel fwd_model(int C)
{
    StripCostModel m;
    m.fixed_bytes = (size_t)(kAFloats + 2 * kG) * sizeof(float) + 64;   // fragments, rows, x padding
    m.px_bytes = (size_t)kHS * sizeof(float) + 16;                      // h + x per pixel
    m.c_sync = 3.0;
    m.c_tile = 1.1;
    m.c_stage0 = 1.0;
    m.c_stage_px = 0.0031;
    m.allow_resident = true;
    m.res_px_bytes = (size_t)2 * kHS * sizeof(float) + 16;   // two h buffers + x
    m.res_own_bytes = (size_t)kCS * sizeof(float) + 1 * sizeof(int);   // c + tile order
    m.res_fixed_bytes = 16 * sizeof(int);                      // counters + alignment of c
    m.res_max_staged = kResX * kThreads / C;                   // x_t fits the registers
    m.c_res_step = 1.6;
    return m;
}

template <int C>
int launch_sweep(const Plan &pl, SweepArgs &args, hipStream_t st)
{
    const void *fn = (const void *)k_sweep_fwd<C>;
    int per_cu = 0;
    if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, k_sweep_fwd<C>, kThreads, pl.lds) !=
        hipSuccess)
        return PLSTM_EHIP;
    if ((long long)per_cu * device_info().cus < pl.blocks) return PLSTM_ENOTCORESIDENT;
    (void)hipFuncSetAttribute(fn, hipFuncAttributeMaxDynamicSharedMemorySize, (int)pl.lds);
    void *kargs[] = {&args};
    if (hipLaunchCooperativeKernel(fn, dim3(pl.blocks), dim3(kThreads), kargs, pl.lds, st) !=
        hipSuccess)
        return PLSTM_EHIP;
    return PLSTM_OK;
}

}  // namespace

bool sweep_fwd_supported(const Geom &g, int dtype)
{
    // bf16 storage: the caller widens x and the parameters to fp32 first
    return (dtype == PLSTM_F32 || dtype == PLSTM_BF16) && g.nd == kDirs && g.KP == 3 &&
           g.KQ == 3 && g.O == kO && g.C >= 1 && g.C <= 4;
}

struct SweepPack {
    h8 *frag;
    float *rows;
    SplitScan *scan;
    unsigned *ctl;
};
static SweepPack carve_pack(Carve &cv)
{
    SweepPack k;
    k.frag = cv.take<h8>((size_t)kDirs * kKG * 512);
    k.rows = cv.take<float>((size_t)kDirs * 2 * kG);
    k.scan = cv.take<SplitScan>(1);
    k.ctl = cv.take<unsigned>(2);
    return k;
}
size_t sweep_fwd_pack_bytes()
{
    Carve cv(nullptr);
    carve_pack(cv);
    return cv.off;
}

size_t sweep_fwd_ws(const Geom &g, bool training)
{
    Carve cv(nullptr);
    if (!training) {
        cv.take<float>(saved_state_count(g));   // h^d
        cv.take<float>(saved_state_count(g));   // c^d
    }
    cv.take<int>(1024 + 1);                     // flags + err
    cv.take<char>(sweep_fwd_pack_bytes());
    return cv.off;
}

int sweep_fwd(const Geom &g, const float *x, const float *wx, const float *wh, const float *b,
              float *hd, float *cell, float *gates, int *flags, void *pack, hipStream_t st,
              bool allow_resident)
{
    const DevInfo di = device_info();
    if (di.cus <= 0) return PLSTM_EHIP;
    const size_t lds_limit = (size_t)(di.max_lds > 0 ? di.max_lds : 65536) - 1024;
    const int budget = di.cus < 1024 ? di.cus : 1024;
    StripCostModel model = fwd_model(g.C);
    model.allow_resident = allow_resident;
    const Plan pl = make_plan(g, budget, model, lds_limit);
    if (pl.blocks > budget) return PLSTM_EUNSUPPORTED;
    for (int d = 0; d < kDirs; ++d) {
        if (pl.chunk_rows[d] < 1) return PLSTM_EUNSUPPORTED;
        // a resident strip's x_t plane must fit the staging registers
        if (pl.resident[d] &&
            (long long)(g.dir[d].P + 2) * (pl.max_w[d] + 2) * g.C > (long long)kResX * kThreads)
            return PLSTM_EUNSUPPORTED;
    }

    SweepArgs args;
    args.g = g;
    Carve cv(pack);
    const SweepPack pk = carve_pack(cv);
    args.x = x; args.frag = pk.frag; args.rows = pk.rows; args.ctl = pk.ctl;
    args.hd = hd; args.cell = cell; args.gates = gates;
    args.flags = flags;
    args.err = flags + 1024;
    args.max_spin = g_wait_spin_limit;
    args.wait_bias = g_wait_bias;
    for (int d = 0; d < kDirs; ++d) {
        args.nstrip[d] = pl.nstrip[d];
        args.first[d] = pl.first[d];
    }
    for (int d = 0; d < kDirs; ++d) {
        args.chunk_rows[d] = pl.chunk_rows[d];
        args.max_w[d] = pl.max_w[d];
        args.resident[d] = pl.resident[d];
    }

    int rc = split_scan(PLSTM_F32, x, (long long)g.N * g.V * g.C, kDirs * kG, g.C * 9, kO * 9, wx, wh,
                        pk.scan, flags, 1024 + 1, st);   // (flags and the error word start from zero)
    if (rc != PLSTM_OK) return rc;
    PackSweepArgs pa;
    pa.C = g.C;
    pa.wx = wx; pa.wh = wh; pa.b = b;
    pa.scan = pk.scan; pa.ctl = pk.ctl; pa.frag = pk.frag; pa.rows = pk.rows;
    for (int d = 0; d < kDirs; ++d) pa.resident[d] = pl.resident[d];
    k_pack_sweep<<<kDirs * 4, 256, 0, st>>>(pa);
    PLSTM_LAUNCH_CHECK();
    timing_begin("sweep_fwd_mfma", st);
    switch (g.C) {
    case 1: rc = launch_sweep<1>(pl, args, st); break;
    case 2: rc = launch_sweep<2>(pl, args, st); break;
    case 3: rc = launch_sweep<3>(pl, args, st); break;
    default: rc = launch_sweep<4>(pl, args, st); break;
    }
    timing_end(1, st);
    if (rc != PLSTM_OK) return rc;
    PoisonList poison;
    poison.ptr[0] = hd;
    poison.count[0] = (long long)saved_state_count(g);
    return wait_check(args.err, poison, st);
}

}  // namespace plstm
