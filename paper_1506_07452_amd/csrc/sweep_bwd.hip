// Backward of the layer for O = 16 hidden units, fp32: back-propagation
// through the six sweeps (the chain rule through Section 2.3, Eq. (7)-(13),
// in reverse plane order) and the parameter gradients.
//
// (1) k_sweep_bwd, persistent, one cooperative launch for all directions, on
//     the forward's strip decomposition.  For plane t (last to first):
//       gh   = dL/dh[plane t] + sum_taps dA_{t+1}[p - tap] W_h^T      (MFMA)
//       gc   = gh o (1 - tanh^2 c_t) + gc_{t+1} f_{t+1}
//       dA_o = gh tanh(c_t) o (1 - o)     dA_i = gc g i (1 - i)
//       dA_g = gc i (1 - g^2)             dA_f = gc c_{t-1} f (1 - f)
//     The transposed 3x3 convolution is a contraction of K = 9 x 64
//     (tap, gate-unit) on split operands (split.h) with units on M and pixels
//     on N: a tap is two K-groups of 32, lane l takes pixel l%16 and eight
//     gate-units (hi and lo, two LDS reads of 16 bytes) for the B operand, the
//     transposed recurrent weights are the A operand, resident in LDS, and each
//     lane ends with four consecutive units of one pixel, so every epilogue
//     load and store is a 16-byte vector.  dA_{t+1} has one scale per strip and
//     step, from its own range of |dA| and those its neighbours publish with
//     their flags; in a step that one scale does not serve (da_wide) each
//     pixel has its own, and a step with a value that is not finite, or weights
//     that one scale does not serve, keep the fp32 instruction on the same LDS.
//     The scale's sign alternates from step to step and strip to strip,
//     so that the instruction's rounding towards -inf cancels in db.  The
//     product gc_t f_t is what plane t - 1 needs, so that is what is kept.
//     dA of every voxel is kept for (2) and for dL/dx.
// (2) dW = sum over voxels of dA (x) [im2col(h_{t-1}), im2col(x_t), 1]: the
//     plane-step path's kernels (split_wgrad.hip).
#include "common.h"
#include "coherent.h"
#include "split.h"
#include "strip_plan.h"
#include "sweep.h"
#include "timing.h"

namespace plstm {
namespace {

typedef float f4 __attribute__((ext_vector_type(4)));

constexpr int kO = 16;
constexpr int kG = 4 * kO;
constexpr int kWaves = 16;             // four waves per SIMD
constexpr int kKG = 18;                    // K-groups: 9 taps x 2 halves of 64 gate-units
constexpr int kWaFloats = kKG * 2 * 64 * 4 + 32;   // W_h^T fragments in LDS; 1 / row scales, 16 words of state
constexpr int kThreads = 64 * kWaves;
// A staged dA pixel is 256 bytes in LDS, eight gate-units after eight: their hi
// halves (16 bytes) and their lo halves.  Its 16-byte chunk c sits at position
// c ^ (pixel & 15), so the 16 pixels a read instruction touches hit 16 different
// bank groups.
__device__ inline int swz(int c, int pix) { return c ^ (pix & 15); }
constexpr int kOutOfRange = 0x7ffffff0;    // buffer offset past any resource: reads zero
typedef __attribute__((address_space(3))) void lds_void;
constexpr int kWaitVmcnt0 = 0x0F70;   // s_waitcnt vmcnt(0), other counters unconstrained

__device__ inline float frcp(float v) { return __builtin_amdgcn_rcpf(v); }

__device__ inline float ftanh(float a) { return 1.0f - 2.0f * frcp(__expf(2.0f * a) + 1.0f); }

struct BwdArgs {
    Geom g;
    const float *wh;
    const float *gates, *cell;   // saved forward activations [6][N][V][64], [6][N][V][16]
    const float *dh;             // dL/dh [N][V][16]
    float *dA;                   // [6][N][V][64] gate pre-activation gradients
    float *gcf;                  // [6][N][V][16] dL/dc_t * f_t, carried to plane t - 1
    // [blocks] steps done << 32 | (range of the plane before the last) << 16 | of the last, a
    // range being DaRange's two exponents in a byte each
    unsigned long long *flags;
    int *err;
    int max_spin;                // polls before a wait gives up
    int wait_bias;               // added to the awaited step (0; failure-path test mode only)
    int nstrip[kDirs], first[kDirs], chunk_rows[kDirs], max_w[kDirs];
    int resident[kDirs];         // 1: the strip's dA stays in LDS for the sweep
};

// The largest of sixteen magnitudes (a NaN apart: it spreads whichever way it is multiplied).
__device__ inline float top_of(f4 a, f4 b, f4 c, f4 d)
{
    float m = 0.0f;
#pragma unroll
    for (int i = 0; i < 4; ++i)
        m = fmaxf(fmaxf(m, fmaxf(fabsf(a[i]), fabsf(b[i]))), fmaxf(fabsf(c[i]), fabsf(d[i])));
    return m;
}

// Epilogue operands of one tile (this lane's pixel, units 4 q4 .. 4 q4 + 3).
struct BwdEpi {
    f4 dh, gi, gf, gg, go, c, gcfn, cp;
};

// sum over taps of dA_{t+1}[p - tap] W_h^T for one 16-pixel tile, times the scales:
// `base` is the lane's LDS pixel, whose row and column neighbours are `rs` and
// `cs` LDS pixels apart.  K-group 2 tap + half: gate-units 32 half + 8 q4 .. + 7 of
// the lane's pixel as B, read one K-group ahead, the matching W_h^T fragment as A
// (read ahead too, the resident strips' 128 registers would not do); the four
// waves of a SIMD hide the rest.
__device__ __forceinline__ f4 contract_bwd(const float *as, const float *was, int base, int rs,
                                           int cs, int q4, int lane)
{
    h8 b[2][2];
    auto load = [&](int kg) {
        const int tap = kg >> 1, half = kg & 1, k = kg & 1;
        // h_t at pixel p fed A_{t+1} at p - (tap offset)
        const int pp = base - ((tap / 3 - 1) * rs + (tap % 3 - 1) * cs);
        // (chunks 8 half + 2 q4 and the next: bits 3 and 0 of the position)
        const int o = (pp * kG + 4 * swz(2 * q4, pp)) ^ (half * 32);
        b[k][0] = *(const h8 *)&as[o];
        b[k][1] = *(const h8 *)&as[o ^ 4];
    };
    f4 acc = {0.0f, 0.0f, 0.0f, 0.0f}, x0 = acc, x1 = acc;
    load(0);
#pragma unroll
    for (int kg = 0; kg < kKG; ++kg) {
        const h8 wl = *(const h8 *)&was[((kg * 2 + 1) * 64 + lane) * 4];
        const h8 wh = *(const h8 *)&was[((kg * 2 + 0) * 64 + lane) * 4];
        if (kg + 1 < kKG) load(kg + 1);
        // keep the reads ahead of this K-group's products
        __builtin_amdgcn_sched_barrier(0);
        const int k = kg & 1;
        x0 = mfma_h(wl, b[k][0], x0);
        acc = mfma_h(wh, b[k][0], acc);
        x1 = mfma_h(wh, b[k][1], x1);
        __builtin_amdgcn_sched_barrier(0);
    }
    return join(acc, x0 + x1);
}

// The same where each pixel has its own scale: a tap's sums start from zero and are
// added up times 1 / its pixel's scale (`pinv`, by LDS pixel).
__device__ __forceinline__ f4 contract_bwd_own(const float *as, const float *was, const float *pinv,
                                               int base, int rs, int cs, int q4, int lane)
{
    f4 acc = {0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll 1
    for (int tap = 0; tap < 9; ++tap) {
        const int ta = (tap * 11) >> 5, pp = base - ((ta - 1) * rs + (tap - 3 * ta - 1) * cs);
        const int o0 = pp * kG + 4 * swz(2 * q4, pp);
        f4 x = {0.0f, 0.0f, 0.0f, 0.0f}, y = x;
#pragma unroll
        for (int half = 0; half < 2; ++half) {
            const int o = o0 ^ (half * 32), kg = 2 * tap + half;
            const h8 bh = *(const h8 *)&as[o], bl = *(const h8 *)&as[o ^ 4];
            const h8 wh = *(const h8 *)&was[((kg * 2 + 0) * 64 + lane) * 4];
            const h8 wl = *(const h8 *)&was[((kg * 2 + 1) * 64 + lane) * 4];
            x = mfma_h(wl, bh, x);
            y = mfma_h(wh, bh, y);
            x = mfma_h(wh, bl, x);
        }
        acc += join(y, x) * pinv[pp];
    }
    return acc;
}
// The same of dA as it is, with the fp32 instruction: a gate-unit a lane group and step.
// Seldom taken, so nothing is read ahead and little is kept in registers.
__device__ __forceinline__ f4 contract_bwd_f32(const float *as, const float *was, bool raw, int base,
                                               int rs, int cs, int q4, int lane)
{
    f4 acc = {0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll 1
    for (int k = 0; k < 2 * kKG; ++k) {
        const int kg = k >> 1, j = k & 1, tap = kg >> 1, half = kg & 1, ta = (tap * 11) >> 5;
        const int pp = base - ((ta - 1) * rs + (tap - 3 * ta - 1) * cs);
        const int o = ((pp * kG + 4 * swz(2 * q4, pp)) ^ (half * 32)) ^ (4 * j);
        const f4 b = *(const f4 *)&as[o];
        const h4 hi = *(const h4 *)&was[((kg * 2 + 0) * 64 + lane) * 4 + 2 * j];
        const h4 lo = *(const h4 *)&was[((kg * 2 + 1) * 64 + lane) * 4 + 2 * j];
        f4 w = *(const f4 *)&was[((kg * 2 + j) * 64 + lane) * 4];
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            w[i] = raw ? w[i] : __builtin_fmaf((float)lo[i], kLoInv, (float)hi[i]);
            acc = __builtin_amdgcn_mfma_f32_16x16x4f32(w[i], b[i], acc, 0, 0, 0);
        }
    }
    return acc;
}

// One launch, against the contraction on v_mfma_f32_16x16x4 (144 instructions of 32
// cycles a tile; now 54 of 16): 48 x 240 x 240 3.75 -> 2.95 ms, which is 15.6 GB of
// activations and dA at 5.3 TB/s; 2 x 8 x 64 x 64 x 1, forward and backward, 0.836 ->
// 0.798 ms (bound by the hand-over between strips).
__global__ void __launch_bounds__(kThreads, 1) k_sweep_bwd(BwdArgs a)
{
    extern __shared__ float smem[];
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
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int q4 = lane >> 4, col = lane & 15;
    const int chunk_rows = a.chunk_rows[d];
    // A fragments of W_h^T in LDS (registers stay free for four waves per SIMD):
    // entry (K-group, hi or lo, lane) holds, for lane l, gate-units
    // 32 half + 8 (l/16) .. + 7 of output unit l%16, times the unit's scale.
    // Then 1 / the scales, and the state of the step:
    float *was = smem;
    float *winv = was + kKG * 2 * 64 * 4;
    unsigned *state = (unsigned *)(winv + 16);
    // by step parity: range of |dA| (DaRange's x and y) of the strip, of its edge tiles
    unsigned *mx = state, *emx = state + 4;
    unsigned *nbe = state + 8;               // ranges of the neighbours' planes, x | y << 8
    float *as = smem + kWaFloats;
    // the weights' largest and smallest magnitudes and counts by unit, only here
    unsigned *wmx = (unsigned *)as, *wmn = wmx + 16, *wnz = wmx + 32, *wsm = wmx + 48;
    if (threadIdx.x < 16) {
        wmx[threadIdx.x] = wnz[threadIdx.x] = wsm[threadIdx.x] = state[threadIdx.x] = 0u;
        wmn[threadIdx.x] = ~0u;
    }
    __syncthreads();
    const float *const wh_d = a.wh + (long long)d * kG * kO * 9;
    const int wrow = threadIdx.x & 15;               // a unit's nine taps of one gate-unit a thread
    static_assert(kThreads == kG * kO, "");
    auto tap_bits = [&](int tap) {
        return __float_as_uint(wh_d[threadIdx.x * 9 + tap]) & 0x7fffffffu;
    };
    {
        unsigned m0 = 0u, m1 = ~0u;
#pragma unroll
        for (int tap = 0; tap < 9; ++tap) {
            m0 = max(m0, tap_bits(tap));
            m1 = min(m1, tap_bits(tap) - 1u);        // (zeros apart)
        }
        atomicMax(&wmx[wrow], m0);
        atomicMin(&wmn[wrow], m1);
    }
    __syncthreads();
    bool wild = wmx[wrow] >= 0x7f800000u;
    if (__syncthreads_or(wmn[wrow] != ~0u && wmn[wrow] + 1u + kStatRange < wmx[wrow])) {   // (seldom)
        for (int tap = 0; tap < 9; ++tap) {
            const unsigned m = tap_bits(tap);
            if (m) atomicAdd(&wnz[wrow], 1u);
            if (m && m + kStatRange < wmx[wrow]) atomicAdd(&wsm[wrow], 1u);
        }
        __syncthreads();
        wild |= wsm[wrow] > wnz[wrow] / 64u;
    }
    const bool raw = __syncthreads_or(wild) != 0;    // fp32 weights
    if (threadIdx.x < 16) winv[threadIdx.x] = raw ? 1.0f : exp2i(-scale_exp(wmx[threadIdx.x]));
    for (int e = threadIdx.x; e < kKG * 64; e += kThreads) {
        const int l = e & 63, kg = e >> 6;
        const int lq = l >> 4, lc = l & 15, tap = kg >> 1;
        const float sc = raw ? 1.0f : exp2i(scale_exp(wmx[lc]));
        f4 v[2];
#pragma unroll
        for (int j = 0; j < 8; ++j)
            v[j >> 2][j & 3] = wh_d[((32 * (kg & 1) + 8 * lq + j) * kO + lc) * 9 + tap] * sc;
        const Split8 sp = split8(v[0], v[1]);
        *(h8 *)&was[((kg * 2 + 0) * 64 + l) * 4] = raw ? __builtin_bit_cast(h8, v[0]) : sp.hi;
        *(h8 *)&was[((kg * 2 + 1) * 64 + l) * 4] = raw ? __builtin_bit_cast(h8, v[1]) : sp.lo;
    }
    __syncthreads();                         // (wmx's words are staged over next)
    // Waits (bounded) for the neighbours' step r and leaves the ranges of the
    // planes they then finished; a neighbour may be one step further.
    auto wait_neighbours = [&](int r) {
        const int nb = threadIdx.x == 0 ? nb_lo : (threadIdx.x == 1 ? nb_hi : -1);
        if (nb < 0) return;
        int spins = 0;
        unsigned long long w;
        while ((int)((w = __hip_atomic_load(&a.flags[nb], __ATOMIC_RELAXED,
                                            __HIP_MEMORY_SCOPE_AGENT)) >> 32) < r + a.wait_bias) {
            __builtin_amdgcn_s_sleep(1);
            if (++spins > a.max_spin) {
                __hip_atomic_store(a.err, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                break;
            }
            if ((spins & 1023) == 0 &&
                __hip_atomic_load(a.err, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT))
                break;
        }
        nbe[threadIdx.x] = ((int)(w >> 32) > r ? w >> 16 : w) & 0xffffu;
    };
    // Publishes r + 1 steps with the ranges of this plane and the one before
    // (`m`: by step parity).
    auto publish = [&](int r, const unsigned *m) {
        const int p = 2 * (r & 1), q = p ^ 2;
        const unsigned cur = m[p] | m[p + 1] << 8, before = m[q] | m[q + 1] << 8;
        const unsigned long long w =
            (unsigned long long)(r + 1) << 32 | before << 16 | cur;
        __hip_atomic_store(&a.flags[blockIdx.x], w, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    };
    // Range of dA_{t+1} at step r (all threads, after the wait's barrier).
    auto step_range = [&](int r) {
        const int q = 2 * ((r & 1) ^ 1);
        DaRange v = {(unsigned short)mx[q], (unsigned short)mx[q + 1]};
#pragma unroll
        for (int k = 0; k < 2; ++k)
            v = da_join(v, DaRange{(unsigned short)(nbe[k] & 255u), (unsigned short)(nbe[k] >> 8)});
        return __builtin_bit_cast(DaRange, __builtin_amdgcn_readfirstlane(__builtin_bit_cast(int, v)));
    };
    auto widen = [&](unsigned *m, DaRange v) {           // (one lane of a wave)
        atomicMax(&m[0], (unsigned)v.x);
        atomicMax(&m[1], (unsigned)v.y);
    };
    auto step_sign = [&](int r) { return (strip + r) & 1 ? -1.0f : 1.0f; };
    // fp32 slot `sl` of LDS pixel `pix`, split in place (by eight lanes a pixel; with `pinv`
    // by a scale of the pixel's own, left there)
    auto split_slot = [&](int pix, int sl, float scale, float *pinv) {
        float *p0 = &as[pix * kG + 4 * swz(2 * sl, pix)], *p1 = &as[pix * kG + 4 * swz(2 * sl + 1, pix)];
        if (pinv) {
            const int ex = pixel_exp(__float_as_uint(max8(top8(*(const f4 *)p0, *(const f4 *)p1))));
            scale = exp2i(ex);
            if (sl == 0) pinv[pix] = exp2i(-ex);
        }
        const Split8 sp = split8(*(const f4 *)p0 * scale, *(const f4 *)p1 * scale);
        *(h8 *)p0 = sp.hi;
        *(h8 *)p1 = sp.lo;
    };

    const long long V = a.g.V;
    const long long dn = ((long long)d * a.g.N + n) * V;
    const float *const gates_dn = a.gates + dn * kG;
    const float *const cell_dn = a.cell + dn * kO;
    float *const dA_dn = a.dA + dn * kG;
    // the slice as a buffer resource for the device-coherent accesses
    // (its byte size fits 32 bits: checked on the host)
    const __amdgpu_buffer_rsrc_t dA_rs = coherent_rsrc(dA_dn, V * kG);
    float *const gcf_dn = a.gcf + dn * kO;
    const float *const dh_n = a.dh + (long long)n * V * kO;
    const int ss = (int)dg.ss, sp = (int)dg.sp, sq = (int)dg.sq;
    const float inv_tq = 1.0f / (float)TQ, inv_w2 = 1.0f / (float)W2;
    // Columns that pass between neighbouring strips (this strip's first and
    // last, and the halo columns beside them).  Their dA is stored and loaded
    // at device coherence (write-through / read-through at agent scope, the
    // accesses relaxed agent-scope atomics use), so a strip's step needs no
    // L2 writeback before its flag and no L2 invalidate after waiting: once a
    // strip's coherent stores have completed (vmcnt) its flag goes up.
    auto is_shared_col = [&](int pc) {
        return (pc == q0 - 1) | (pc == q1) | ((pc == q0) & (nb_lo >= 0)) |
               ((pc == q1 - 1) & (nb_hi >= 0));
    };


    if (a.resident[d]) {
        // ============ resident strip: dA of the whole strip stays in LDS ============
        // dA_t overwrites dA_{t+1} in place: each wave keeps its tiles' dA in
        // registers until every wave's contraction has read dA_{t+1} and the
        // neighbours' exponents are there (one barrier), then writes them split.
        // Only the two halo columns come from the neighbours each step.  Pixels are numbered column by column
        // (LDS pixel (column + 1) (P + 2) + row + 1); the tiles touching a
        // column next to a neighbour strip run first and the step is
        // published as soon as they are stored.  At most two tiles per wave
        // (checked on the host).
        const int P = dg.P, P2 = P + 2;
        const int npl = P2 * W2;
        const int npx = P * TQ;
        const int nmt = (npx + 15) >> 4;
        float *const px_inv = as + (size_t)npl * kG;    // 1 / scale of each pixel, where it has one
        int *order = (int *)(px_inv + npl);            // tile order, edge tiles first
        int *cnt = order + nmt;                         // edge tiles stored this step
        const float inv_p = 1.0f / (float)P;
        for (int e = threadIdx.x; e < npl * (kG / 4); e += kThreads)
            *(f4 *)&as[e * 4] = f4{0.0f, 0.0f, 0.0f, 0.0f};   // dA_T = 0, halo rows
        // (pixels off the plane stay zero: their scale is only to be finite)
        for (int e = threadIdx.x; e < npl; e += kThreads) px_inv[e] = 0.0f;
        if (threadIdx.x == 0) {
            int k = 0, ne = 0;
            for (int pass = 0; pass < 2; ++pass)
                for (int mt = 0; mt < nmt; ++mt) {
                    const int c0 = (mt * 16) / P, c1 = min(mt * 16 + 15, npx - 1) / P;
                    const bool edge = (c0 == 0 && nb_lo >= 0) || (c1 == TQ - 1 && nb_hi >= 0);
                    if (edge == (pass == 0)) order[k++] = mt;
                    ne += (pass == 0 && edge) ? 1 : 0;
                }
            cnt[0] = 0;
            cnt[1] = ne;
        }
        __syncthreads();
        const int n_edge = cnt[1];
        // A lane handles the same pixel of its tiles at every step, so it
        // keeps (gc f)_t for the next step and the c_{t-1} it loaded, which is
        // the next step's c_t, in registers: neither is loaded again and gc f
        // is never stored.
        f4 carry_gcf[2], carry_c[2];
        f4 hold[2][4];               // dA_{t+1} of this lane's pixel
        int hbase[2];
#pragma unroll
        for (int it = 0; it < 2; ++it) {
            carry_gcf[it] = carry_c[it] = f4{0.0f, 0.0f, 0.0f, 0.0f};
            hbase[it] = -1;
        }
        for (int r = 0; r < dg.T; ++r) {
            const int t = dg.T - 1 - r;
            const int s = dg.sign > 0 ? t : dg.T - 1 - t;
            const bool has_next = t + 1 < dg.T, has_prev = t > 0;
            const int splane = s * ss;
            const int nplane = has_next ? (s + dg.sign) * ss : splane;
            const int pplane = has_prev ? (s - dg.sign) * ss : splane;
            float inv = 0.0f;
            bool f32 = false, own = false;
            if (r > 0) {
                wait_neighbours(r);
                __syncthreads();
                const DaRange range = step_range(r);
                const int ex = da_exp(range);
                const float scale = step_sign(r) * exp2i(ex);
                f32 = raw || range.x == 255;
                own = !f32 && da_wide(range);
                inv = f32 || own ? 1.0f : step_sign(r) * exp2i(-ex);
                // every contraction has read dA_{t+2}: overwrite it with dA_{t+1}
#pragma unroll
                for (int it = 0; it < 2; ++it) {
                    if (hbase[it] < 0) continue;
                    const int pb = hbase[it];
                    float sc = scale;
                    if (__builtin_expect(own, 0)) {
                        float m = top_of(hold[it][0], hold[it][1], hold[it][2], hold[it][3]);
#pragma unroll
                        for (int o = 32; o > 8; o >>= 1) m = fmaxf(m, __shfl_xor(m, o));
                        const int px = pixel_exp(__float_as_uint(m));
                        sc = exp2i(px);
                        px_inv[pb] = exp2i(-px);
                    }
#pragma unroll
                    for (int g = 0; g < 4; ++g) {
                        if (f32) {
                            *(f4 *)&as[pb * kG + 4 * swz(4 * g + q4, pb)] = hold[it][g];
                            continue;
                        }
                        const Split4 sp = split4(hold[it][g] * sc);
                        // gate-units 16 g + 4 q4 .. + 3: half of slot 2 g + q4 / 2
                        const int c = 2 * (2 * g + (q4 >> 1)), o = 2 * (q4 & 1);
                        *(h4 *)&as[pb * kG + 4 * swz(c, pb) + o] = sp.hi;
                        *(h4 *)&as[pb * kG + 4 * swz(c + 1, pb) + o] = sp.lo;
                    }
                }
                // ---- the neighbours' edge columns of dA_{t+1} -> halo columns
                // One instruction moves four consecutive rows of a halo
                // column (lane l: chunk position l%16 of row 4 j + l/16);
                // lanes past the last row are inactive, so the halo rows
                // above and below the plane keep their zeros.  The wave then
                // splits what it moved.
                const int nslot = (P + 3) >> 2;
                for (int i = wave; i < 2 * nslot; i += kWaves) {
                    const int side = i >= nslot ? 1 : 0;
                    const int j = i - side * nslot;
                    if ((side ? nb_hi : nb_lo) < 0) continue;
                    const int row = 4 * j + (lane >> 4);
                    const int lcol = side ? TQ + 1 : 0;
                    const int pix = lcol * P2 + 1 + row;
                    const int pc = side ? q1 : q0 - 1;
                    const int boff =
                        ((nplane + row * sp + pc * sq) * kG + (col ^ (pix & 15)) * 4) *
                        (int)sizeof(float);
                    lds_void *dst = (lds_void *)&as[(size_t)(lcol * P2 + 1 + 4 * j) * kG];
                    if (row < P)
                        __builtin_amdgcn_raw_ptr_buffer_load_lds(dA_rs, dst, 16, boff, 0, 0,
                                                                 kCachePolicySC1);
                }
                __builtin_amdgcn_s_waitcnt(kWaitVmcnt0);
                asm volatile("" ::: "memory");
                for (int i = f32 ? 2 * nslot : wave; i < 2 * nslot; i += kWaves) {
                    const int side = i >= nslot ? 1 : 0;
                    const int row = 4 * (i - side * nslot) + (lane >> 3);
                    if ((side ? nb_hi : nb_lo) < 0 || lane >= 32 || row >= P) continue;
                    split_slot((side ? TQ + 1 : 0) * P2 + 1 + row, lane & 7, scale, own ? px_inv : nullptr);
                }
                if (threadIdx.x == 0) {
                    cnt[0] = 0;
                    const int p = 2 * (r & 1);
                    mx[p] = mx[p + 1] = emx[p] = emx[p + 1] = 0u;
                }
                __syncthreads();
            }
#pragma unroll
            for (int it = 0; it < 2; ++it) {
                const int k = wave + it * kWaves;
                hbase[it] = -1;
                if (k < nmt) {
                    const int mt = order[k];
                    const int pa = min(mt * 16 + col, npx - 1);
                    const int ca = fdiv_floor(pa, inv_p), ra = pa - ca * P;
                    // (hidden from the compiler, which would keep every tap's address
                    // of both tiles in registers over the steps: 22 spilled)
                    int base = (ca + 1) * P2 + ra + 1;
                    asm volatile("" : "+v"(base));
                    const int vo = splane + ra * sp + (ca + q0) * sq;
                    const bool shared = is_shared_col(ca + q0);
                    BwdEpi e;
                    const int vop = vo - splane + pplane;
                    e.dh = *(const f4 *)&dh_n[vo * kO + 4 * q4];
                    e.gi = *(const f4 *)&gates_dn[vo * kG + 0 * kO + 4 * q4];
                    e.gf = *(const f4 *)&gates_dn[vo * kG + 1 * kO + 4 * q4];
                    e.gg = *(const f4 *)&gates_dn[vo * kG + 2 * kO + 4 * q4];
                    e.go = *(const f4 *)&gates_dn[vo * kG + 3 * kO + 4 * q4];
                    e.c = r == 0 ? *(const f4 *)&cell_dn[vo * kO + 4 * q4] : carry_c[it];
                    e.gcfn = carry_gcf[it];
                    e.cp = *(const f4 *)&cell_dn[vop * kO + 4 * q4];
                    __builtin_amdgcn_sched_barrier(0);
                    f4 acc = {0.0f, 0.0f, 0.0f, 0.0f};
                    if (has_next) {
                        if (__builtin_expect(f32, 0))
                            acc = contract_bwd_f32(as, was, raw, base, 1, P2, q4, lane);
                        else if (__builtin_expect(own, 0))
                            acc = contract_bwd_own(as, was, px_inv, base, 1, P2, q4, lane);
                        else
                            acc = contract_bwd(as, was, base, 1, P2, q4, lane);
                        acc = acc * inv * *(const f4 *)&winv[4 * q4];
                    }
                    f4 dAi, dAf, dAg, dAo, gcf;
#pragma unroll
                    for (int i = 0; i < 4; ++i) {
                        const float gh = acc[i] + e.dh[i];
                        const float tc = ftanh(e.c[i]);
                        const float gcs = gh * e.go[i] * (1.0f - tc * tc) +
                                          (has_next ? e.gcfn[i] : 0.0f);
                        const float cprev = has_prev ? e.cp[i] : 0.0f;
                        gcf[i] = gcs * e.gf[i];
                        dAi[i] = gcs * e.gg[i] * e.gi[i] * (1.0f - e.gi[i]);
                        dAf[i] = gcs * cprev * e.gf[i] * (1.0f - e.gf[i]);
                        dAg[i] = gcs * e.gi[i] * (1.0f - e.gg[i] * e.gg[i]);
                        dAo[i] = gh * tc * e.go[i] * (1.0f - e.go[i]);
                    }
                    const int o4 = vo * kG + 4 * q4;
                    if (shared) {
                        store_coherent(dA_rs, o4 + 0 * kO, dAi);
                        store_coherent(dA_rs, o4 + 1 * kO, dAf);
                        store_coherent(dA_rs, o4 + 2 * kO, dAg);
                        store_coherent(dA_rs, o4 + 3 * kO, dAo);
                    } else {
                        float *dst = &dA_dn[o4];
                        *(f4 *)&dst[0 * kO] = dAi;
                        *(f4 *)&dst[1 * kO] = dAf;
                        *(f4 *)&dst[2 * kO] = dAg;
                        *(f4 *)&dst[3 * kO] = dAo;
                    }
                    // (beside the stores)
                    const float tm = top_of(dAi, dAf, dAg, dAo);
                    const DaRange tr = da_wave(__float_as_uint(tm));
                    if (lane == 0) {
                        widen(&mx[2 * (r & 1)], tr);
                        if (k < n_edge) widen(&emx[2 * (r & 1)], tr);
                    }
                    carry_gcf[it] = gcf;
                    carry_c[it] = e.cp;
                    hold[it][0] = dAi;
                    hold[it][1] = dAf;
                    hold[it][2] = dAg;
                    hold[it][3] = dAo;
                    hbase[it] = base;
                    if (k < n_edge) {
                        // this edge tile's coherent stores have completed:
                        // count it; the wave that counts the last publishes
                        __builtin_amdgcn_s_waitcnt(kWaitVmcnt0);
                        __threadfence_block();
                        if (lane == 0 && atomicAdd(cnt, 1) == n_edge - 1) {
                            __threadfence_block();
                            publish(r, emx);
                        }
                    }
                }
            }
            // (a strip without neighbours is waited for by none)
        }
        return;
    }

    float *const px_inv = as + (size_t)(chunk_rows + 2) * (a.max_w[d] + 2) * kG;
    for (int r = 0; r < dg.T; ++r) {
        const int t = dg.T - 1 - r;                   // plane processed at this step
        const int s = dg.sign > 0 ? t : dg.T - 1 - t;
        const bool has_next = t + 1 < dg.T, has_prev = t > 0;
        // ---- wait for the neighbours' dA_{t+1} --------------------------
        float scale = 0.0f, inv = 0.0f;
        DaRange wave_range = {0, 0};        // of this wave's tiles
        bool f32 = false, own = false;
        if (r > 0) {
            wait_neighbours(r);
            __syncthreads();
            const DaRange range = step_range(r);
            const int ex = da_exp(range);
            scale = step_sign(r) * exp2i(ex);
            f32 = raw || range.x == 255;
            own = !f32 && da_wide(range);
            inv = f32 || own ? 1.0f : step_sign(r) * exp2i(-ex);
            if (threadIdx.x == 0) mx[2 * (r & 1)] = mx[2 * (r & 1) + 1] = 0u;
            // (ordered before this step's maxima by the chunks' barriers)
        }
        const int splane = s * ss;
        const int nplane = has_next ? (s + dg.sign) * ss : splane;   // in-slice when read
        const int pplane = has_prev ? (s - dg.sign) * ss : splane;
        for (int r0 = 0; r0 < dg.P; r0 += chunk_rows) {
            const int CH = min(chunk_rows, dg.P - r0);
            const int npl = (CH + 2) * W2;
            // ---- stage dA_{t+1} (chunk + halo) straight into LDS ------------
            // Direct-to-LDS buffer loads (no registers, all in flight at
            // once): one instruction moves 4 pixels, lane l the 16-byte chunk
            // at position l%16 of pixel 4 i + l/16, which holds its chunk
            // (l%16) ^ (pixel & 15) (see `swz`).  Off-plane pixels, the halo
            // past the volume and the plane after the last get an
            // out-of-range offset and the hardware writes zeros.
            const int nslots = (npl + 3) >> 2;
            for (int i = wave; i < nslots; i += kWaves) {
                const int pix = 4 * i + (lane >> 4);
                const int chunk = col ^ (pix & 15);
                const int rr = fdiv_floor(pix, inv_w2);
                const int pr = rr + r0 - 1, pc = pix - rr * W2 + q0 - 1;
                const bool ok = has_next & (pr >= 0) & (pr < dg.P) & (pc >= 0) & (pc < dg.Q);
                const int boff =
                    ok ? ((nplane + pr * sp + pc * sq) * kG + chunk * 4) * (int)sizeof(float)
                       : kOutOfRange;
                lds_void *dst = (lds_void *)&as[i * 4 * kG];
                if (pix < npl) {
                    if (is_shared_col(pc))   // read at device coherence (written that way)
                        __builtin_amdgcn_raw_ptr_buffer_load_lds(dA_rs, dst, 16, boff, 0, 0,
                                                                 kCachePolicySC1);
                    else
                        __builtin_amdgcn_raw_ptr_buffer_load_lds(dA_rs, dst, 16, boff, 0, 0, 0);
                }
            }
            __builtin_amdgcn_s_waitcnt(kWaitVmcnt0);
            asm volatile("" ::: "memory");
            // each wave splits the pixels it moved (eight slots a pixel)
            if (has_next && !f32)
                for (int i = wave + (lane >> 5) * kWaves; i < nslots; i += 2 * kWaves) {
                    const int pix = 4 * i + ((lane >> 3) & 3);
                    if (pix < npl) split_slot(pix, lane & 7, scale, own ? px_inv : nullptr);
                }
            __syncthreads();
            // ---- 16-pixel tiles ------------------------------------------
            // Each tile's epilogue operands are loaded before its contraction.
            // Lanes past the chunk redo its last pixel (the same values to
            // the same addresses).
            const int npx = CH * TQ;
            const int nmt = (npx + 15) >> 4;
            auto pixel = [&](int mt, int &base, int &vo, bool &shared) {
                const int pb = min(mt * 16 + col, npx - 1);
                const int rb = fdiv_floor(pb, inv_tq);
                const int cb = pb - rb * TQ;
                base = (rb + 1) * W2 + cb + 1;
                vo = splane + (rb + r0) * sp + (cb + q0) * sq;
                shared = is_shared_col(cb + q0);
            };
            auto load_epi = [&](int vo, BwdEpi &e) {
                const int von = vo - splane + nplane, vop = vo - splane + pplane;
                e.dh = *(const f4 *)&dh_n[vo * kO + 4 * q4];
                e.gi = *(const f4 *)&gates_dn[vo * kG + 0 * kO + 4 * q4];
                e.gf = *(const f4 *)&gates_dn[vo * kG + 1 * kO + 4 * q4];
                e.gg = *(const f4 *)&gates_dn[vo * kG + 2 * kO + 4 * q4];
                e.go = *(const f4 *)&gates_dn[vo * kG + 3 * kO + 4 * q4];
                e.c = *(const f4 *)&cell_dn[vo * kO + 4 * q4];
                e.gcfn = *(const f4 *)&gcf_dn[von * kO + 4 * q4];
                e.cp = *(const f4 *)&cell_dn[vop * kO + 4 * q4];
            };
            auto epilogue = [&](int vo, bool shared, f4 acc, const BwdEpi &e) {
                f4 dAi, dAf, dAg, dAo, gcf;
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    const float gh = acc[i] + e.dh[i];
                    const float tc = ftanh(e.c[i]);
                    const float gcs = gh * e.go[i] * (1.0f - tc * tc) +
                                      (has_next ? e.gcfn[i] : 0.0f);
                    const float cprev = has_prev ? e.cp[i] : 0.0f;
                    gcf[i] = gcs * e.gf[i];
                    dAi[i] = gcs * e.gg[i] * e.gi[i] * (1.0f - e.gi[i]);
                    dAf[i] = gcs * cprev * e.gf[i] * (1.0f - e.gf[i]);
                    dAg[i] = gcs * e.gi[i] * (1.0f - e.gg[i] * e.gg[i]);
                    dAo[i] = gh * tc * e.go[i] * (1.0f - e.go[i]);
                }
                const float tm = top_of(dAi, dAf, dAg, dAo);
                wave_range = da_join(wave_range, da_wave(__float_as_uint(tm)));
                const int o4 = vo * kG + 4 * q4;
                float *dst = &dA_dn[o4];
                if (shared) {
                    store_coherent(dA_rs, o4 + 0 * kO, dAi);
                    store_coherent(dA_rs, o4 + 1 * kO, dAf);
                    store_coherent(dA_rs, o4 + 2 * kO, dAg);
                    store_coherent(dA_rs, o4 + 3 * kO, dAo);
                } else {
                    *(f4 *)&dst[0 * kO] = dAi;
                    *(f4 *)&dst[1 * kO] = dAf;
                    *(f4 *)&dst[2 * kO] = dAg;
                    *(f4 *)&dst[3 * kO] = dAo;
                }
                *(f4 *)&gcf_dn[vo * kO + 4 * q4] = gcf;
            };
            for (int mt = wave; mt < nmt; mt += kWaves) {
                int base, vo;
                bool shared;
                pixel(mt, base, vo, shared);
                BwdEpi e;
                load_epi(vo, e);
                // keep the loads above the contraction (the scheduler would
                // otherwise sink them to their use and expose their latency)
                __builtin_amdgcn_sched_barrier(0);
                f4 acc = {0.0f, 0.0f, 0.0f, 0.0f};
                if (has_next) {
                    if (__builtin_expect(f32, 0))
                        acc = contract_bwd_f32(as, was, raw, base, W2, 1, q4, lane);
                    else if (__builtin_expect(own, 0))
                        acc = contract_bwd_own(as, was, px_inv, base, W2, 1, q4, lane);
                    else
                        acc = contract_bwd(as, was, base, W2, 1, q4, lane);
                    acc = acc * inv * *(const f4 *)&winv[4 * q4];
                }
                epilogue(vo, shared, acc, e);
            }
            __syncthreads();
        }
        // ---- publish dA_t: every wave's coherent stores have completed ---
        if (lane == 0) widen(&mx[2 * (r & 1)], wave_range);
        __builtin_amdgcn_s_waitcnt(kWaitVmcnt0);
        __syncthreads();
        if (threadIdx.x == 0) publish(r, mx);
    }
}

__global__ void k_fill_zero(int *p, int n)
{
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) p[i] = 0;
}

StripCostModel bwd_model(bool allow_resident)
{
    StripCostModel m;
    m.fixed_bytes = kWaFloats * sizeof(float);
    m.px_bytes = (kG + 1) * sizeof(float);        // dA, 1 / scale
    m.c_sync = 3.0;
    m.c_tile = 2.9;         // of the fp32 instruction's 144 a tile; not fitted again for split operands
    m.c_stage0 = 1.0;
    m.c_stage_px = 0.008;
    m.allow_resident = allow_resident;
    m.res_px_bytes = (kG + 1) * sizeof(float);    // dA_{t+1} / dA_t, in place; 1 / scale
    m.res_own_bytes = 1;                          // tile order (4 bytes per 16 pixels)
    m.res_fixed_bytes = 16 * sizeof(int);         // counters
    m.res_max_staged = 1 << 30;
    m.res_max_own = 2 * kWaves * 16;              // two tiles per wave
    m.c_res_step = 2.0;
    return m;
}

}  // namespace

bool sweep_bwd_supported(const Geom &g)
{
    // dA slices are addressed as buffer resources: bytes must fit 32 bits
    return step_supported(g) && g.nd == kDirs && g.KP == 3 && g.KQ == 3 && g.O == kO && g.C >= 1 &&
           g.C <= 4 && g.V * kG * (long long)sizeof(float) < (1LL << 31);
}

size_t sweep_bwd_ws(const Geom &g)
{
    Carve cv(nullptr);
    cv.take<float>((size_t)kDirs * g.N * g.V * kG);                     // dA
    cv.take<float>((size_t)kDirs * g.N * g.V * kO);                     // dL/dc * f
    cv.take<int>(2 * 1024 + 1);                                          // flags + err
    cv.take<char>(step_wgrad_ws(g, true));                               // weight gradients
    cv.take<char>(step_dx_ws(g));                                        // dL/dx fragments
    return cv.off;
}

int sweep_bwd(const Geom &g, const float *x, const float *wx, const float *wh, const Saved &sv,
              const float *dh, float *dx, float *dwx, float *dwh, float *db, void *ws,
              hipStream_t st, bool allow_resident)
{
    const DevInfo di = device_info();
    if (di.cus <= 0) return PLSTM_EHIP;
    const size_t lds_limit = (size_t)(di.max_lds > 0 ? di.max_lds : 65536) - 1024;
    const int budget = di.cus < 1024 ? di.cus : 1024;
    const Plan pl = make_plan(g, budget, bwd_model(allow_resident), lds_limit);
    if (pl.blocks > budget) return PLSTM_EUNSUPPORTED;
    for (int d = 0; d < kDirs; ++d) {
        if (pl.chunk_rows[d] < 1) return PLSTM_EUNSUPPORTED;
        // a resident strip: at most two 16-pixel tiles per wave
        if (pl.resident[d] && (long long)g.dir[d].P * pl.max_w[d] > 2 * kWaves * 16)
            return PLSTM_EUNSUPPORTED;
    }

    Carve cv(ws);
    float *dA = cv.take<float>((size_t)kDirs * g.N * g.V * kG);
    float *gcf = cv.take<float>((size_t)kDirs * g.N * g.V * kO);
    int *flags = cv.take<int>(2 * 1024 + 1);     // (256-byte aligned: 64-bit words)
    void *wgws = cv.take<char>(step_wgrad_ws(g, true));
    float *fragx = (float *)cv.take<char>(step_dx_ws(g));

    BwdArgs args;
    args.g = g;
    args.wh = wh;
    args.gates = sv.gates; args.cell = sv.cell;
    args.dh = dh;
    args.dA = dA; args.gcf = gcf;
    args.flags = (unsigned long long *)flags; args.err = flags + 2 * 1024;
    args.max_spin = g_wait_spin_limit;
    args.wait_bias = g_wait_bias;
    for (int d = 0; d < kDirs; ++d) {
        args.nstrip[d] = pl.nstrip[d];
        args.first[d] = pl.first[d];
        args.chunk_rows[d] = pl.chunk_rows[d];
        args.max_w[d] = pl.max_w[d];
        args.resident[d] = pl.resident[d];
    }
    int per_cu = 0;
    if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, k_sweep_bwd, kThreads, pl.lds) !=
        hipSuccess)
        return PLSTM_EHIP;
    if ((long long)per_cu * di.cus < pl.blocks) return PLSTM_ENOTCORESIDENT;
    (void)hipFuncSetAttribute((const void *)k_sweep_bwd,
                              hipFuncAttributeMaxDynamicSharedMemorySize, (int)pl.lds);

    k_fill_zero<<<(2049 + 255) / 256, 256, 0, st>>>(flags, 2049);
    PLSTM_LAUNCH_CHECK();
    timing_begin("sweep_bwd_mfma", st);
    void *kargs[] = {&args};
    if (hipLaunchCooperativeKernel((const void *)k_sweep_bwd, dim3(pl.blocks), dim3(kThreads),
                                   kargs, pl.lds, st) != hipSuccess)
        return PLSTM_EHIP;
    timing_end(1, st);

    int rc = step_wgrad(g, x, sv.hd, dA, gcf, wgws, dwx, dwh, db, "wgrad_mfma", st);
    if (rc != PLSTM_OK) return rc;
    if (dx) {
        rc = step_dx(g, wx, dA, fragx, dx, st);
        if (rc != PLSTM_OK) return rc;
    }
    PoisonList poison;
    poison.ptr[0] = dwx; poison.count[0] = (long long)kDirs * kG * g.C * 9;
    poison.ptr[1] = dwh; poison.count[1] = (long long)kDirs * kG * kO * 9;
    poison.ptr[2] = db;  poison.count[2] = (long long)kDirs * kG;
    poison.ptr[3] = dx;  poison.count[3] = dx ? (long long)g.N * g.V * g.C : 0;
    return wait_check(args.err, poison, st);
}

}  // namespace plstm
