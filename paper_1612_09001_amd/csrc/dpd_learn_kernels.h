// The passes of the coefficient-learning step over one template: the
// predistorter (Eq. 1 / Algorithm 1), the two-stage transmitter model (A
// memoryless with order 1 in each branch, B with orders {1,3,5} and three
// taps), the loss, the transmitter's adjoint and the predistorter's coefficient
// gradient
//     dE/dM_{j,k}[r][c] = sum_m G_{m+k}[r] (s_m^j v_m)[c],   G = dE/dz,
// with v_m = (Re x_m, Im x_m), s_m = |x_m|^2.
//   kLnFwd   x -> z, E, dE/dy
//   kLnBwd   x, z, dE/dy -> coefficient gradient (and dE/dz)
//   kLnBoth  x -> z, E, dE/dy and the coefficient gradient: nothing but x is read
// On rows of whole 256s all three walk the data in the same way and use the same
// arithmetic in the same order, so kLnBoth gives the bits of the other two.
//
// What bounds it: VALU issue (336 instructions per sample against 24
// bytes), so every value is computed once and the two passes as one save the
// second pass's loads, staging and stage A.  Measured on 64 rows of 2^18 samples
// (a whole step with its finalisation): NI = 4, L = 6 144 us, NI = 4, L = 8 163, NI =
// 2, L = 2 94; as two calls of 24 bytes per sample each 185, 203 and 154 us.  Rows that
// are not whole 256s (16 x 40001, L = 6): 39 us.
//
// Each wave takes a contiguous run of chunks of 64 S samples of the flattened rows
// and walks it forward.  Lane l filters S samples S l .. S l + S - 1 of a chunk; z
// and dE/dy at the two samples before them, which stage B's memory needs, come from
// lane l - 1 by a DPP shift, for lane 0 from lane 63 of the chunk before.  The
// adjoint looks ahead, so it trails: G needs dE/dy two samples on and is formed
// for samples S l - 2 .. S l + S - 3; the gradient needs G up to L - 1 samples on
// and takes the basis at S l - (L + 1) + 0 .. S - 1, with G through LDS (its first L
// - 1 values are the last of the chunk before).  A row's last chunk is followed by
// the L + 1 samples still open, with zeros past the row end.  A run that starts
// inside a row evaluates the L + 3 samples before it directly, one per lane.
// Samples past a row's end are zeros in x and contribute nothing (dE/dy = 0).
//
// The per-lane FP32 sums of the gradient cover at most 128 samples, are added up
// over the wave in FP32 and go to its FP64 totals; for rows at odd 8-byte starts or
// strides ("fine", as in dpd_backward) they cover at most 64 samples, one per 2^18
// of the input but at least a chunk's, and are added up in FP64 (inputs so short that
// a chunk's are too many go through dE/dz to bwd_dc_short_kernel).  Loss and gradient
// leave as FP32 partials, one per block.
#pragma once

#include "dpd_bwd_kernels.h"
#include "dpd_cascade.h"
#include "dpd_fwd_kernels.h"
#include "dpd_table.h"

namespace dpd {

constexpr int kLnNIB = 3, kLnLB = 3;     // stage B: orders {1,3,5}, 3 taps
constexpr int kLnMaxNI = 5;              // predistorter: orders up to 9
constexpr int kLnMaxL = kSpecL;          // predistorter: up to 8 taps
constexpr int kLnFlush = 128;            // samples per FP32 gradient sum of a lane (at most)
enum { kLnFwd = 0, kLnBwd = 1, kLnBoth = 2, kLnModes = 3 };
// Walks: four samples per lane (chunks of 256) or eight, rows of whole chunks or
// of any length.
enum { kLn4 = 0, kLn4Any = 1, kLn8 = 2, kLn8Any = 3, kLnWalks = 4 };
constexpr int ln_s(int walk) { return walk < kLn8 ? 4 : 8; }

struct LnParams {
    const float *M;          // predistorter table (used when raw is null)
    const float2 *raw;       // or the K raw coefficients, precombined by every block
    CoefMap map;
    const float *A, *B;      // transmitter stage tables
    const float2 *x;         // rows x n at stride ld
    float2 *z, *gy;          // same layout: written, or read by kLnBwd
    float2 *gz;              // kLnBwd: dE/dz out (nullptr: not written)
    float *lpart;            // loss partials, one per block (two where a run has two parts)
    float *gpart;            // gradient partials, [block][4 L NI + 2]
    int64_t rows, n, ld;
    int64_t tpr;             // chunks per row
    float scale, gscale;
    int32_t flush;           // samples that a lane's FP32 gradient sums cover at most
    int32_t fine;            // kLnBwd: the sums over a wave's lanes in FP64 (else FP32)
    int32_t *step;           // learning-step counter advanced by one (nullptr: none)
};

typedef hipError_t (*LnLaunch)(const LnParams &, hipStream_t, int grid);
struct LnTable {
    LnLaunch fn[kLnMaxNI][kLnMaxL][kLnWalks][kLnModes];   // nullptr: not built
};
void register_learn_ni1(LnTable &);
void register_learn_ni2(LnTable &);
void register_learn_ni3(LnTable &);
void register_learn_ni4(LnTable &);
void register_learn_ni5(LnTable &);

// lane l receives v of lane l - 1; lane 0 receives `first` (wave-uniform)
__device__ __forceinline__ float shift_up(float v, float first)
{
    return __int_as_float(__builtin_amdgcn_update_dpp(__float_as_int(first), __float_as_int(v), 0x138, 0xf, 0xf, false));
}
// lane l receives v of lane l + 1; lane 63 receives 0
__device__ __forceinline__ float shift_down(float v)
{
    return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), 0x130, 0xf, 0xf, false));
}
__device__ __forceinline__ float lane_of(float v, int l)
{
    return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), l));
}

// Stage A at one power level: u = c + M0 z.
__device__ __forceinline__ float2 ln_stage_a(const float (&ta)[6], float zr, float zi)
{
    return make_float2(__builtin_fmaf(ta[0], zr, __builtin_fmaf(ta[1], zi, ta[4])),
                       __builtin_fmaf(ta[2], zr, __builtin_fmaf(ta[3], zi, ta[5])));
}

// Stage B's output at a sample from u[0..LB-1] (oldest first) and |u|^2.
__device__ __forceinline__ float2 ln_stage_b(const float *tb, const float2 *u, const float *su)
{
    constexpr int NIB = kLnNIB, LB = kLnLB;
    float yr = tb[4 * LB * NIB], yi = tb[4 * LB * NIB + 1];
#pragma unroll
    for (int k = 0; k < LB; ++k) {
        const int w = LB - 1 - k;
        const float *t = tb + 4 * NIB * k;
        float w00 = t[4 * (NIB - 1)], w01 = t[4 * (NIB - 1) + 1];
        float w10 = t[4 * (NIB - 1) + 2], w11 = t[4 * (NIB - 1) + 3];
#pragma unroll
        for (int j = NIB - 2; j >= 0; --j) {
            w00 = __builtin_fmaf(w00, su[w], t[4 * j + 0]);
            w01 = __builtin_fmaf(w01, su[w], t[4 * j + 1]);
            w10 = __builtin_fmaf(w10, su[w], t[4 * j + 2]);
            w11 = __builtin_fmaf(w11, su[w], t[4 * j + 3]);
        }
        yr = __builtin_fmaf(w00, u[w].x, __builtin_fmaf(w01, u[w].y, yr));
        yi = __builtin_fmaf(w10, u[w].x, __builtin_fmaf(w11, u[w].y, yi));
    }
    return make_float2(yr, yi);
}

// dE/dz at a sample from u = A(z) there and dE/dy at it and the LB - 1 after:
// the arithmetic of dpd_cascade_backward at one level of A.
__device__ __forceinline__ float2 ln_adjoint(const float (&ta)[6], const float *tb, float2 u, const float2 *g)
{
    const float2 gu = cas_b_adjoint<kLnNIB, kLnLB>(tb, g, u);
    return make_float2(__builtin_fmaf(ta[0], gu.x, ta[2] * gu.y), __builtin_fmaf(ta[1], gu.x, ta[3] * gu.y));
}

// dE/dM and dE/dc of N samples per lane: G at each and the L - 1 after (ga, gb)
// against the basis (va, vb, |v|^2).
template <int NI, int L, int N>
__device__ __forceinline__ void ln_accumulate(float (&acc)[4 * L * NI + 2], const float (&ga)[N + L - 1],
                                              const float (&gb)[N + L - 1], const float (&va)[N], const float (&vb)[N])
{
    constexpr int E = 4 * L * NI + 2;
    float sq[N], pw[N];
#pragma unroll
    for (int i = 0; i < N; ++i) {
        sq[i] = __builtin_fmaf(va[i], va[i], vb[i] * vb[i]);
        pw[i] = 1.f;
    }
#pragma unroll
    for (int j = 0; j < NI; ++j) {
        float ba[N], bb[N];
#pragma unroll
        for (int i = 0; i < N; ++i) {
            ba[i] = j == 0 ? va[i] : pw[i] * va[i];
            bb[i] = j == 0 ? vb[i] : pw[i] * vb[i];
        }
#pragma unroll
        for (int k = 0; k < L; ++k) {
#pragma unroll
            for (int i = 0; i < N; ++i) {
                const float a = ga[i + k], b = gb[i + k];
                float *u = &acc[4 * (k * NI + j)];
                u[0] = __builtin_fmaf(a, ba[i], u[0]);
                u[1] = __builtin_fmaf(a, bb[i], u[1]);
                u[2] = __builtin_fmaf(b, ba[i], u[2]);
                u[3] = __builtin_fmaf(b, bb[i], u[3]);
            }
        }
#pragma unroll
        for (int i = 0; i < N; ++i) pw[i] = j == 0 ? sq[i] : pw[i] * sq[i];
        // one level at a time (the empty asm statements consume its sums), so
        // that only its basis is in registers
#pragma unroll
        for (int k = 0; k < L; ++k)
#pragma unroll
            for (int q = 0; q < 4; ++q) asm volatile("" ::"v"(acc[4 * (k * NI + j) + q]));
        __builtin_amdgcn_sched_barrier(0);
    }
#pragma unroll
    for (int i = 0; i < N; ++i) {
        acc[E - 2] += ga[i];
        acc[E - 1] += gb[i];
    }
}

// Blocks per CU the registers are held to: two, one where the gradient's
// accumulators alone take more than half of 256 (the step at NI = 5, L = 7, 142
// accumulators, 64 rows of 2^18: 286 us with two, spilling, and 237 with one).  With
// four samples per lane nothing spills up to 130, but for one register in the
// backward pass at NI = 5, L = 6.
constexpr int ln_blocks(int mode, int E) { return mode == kLnFwd || E <= 130 ? 2 : 1; }

// Where the gradient leaves one block per CU, a run of the one pass on rows of whole
// chunks has two parts for the loss, each with sums of its own, and the forward pass
// gives the second part to another wave: two blocks per CU, and the same bits (64
// rows of 2^18 at NI = 5, L = 7: 123 us with one, 92 with two).
constexpr bool ln_parts(int E, int walk) { return ln_blocks(kLnBoth, E) == 1 && (walk == kLn4 || walk == kLn8); }

template <int NI, int L, int MODE, int WALK>
__global__ void __launch_bounds__(kBlock, ln_blocks(MODE, 4 * L * NI + 2)) learn_kernel(LnParams p)
{
    constexpr bool RAGGED = WALK == kLn8Any || WALK == kLn4Any;
    constexpr bool FWD = MODE != kLnBwd, GRAD = MODE != kLnFwd, READ = MODE == kLnBwd;
    constexpr int LB = kLnLB, NB = 4 * kLnLB * kLnNIB + 2;
    static_assert(LB == 3, "two samples are handed on between lanes and chunks");
    constexpr int S = ln_s(WALK), C = 64 * S, NV = S / 2, WAVES = kBlock / 64;
    constexpr int D = L + 1;                         // samples the gradient trails
    constexpr int HX = GRAD ? D : L - 1;             // samples of x before the chunk
    using PL = PadLayout<HX + 1, S>;
    constexpr int W = S + L - 1;
    constexpr int NC = 4 * L * NI + 2, E = NC;
    constexpr int OSLOTS = C + L - 1 + (C + L - 1) / S + 1;
    __shared__ __align__(16) float mtab[FWD ? NC + 2 : 1];
    __shared__ __align__(16) float2 xs[WAVES][PL::SLOTS];
    __shared__ __align__(16) float ss[WAVES][FWD ? PL::SLOTS : 1];
    __shared__ __align__(16) float2 os[WAVES][OSLOTS];          // outputs on their way out, then G
    __shared__ __align__(16) float2 ys[WAVES][READ ? C + C / S : 1];
    __shared__ double red[GRAD ? WAVES * E : WAVES];

    const int tid = threadIdx.x, lane = tid & 63;
    const int wv = __builtin_amdgcn_readfirstlane(tid >> 6);
    if constexpr (FWD) {
        for (int e = tid; e < NC; e += kBlock) mtab[e] = table_entry(p.M, p.raw, p.map, e);
        __syncthreads();
    }
    // the stage tables: wave-uniform (scalar) operands
    float ta[6], tb[NB];
#pragma unroll
    for (int e = 0; e < 6; ++e) ta[e] = p.A[e];
#pragma unroll
    for (int e = 0; e < NB; ++e) tb[e] = p.B[e];
    float2 *X = xs[wv], *O = os[wv], *Y = ys[wv];
    float *SX = ss[wv];
    const auto oslot = [](int d) { return d + d / S; };

    float acc[GRAD ? E : 1];
    constexpr int NGT = GRAD ? (E + 63) / 64 : 1;
    double tot[NGT];   // FP64 totals, entry 64 g + l in lane l of tot[g]
#pragma unroll
    for (int e = 0; e < (GRAD ? E : 1); ++e) acc[e] = 0.f;
#pragma unroll
    for (int g = 0; g < NGT; ++g) tot[g] = 0.0;
    const auto flush = [&]() {
        if constexpr (GRAD) {
            if (READ && p.fine)
                wave_sums_into<double, E>(acc, tot, lane);
            else
                wave_sums_into<float, E>(acc, tot, lane);
#pragma unroll
            for (int e = 0; e < E; ++e) acc[e] = 0.f;
        }
    };
    LossSum ls;

    const int64_t total = p.rows * p.tpr;
    constexpr bool PARTS = FWD && ln_parts(E, WALK);
    constexpr bool APART = PARTS && !GRAD;   // a wave takes one part of a run
    const int64_t block = xcd_remap(blockIdx.x, gridDim.x);
    const int64_t nw = (int64_t)gridDim.x * WAVES / (APART ? 2 : 1);
    const int64_t gw = (block * WAVES + wv) / (APART ? 2 : 1);
    const int64_t per = (total + nw - 1) / nw, part = (per + 1) / 2;
    int64_t c_begin = gw * per < total ? gw * per : total;
    int64_t c_end = c_begin + per < total ? c_begin + per : total;
    if constexpr (APART) {
        const int64_t mid = c_begin + part < c_end ? c_begin + part : c_end;
        if (wv & 1)
            c_begin = mid;
        else
            c_end = mid;
    }
    double first = 0.0;   // the loss of the run's first part
    // the learning step's counter (read by the finalisation launch after this one)
    if (p.step != nullptr && blockIdx.x == 0 && tid == 0) *p.step += 1;

    struct Regs {
        v4f_s x[NV];
        v4f_s z[READ ? NV : 1], y[READ ? NV : 1];
        float2 h;   // x at t0 - HX + lane (lanes < HX; replaced by zero at a row start)
    };
    // samples [t0, t0 + C) of a row buffer, lane l, part i: 2 (l + 64 i) on
    const auto load16 = [&](v4f_s(&r)[NV], const float2 *row, int64_t t0) {
        if (!RAGGED || t0 + C <= p.n) {
            const v4f_s *q = reinterpret_cast<const v4f_s *>(row + t0);
#pragma unroll
            for (int i = 0; i < NV; ++i) r[i] = __builtin_nontemporal_load(q + lane + 64 * i);
        } else {
#pragma unroll
            for (int i = 0; i < NV; ++i) {
                const int64_t m = t0 + 2 * (lane + 64 * i);
                const float2 a = m < p.n ? row[m] : make_float2(0.f, 0.f);
                const float2 b = m + 1 < p.n ? row[m + 1] : make_float2(0.f, 0.f);
                r[i] = v4f_s{a.x, a.y, b.x, b.y};
            }
        }
    };
    const auto load = [&](Regs &R, int64_t row, int64_t t0) {
        __builtin_amdgcn_s_setprio(2);   // the prefetch at raised wave priority
        const int64_t base = row * p.ld;
        load16(R.x, p.x + base, t0);
        if constexpr (READ) {
            load16(R.z, p.z + base, t0);
            load16(R.y, p.gy + base, t0);
        }
        if constexpr (HX > 0) {
            const int64_t m = t0 - HX + (lane < HX ? lane : HX - 1);
            R.h = p.x[base + (t0 > 0 ? m : 0)];
        }
        __builtin_amdgcn_s_setprio(0);
    };
    const auto put16 = [&](float2 *dst, int off, const v4f_s(&r)[NV]) {
#pragma unroll
        for (int i = 0; i < NV; ++i) {
            const int j = 2 * (lane + 64 * i);
            const int q = off + j + j / S;
            dst[q] = make_float2(r[i].x, r[i].y);
            dst[q + 1] = make_float2(r[i].z, r[i].w);
        }
    };
    const auto stage = [&](const Regs &R, int64_t t0) {
        wave_lds_order();   // the previous chunk's LDS reads are done
        if (HX > 0 && lane < HX) {
            const float2 h = t0 > 0 ? R.h : make_float2(0.f, 0.f);
            const int q = PL::slot(lane - HX);
            X[q] = h;
            if constexpr (FWD) SX[q] = __builtin_fmaf(h.x, h.x, h.y * h.y);
        }
        put16(X, PL::OFF, R.x);
        if constexpr (FWD) {
#pragma unroll
            for (int i = 0; i < NV; ++i) {
                const v4f_s v = R.x[i];
                const int j = 2 * (lane + 64 * i);
                const int q = PL::OFF + j + j / S;
                SX[q] = __builtin_fmaf(v.x, v.x, v.y * v.y);
                SX[q + 1] = __builtin_fmaf(v.z, v.z, v.w * v.w);
            }
        }
        if constexpr (READ) {
            put16(O, 0, R.z);
            put16(Y, 0, R.y);
        }
        wave_lds_order();
    };
    // eight values per lane out through LDS: every store instruction writes 1 KiB
    const auto store = [&](float2 *row, int64_t t0, const float (&a)[S], const float (&b)[S]) {
        wave_lds_order();
#pragma unroll
        for (int i = 0; i < S; ++i) O[lane * (S + 1) + i] = make_float2(a[i], b[i]);
        wave_lds_order();
        v4f_s *q = reinterpret_cast<v4f_s *>(row + t0);
#pragma unroll
        for (int i = 0; i < NV; ++i) {
            const int j = 2 * (lane + 64 * i);
            const float2 u = O[oslot(j)], w = O[oslot(j) + 1];
            if (!RAGGED || t0 + j + 1 < p.n)
                __builtin_nontemporal_store(v4f_s{u.x, u.y, w.x, w.y}, q + lane + 64 * i);
            else if (t0 + j < p.n)
                row[t0 + j] = u;
        }
    };

    // z and dE/dy at the two samples before the chunk (wave-uniform: re, im at
    // t0 - 2, then at t0 - 1), and G at t0 - D + lane (lanes < L - 1)
    float cz[4] = {0.f, 0.f, 0.f, 0.f}, cg[4] = {0.f, 0.f, 0.f, 0.f};
    float2 carry = make_float2(0.f, 0.f);
    int held = 0;   // samples in the FP32 sums

    // the samples before a run that starts inside a row, one per lane: lane j
    // (< L + 3) takes t0 - (L + 3) + j
    const auto before = [&](int64_t row, int64_t t0) {
        const int64_t m = t0 - (L + 3) + (lane < L + 3 ? lane : L + 2);
        const float2 *xr = p.x + row * p.ld;
        float zr, zi, gr = 0.f, gi = 0.f;
        float2 u;
        if constexpr (FWD) {
            float a[L], b[L], sv[L];
#pragma unroll
            for (int w = 0; w < L; ++w) {
                const float2 v = xr[m - (L - 1) + w];
                a[w] = v.x;
                b[w] = v.y;
                sv[w] = __builtin_fmaf(v.x, v.x, v.y * v.y);
            }
            float z1[1], z2[1];
            fir_outputs_lds<NI, L, 1>(a, b, sv, mtab, z1, z2);
            zr = z1[0];
            zi = z2[0];
            u = ln_stage_a(ta, zr, zi);
            float2 uw[LB];
            float su[LB];
            uw[2] = u;
            uw[1] = make_float2(shift_up(u.x, 0.f), shift_up(u.y, 0.f));
            uw[0] = make_float2(shift_up(uw[1].x, 0.f), shift_up(uw[1].y, 0.f));
#pragma unroll
            for (int w = 0; w < LB; ++w) su[w] = __builtin_fmaf(uw[w].x, uw[w].x, uw[w].y * uw[w].y);
            const float2 y = ln_stage_b(tb, uw, su);
            gr = p.gscale * __builtin_fmaf(p.scale, y.x, -a[L - 1]);
            gi = p.gscale * __builtin_fmaf(p.scale, y.y, -b[L - 1]);
        } else {
            const float2 zv = p.z[row * p.ld + m], gv = p.gy[row * p.ld + m];
            zr = zv.x;
            zi = zv.y;
            gr = gv.x;
            gi = gv.y;
            u = ln_stage_a(ta, zr, zi);
        }
        cz[0] = lane_of(zr, L + 1);
        cz[1] = lane_of(zi, L + 1);
        cz[2] = lane_of(zr, L + 2);
        cz[3] = lane_of(zi, L + 2);
        cg[0] = lane_of(gr, L + 1);
        cg[1] = lane_of(gi, L + 1);
        cg[2] = lane_of(gr, L + 2);
        cg[3] = lane_of(gi, L + 2);
        if constexpr (GRAD && L > 1) {
            float2 g[LB];
            g[0] = make_float2(gr, gi);
            g[1] = make_float2(shift_down(g[0].x), shift_down(g[0].y));
            g[2] = make_float2(shift_down(g[1].x), shift_down(g[1].y));
            const float2 G = ln_adjoint(ta, tb, u, g);   // lane j: at t0 - (L + 3) + j
            carry = make_float2(shift_down(shift_down(G.x)), shift_down(shift_down(G.y)));
        }
    };

    // one staged chunk
    const auto compute = [&](int64_t row, int64_t t0, bool last) {
        const int64_t base = row * p.ld;
        if constexpr (GRAD) {
            const int more = S + (last ? 1 : 0);
            if (held + more > p.flush) {
                flush();
                held = 0;
            }
            held += more;
        }
        float zr[S], zi[S], gr[S], gi[S];
        constexpr int ZW = S + LB - 1;
        float2 uu[ZW];   // u at 8l - 2 ..
        if constexpr (FWD) {
            float a[W], b[W], sw[W];
#pragma unroll
            for (int w = 0; w < W; ++w) {
                const int q = lane * (S + 1) + PL::slot(w - (L - 1));
                const float2 v = X[q];
                a[w] = v.x;
                b[w] = v.y;
                sw[w] = SX[q];
            }
            // an opaque zero keeps the table reads inside the chunk loop
            int zo = 0;
            asm volatile("" : "+v"(zo));
            fir_outputs_lds<NI, L, S>(a, b, sw, mtab + zo, zr, zi);
        } else {
            // the two samples that the next lane needs; the others are read when
            // their turn comes
#pragma unroll
            for (int i = S - 2; i < S; ++i) {
                const float2 v = O[lane * (S + 1) + i], g = Y[lane * (S + 1) + i];
                zr[i] = v.x;
                zi[i] = v.y;
                gr[i] = g.x;
                gi[i] = g.y;
            }
        }
        __builtin_amdgcn_sched_barrier(0);
        float zh[4], gh[4];   // z, dE/dy at the two samples before the lane's
        zh[0] = shift_up(zr[S - 2], cz[0]);
        zh[1] = shift_up(zi[S - 2], cz[1]);
        zh[2] = shift_up(zr[S - 1], cz[2]);
        zh[3] = shift_up(zi[S - 1], cz[3]);
        cz[0] = lane_of(zr[S - 2], 63);
        cz[1] = lane_of(zi[S - 2], 63);
        cz[2] = lane_of(zr[S - 1], 63);
        cz[3] = lane_of(zi[S - 1], 63);
        if constexpr (FWD) {
#pragma unroll
            for (int w = 0; w < ZW; ++w) {
                const float2 u = w < LB - 1 ? ln_stage_a(ta, zh[2 * w], zh[2 * w + 1])
                                            : ln_stage_a(ta, zr[w - (LB - 1)], zi[w - (LB - 1)]);
                // stage B sees zeros before the row start
                const bool none = t0 == 0 && lane == 0 && w < LB - 1;
                uu[w] = none ? make_float2(0.f, 0.f) : u;
            }
            __builtin_amdgcn_sched_barrier(0);
            float su[ZW];
#pragma unroll
            for (int w = 0; w < ZW; ++w) su[w] = __builtin_fmaf(uu[w].x, uu[w].x, uu[w].y * uu[w].y);
#pragma unroll
            for (int i = 0; i < S; ++i) {
                const float2 y = ln_stage_b(tb, uu + i, su + i);
                const float2 v = X[lane * (S + 1) + PL::OFF + i];
                const bool in = !RAGGED || t0 + lane * S + i < p.n;
                const float rr = in ? __builtin_fmaf(p.scale, y.x, -v.x) : 0.f;
                const float ri = in ? __builtin_fmaf(p.scale, y.y, -v.y) : 0.f;
                ls.f = __builtin_fmaf(rr, rr, __builtin_fmaf(ri, ri, ls.f));
                gr[i] = p.gscale * rr;
                gi[i] = p.gscale * ri;
            }
            ls.step_done();
            store(p.z + base, t0, zr, zi);
            store(p.gy + base, t0, gr, gi);
        }
        if constexpr (GRAD) {
            gh[0] = shift_up(gr[S - 2], cg[0]);
            gh[1] = shift_up(gi[S - 2], cg[1]);
            gh[2] = shift_up(gr[S - 1], cg[2]);
            gh[3] = shift_up(gi[S - 1], cg[3]);
            cg[0] = lane_of(gr[S - 2], 63);
            cg[1] = lane_of(gi[S - 2], 63);
            cg[2] = lane_of(gr[S - 1], 63);
            cg[3] = lane_of(gi[S - 1], 63);
            __builtin_amdgcn_sched_barrier(0);
            // kLnBwd, whose three prefetched streams leave few registers, takes four
            // samples at a time, z and dE/dy from LDS
            constexpr int NG = READ ? 4 : S;
            float2 G[S];
#pragma unroll
            for (int i0 = 0; i0 < S; i0 += NG) {
                float2 g[NG + LB - 1];
#pragma unroll
                for (int w = 0; w < NG + LB - 1; ++w) {
                    const int m = i0 + w - (LB - 1);
                    g[w] = m < 0  ? make_float2(gh[2 * (m + LB - 1)], gh[2 * (m + LB - 1) + 1])
                           : READ ? Y[lane * (S + 1) + m]
                                  : make_float2(gr[m], gi[m]);
                }
#pragma unroll
                for (int i = 0; i < NG; ++i) {
                    const int m = i0 + i - (LB - 1);
                    float2 u;
                    if constexpr (READ) {
                        const float2 v = m < 0 ? make_float2(zh[2 * (m + LB - 1)], zh[2 * (m + LB - 1) + 1])
                                               : O[lane * (S + 1) + m];
                        u = ln_stage_a(ta, v.x, v.y);
                    } else {
                        u = uu[i0 + i];
                    }
                    const float2 v = ln_adjoint(ta, tb, u, g + i);
                    const bool none = t0 == 0 && lane == 0 && m < 0;   // before the row
                    G[i0 + i] = none ? make_float2(0.f, 0.f) : v;
                }
                if constexpr (READ) {
#pragma unroll
                    for (int i = 0; i < NG; ++i) asm volatile("" ::"v"(G[i0 + i].x), "v"(G[i0 + i].y));
                    __builtin_amdgcn_sched_barrier(0);
                }
            }
            // G into LDS: slot q is sample t0 - D + q
            wave_lds_order();
#pragma unroll
            for (int i = 0; i < S; ++i) O[oslot(L - 1 + i) + lane * (S + 1)] = G[i];
            if (L > 1 && lane < L - 1) O[oslot(lane)] = carry;
            wave_lds_order();
            if constexpr (L > 1) {
                const float2 v = O[oslot(C + (lane < L - 1 ? lane : 0))];
                carry = lane < L - 1 ? v : make_float2(0.f, 0.f);
            }
            if (READ && p.gz != nullptr) {
                float2 *gzr = p.gz + base;
#pragma unroll
                for (int i = 0; i < NV; ++i) {
                    const int j = 2 * (lane + 64 * i);
                    const int64_t m = t0 - (LB - 1) + j;
                    const float2 u = O[oslot(L - 1 + j)], w = O[oslot(L + j)];
                    if (m >= 0 && (!RAGGED || m + 1 < p.n))
                        __builtin_nontemporal_store(v4f_s{u.x, u.y, w.x, w.y}, reinterpret_cast<v4f_s *>(gzr + m));
                    else if (RAGGED && m >= 0 && m < p.n)
                        gzr[m] = u;
                }
            }
            // kLnBwd two samples at a time, for its registers (the sums come in the
            // same order whatever the piece; NI = 4, L = 6, 64 rows of 2^18: 97 us, four
            // at a time 109)
            constexpr int NA = READ ? 2 : S;
#pragma unroll
            for (int i0 = 0; i0 < S; i0 += NA) {
                float ga[NA + L - 1], gb[NA + L - 1], va[NA], vb[NA];
#pragma unroll
                for (int w = 0; w < NA + L - 1; ++w) {
                    const float2 v = O[oslot(i0 + w) + lane * (S + 1)];
                    ga[w] = v.x;
                    gb[w] = v.y;
                }
#pragma unroll
                for (int i = 0; i < NA; ++i) {
                    const float2 v = X[lane * (S + 1) + PL::slot(i0 + i - D)];
                    va[i] = v.x;
                    vb[i] = v.y;
                }
                ln_accumulate<NI, L, NA>(acc, ga, gb, va, vb);
            }
            if (last) {
                // the row's last D samples, one per lane, with the two values of
                // G that needed dE/dy past the row end (zero)
                const int e = lane - (L - 1);
                float2 gt[LB];
                gt[0] = e == 0 ? make_float2(cg[0], cg[1]) : e == 1 ? make_float2(cg[2], cg[3]) : make_float2(0.f, 0.f);
                gt[1] = e == 0 ? make_float2(cg[2], cg[3]) : make_float2(0.f, 0.f);
                gt[2] = make_float2(0.f, 0.f);
                const float2 ut = e == 0 ? ln_stage_a(ta, cz[0], cz[1]) : ln_stage_a(ta, cz[2], cz[3]);
                const float2 v = ln_adjoint(ta, tb, ut, gt);
                if (READ && p.gz != nullptr) {
                    const int64_t m = t0 + C - (LB - 1) + e;
                    if ((e == 0 || e == 1) && (!RAGGED || m < p.n)) p.gz[base + m] = v;
                }
                wave_lds_order();
                O[lane] = lane < L - 1 ? carry : e < LB - 1 ? v : make_float2(0.f, 0.f);
                wave_lds_order();
                float ga[L], gb[L], va[1], vb[1];
                const bool own = lane < D;
#pragma unroll
                for (int w = 0; w < L; ++w) {
                    const float2 q = O[(own ? lane : 0) + w];
                    ga[w] = own ? q.x : 0.f;
                    gb[w] = own ? q.y : 0.f;
                }
                const int d = C - D + (own ? lane : 0);
                const float2 q = X[PL::OFF + d + d / S];
                va[0] = q.x;
                vb[0] = q.y;
                ln_accumulate<NI, L, 1>(acc, ga, gb, va, vb);
            }
        }
        if (last) {
            carry = make_float2(0.f, 0.f);
#pragma unroll
            for (int e = 0; e < 4; ++e) cz[e] = cg[e] = 0.f;
        }
    };

    if (c_begin < c_end) {
        int64_t row = c_begin / p.tpr, k = c_begin - (c_begin / p.tpr) * p.tpr;
        Regs R;
        load(R, row, k * C);
        if (k > 0) before(row, k * C);
        stage(R, k * C);
        for (int64_t left = c_end - c_begin; left > 0; --left) {
            const int64_t crow = row, ck = k;
            if (++k == p.tpr) {
                k = 0;
                ++row;
            }
            if (left > 1) load(R, row, k * C);
            if constexpr (PARTS && !APART) {
                if (c_end - left == c_begin + part) {
                    first = ls.total();
                    ls = LossSum();
                }
            }
            compute(crow, ck * C, ck == p.tpr - 1);
            if (left > 1) stage(R, k * C);
        }
    }

    // wave -> block: one FP32 partial of the loss and of each gradient entry, in
    // fixed order, FP64
    if constexpr (FWD) {
        const auto all = [](double t) {
#pragma unroll
            for (int off = 32; off >= 1; off >>= 1) t += __shfl_xor(t, off, 64);
            return t;
        };
        constexpr int NP = PARTS && !APART ? 2 : 1;   // partials of this block
        if constexpr (NP == 2) {
            const bool whole = c_begin + part >= c_end;   // no second part
            const double t0 = all(whole ? ls.total() : first), t1 = all(whole ? 0.0 : ls.total());
            if (lane == 0) {
                red[2 * wv] = t0;
                red[2 * wv + 1] = t1;
            }
        } else {
            const double t = all(ls.total());
            if (lane == 0) red[wv] = t;
        }
        __syncthreads();
        if (tid < NP) {
            double u = red[WAVES * tid];
#pragma unroll
            for (int w = 1; w < WAVES; ++w) u += red[WAVES * tid + w];
            p.lpart[(PARTS ? block : blockIdx.x) * NP + tid] = (float)u;
        }
        __syncthreads();
    }
    if constexpr (GRAD) {
        flush();
#pragma unroll
        for (int g = 0; g < NGT; ++g)
            if (64 * g + lane < E) red[wv * E + 64 * g + lane] = tot[g];
        __syncthreads();
        for (int e = tid; e < E; e += kBlock) {
            double t = 0.0;
#pragma unroll
            for (int w = 0; w < WAVES; ++w) t += red[w * E + e];
            p.gpart[(int64_t)blockIdx.x * E + e] = (float)t;
        }
    }
}

template <int NI, int L, int MODE, int WALK>
hipError_t launch_learn(const LnParams &p, hipStream_t stream, int grid)
{
    hipLaunchKernelGGL((learn_kernel<NI, L, MODE, WALK>), dim3((uint32_t)grid), dim3(kBlock), 0, stream, p);
    return hipGetLastError();
}

template <int NI, int L, int WALK, int... MODE>
void register_learn_walk(LnTable &t)
{
    ((t.fn[NI - 1][L - 1][WALK][MODE] = &launch_learn<NI, L, MODE, WALK>), ...);
}

template <int NI, int L>
void register_learn_one(LnTable &t)
{
    register_learn_walk<NI, L, kLn4, kLnFwd, kLnBwd, kLnBoth>(t);
    register_learn_walk<NI, L, kLn4Any, kLnBwd>(t);
    register_learn_walk<NI, L, kLn8Any, kLnFwd>(t);
    if constexpr (ln_blocks(kLnBoth, 4 * L * NI + 2) == 1) register_learn_walk<NI, L, kLn8, kLnFwd, kLnBwd, kLnBoth>(t);
}

}  // namespace dpd
