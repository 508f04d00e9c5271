// Backward (adjoint) kernels of the APH predistorter for gfx950.
//
// The forward map of Eq. (1), written with s = |x|^2, v = (Re x, Im x) and the
// precombined real 2x2 matrices M_{j,k} (order 2j+1, tap k), is
//     z_n = c + sum_k sum_j M_{j,k} s_{n-k}^j v_{n-k}.
// For a real loss E with G_n = dE/dRe z_n + j dE/dIm z_n (as a real 2-vector):
//   coefficients:  dE/dM_{j,k}[r][c] = sum_m G_{m+k}[r] * (s_m^j v_m)[c],
//                  dE/dc = sum_n G_n;
//   inputs:        dE/dv_m = sum_j [ s^j U_j + 2 j s^(j-1) v (v . U_j) ],
//                  U_j(m) = sum_k M_{j,k}^T G_{m+k}   (G_n = 0 for n >= N),
// i.e. the transpose of the filter (a correlation with the taps) followed by
// the transposed Jacobian of the pointwise basis.  The basis is recomputed
// from x; nothing from the forward pass is stored.  The chain rule through
// M = [[hr+gr, gi-hi], [hi+gi, hr-gr]] to the coefficients of the paper's
// stacking happens in the FP64 finalisation kernel.
//
// Reduction of the coefficient gradient is deterministic: each lane sums its
// own samples in a fixed order (FP32, at most kBwdFlush chunks at a time, row
// ends included), the wave adds those sums in a fixed tree to its FP64 totals, the
// block adds its waves' totals in order, one partial per block goes to the
// workspace, and a single block sums the partials in FP64 in block order.
#pragma once

#include <algorithm>

#include "dpd_fwd_kernels.h"
#include "dpd_reduce.h"
#include "dpd_table.h"

namespace dpd {

struct BwdParams {
    const float2 *x;
    const float2 *gz;
    float2 *gx;           // nullptr: no input gradient
    float *partials;      // [gridDim.x][E] (E = 4*L*NI + 2), nullptr: no coeff gradient
    int32_t E;            // E of the whole filter (a pass may cover some of its taps)
    int64_t n, ld, rows;
    int64_t tpr;          // full chunks per row (n / (64*S)); the ragged end is extra
    int32_t flush;        // chunks that a lane's FP32 sums cover
    int32_t pack;         // rows shorter than a chunk: several to a chunk
    int32_t fine;         // the sums over a wave's lanes in FP64 (else FP32)
    const float *M;       // precombined table
    const float2 *raw;    // or the K raw coefficients, precombined by every block
    CoefMap map;
};

typedef hipError_t (*BwdLaunch)(const BwdParams &, hipStream_t, int grid);

// Filters of up to kSpecL taps: one pass, want 0 = dx, 1 = dcoef, 2 = both.
// Longer ones: dx in one pass (want 0), the coefficient gradient in two, taps
// 0..7 as want 1 of kSpecL taps and taps 8.. by `tail` (their accumulators
// would not fit the registers at once).  Measured: 256 rows of 20001 samples, six
// taps, dx and dcoef 47 us where odd row starts took one thread per sample and a pass
// over the rows per sixteen entries, 946 us.
// want 3: dcoef of short "fine" inputs (bwd_dc_short_kernel), up to kSpecL taps.
struct BwdTable {
    BwdLaunch fn[kSpecNI][kMaxL][4];
    const void *kern[kSpecNI][kMaxL][4];
    BwdLaunch tail[kSpecNI][kSpecL][2];   // [.][taps beyond kSpecL - 1][short], dcoef
};

void register_bwd_ni1(BwdTable &);
void register_bwd_ni2(BwdTable &);
void register_bwd_ni3(BwdTable &);
void register_bwd_ni4(BwdTable &);
void register_bwd_ni5(BwdTable &);
void register_bwd_ni6(BwdTable &);
void register_bwd_ni7(BwdTable &);
void register_bwd_ni8(BwdTable &);

constexpr int kBwdS = 4;   // consecutive samples per lane
// Chunks a lane's FP32 coefficient-gradient sums cover before the wave adds them
// up and adds the result to its FP64 totals: 32 chunks = 128 samples per lane,
// added up in FP32.  Rows at odd 8-byte starts or strides and filters of more than
// kSpecL taps ("fine") are summed with less rounding: one chunk per 2^20 samples of
// the input, at most 64 samples per lane, added up in FP64; inputs below kBwdShort
// samples, where a chunk's four samples per lane would already be more than that, by
// bwd_dc_short_kernel, one sample per lane and 2^18 of the input.
constexpr int kBwdFlush = 32;
constexpr int64_t kBwdShort = (int64_t)1 << 20;
constexpr int64_t bwd_flush_fine(int64_t samples)
{
    return samples < kBwdShort ? std::max<int64_t>(samples >> 18, 1) : std::min<int64_t>(samples >> 20, 16);
}

// FP64 sums of table entry q's four coefficient-gradient partials (two for
// q = L NI, the c entry) over nblk blocks: each thread its strided share of
// the blocks in order, then the DPP lane sum of each wave and the four waves
// in order (bitwise reproducible).  u is valid in thread 0.
__device__ __forceinline__ void dcoef_block_sums(const float *__restrict__ partials, int nblk, const CoefMap &map,
                                                 int q, double (&red)[kBlock / 64][4], double (&u)[4])
{
    const int E = 4 * map.L * map.NI + 2;
    const bool dc = q == map.L * map.NI;
    double a[4] = {0.0, 0.0, 0.0, 0.0};
    for (int b = threadIdx.x; b < nblk; b += kBlock) {
        const float *pp = partials + (int64_t)b * E + 4 * q;
        a[0] += (double)pp[0];
        a[1] += (double)pp[1];
        if (!dc) {
            a[2] += (double)pp[2];
            a[3] += (double)pp[3];
        }
    }
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
        a[e] = wave_sum_to_lane63(a[e]);
        if (lane == 63) red[wv][e] = a[e];
    }
    __syncthreads();
#pragma unroll
    for (int e = 0; e < 4; ++e) {
        u[e] = red[0][e];
        for (int w = 1; w < kBlock / 64; ++w) u[e] += red[w][e];
    }
}

// The chain rule from table entry q's sums to the coefficients of the
// section 2.2 stacking (M = [[hr+gr, gi-hi], [hi+gi, hr-gr]], order 2j+1,
// tap k): u1 = dE/dm00, u4 = dE/dm01, u3 = dE/dm10, u2 = dE/dm11,
//   grad h = (u1 + u2) + j (u3 - u4),  grad hbar = (u1 - u2) + j (u3 + u4),
//   grad c = sum G (q = L NI).
// Returns how many coefficients (0..2) entry q feeds: idx[i], grad[i].
__device__ __forceinline__ int dcoef_block_grads(const CoefMap &map, int q, const double (&u)[4], int (&idx)[2],
                                                 float2 (&grad)[2])
{
    const int L = map.L, NI = map.NI;
    if (q == L * NI) {
        idx[0] = (map.n_main + map.n_conj) * L;
        grad[0] = make_float2((float)u[0], (float)u[1]);
        return 1;
    }
    const int k = q / NI, j = q - k * NI;
    const double u1 = u[0], u4 = u[1], u3 = u[2], u2 = u[3];
    int c = 0;
    if (map.main_idx[j] >= 0) {
        idx[c] = map.main_idx[j] * L + k;
        grad[c++] = make_float2((float)(u1 + u2), (float)(u3 - u4));
    }
    if (map.conj_idx[j] >= 0) {
        idx[c] = (map.n_main + map.conj_idx[j]) * L + k;
        grad[c++] = make_float2((float)(u1 - u2), (float)(u3 + u4));
    }
    return c;
}

template <bool B>
struct BwdTag {
    static constexpr bool value = B;
};

// Blocks per CU the registers are held to.  One wave per SIMD issues half of what
// two do, so the kernel of both gradients is held to two blocks where it would
// just miss them and that costs no spills in its loop (2^24 samples: NI = 4, L = 7
// 167 -> 126 us; NI = 5, L = 6 187 -> 135; NI = 5, L = 8, not held, 254 us would be
// 458).  Up to 110 accumulators two blocks fit by themselves.
constexpr int bwd_blocks(int NI, int L, bool both)
{
    const int E = 4 * L * NI + 2;
    return both && E > 110 && E + L <= 136 ? 2 : 1;
}

// dx by Horner in s, power levels from the highest down, or by explicit powers,
// levels upwards.  Horner rounds less (relative error of dx against 64 bits 0.80e-7
// over twelve shapes, explicit powers 0.86e-7); with both gradients it needs every
// power of s at once, for which the kernels of six levels and more have no
// registers left (2^22 samples at NI = L = 8: 112 us and 118).
constexpr bool bwd_horner(int NI, bool dx, bool dc) { return dx && (!dc || NI <= 5); }

// Persistent grid over the full chunks (C = 64*S samples) of all rows, wave g
// taking chunks g, g + nw, ... (rows flattened), then the ragged row ends.
// Per chunk the wave stages G (the chunk plus the L-1 samples after it; zero
// past the row end) and x (the chunk) in padded wave-private LDS buffers,
// with nontemporal 1 KiB-contiguous loads issued one chunk ahead: a chunk's
// registers are staged right after the previous chunk's stores, and the next
// chunk's loads go out into the same registers before the staged chunk is
// filtered, so the compiler's counter waits never cover the prefetch.  Each
// lane owns S consecutive samples m and reads G_{m..m+S+L-2}.  One pass over
// the power levels j produces both gradients: U_j by taps for dx = P + 2 Q v (P =
// sum s^j U_j, Q = sum j s^(j-1) v.U_j), and G (x) s^j v into the per-lane
// coefficient accumulators.  K0: the first tap of a pass over taps K0 .. K0 + L - 1 of a
// longer filter (coefficient gradient only).  Rows may start at any sample:
// 16-byte accesses need no 16-byte alignment here (v4f_s).
template <int NI, int L, bool DX, bool DC, int K0 = 0>
__global__ void __launch_bounds__(kBlock, bwd_blocks(NI, L, DX && DC)) bwd_kernel(BwdParams p)
{
    static_assert(!DX || K0 == 0, "the input gradient needs every tap");
    static_assert(K0 % kBwdS == 0, "the window of a pass starts on a pad group");
    constexpr int S = kBwdS;
    constexpr int C = 64 * S;
    constexpr int W = S + L - 1;
    constexpr int NV = S / 2;
    constexpr int WAVES = kBlock / 64;
    constexpr int NM = 4 * L * NI;                              // matrix floats (c has no gradient path here)
    constexpr int E = NM + (K0 == 0 ? 2 : 0);                   // c belongs to the first pass
    constexpr int HS = K0 + L - 1;                              // right halo
    constexpr bool HORNER = bwd_horner(NI, DX, DC);
    constexpr int GSLOTS = C + HS + (C + HS) / S + 1;
    constexpr int XSLOTS = C + C / S;
    __shared__ __align__(16) float2 gs[WAVES][GSLOTS];
    __shared__ __align__(16) float2 xsh[WAVES][XSLOTS];
    __shared__ __align__(16) float mt[DX ? NM : 1];
    __shared__ double red[DC ? WAVES * E : 1];   // per-wave FP64 totals of the coefficient gradient

    const int tid = threadIdx.x, lane = tid & 63;
    const int wv = __builtin_amdgcn_readfirstlane(tid >> 6);
    // Every argument is read here, in one go: one wait instead of a chain of them,
    // and no scalar load is in flight at the chunk loop's head, where it would make
    // the compiler wait for all LDS reads of a window at once (2^24 samples at NI = 4,
    // L = 6, coefficient gradient alone: 69 us and 64).
    const uint32_t nb = gridDim.x;
    asm volatile("" ::"s"(p.x), "s"(p.gz), "s"(p.n), "s"(p.ld), "s"(p.rows), "s"(p.tpr), "s"(p.pack), "s"(nb));
    if constexpr (DX) asm volatile("" ::"s"(p.gx), "s"(p.M), "s"(p.raw));
    if constexpr (DC) asm volatile("" ::"s"(p.partials), "s"(p.E), "s"(p.flush), "s"(p.fine));
    if constexpr (DX) {
        if (__builtin_expect(p.raw != nullptr, 0)) {
            for (int e = tid; e < NM; e += kBlock) mt[e] = table_entry(p.M, p.raw, p.map, e);
        } else {
            for (int e = tid; e < NM; e += kBlock) mt[e] = p.M[e];
        }
        __syncthreads();
    }
    float2 *G = gs[wv];
    float2 *X = xsh[wv];
    // slot of chunk-relative sample d: one pad after every S
    auto slot = [](int d) { return d + d / S; };
    const int hl = HS > 0 ? (lane < HS ? lane : HS - 1) : 0;

    float acc[DC ? E : 1];
#pragma unroll
    for (int e = 0; e < (DC ? E : 1); ++e) acc[e] = 0.f;
    // The per-lane FP32 sums cover at most kBwdFlush chunks: then they are
    // summed over the wave and added to the wave's FP64 totals (entry
    // 64 g + l in lane l of tot[g]), so the rounding error does not grow with
    // the stream length.
    constexpr int NGT = DC ? (E + 63) / 64 : 1;
    double tot[NGT];
#pragma unroll
    for (int g = 0; g < NGT; ++g) tot[g] = 0.0;
    auto flush = [&]() {
        if constexpr (DC) {
            if (p.fine)
                wave_sums_into<double, E>(acc, tot, lane);
            else
                wave_sums_into<float, E>(acc, tot, lane);
#pragma unroll
            for (int e = 0; e < E; ++e) acc[e] = 0.f;
        }
    };

    struct Regs {
        float4 g[NV];
        float4 x[NV];
        float2 gh;   // raw G_{t0 + C + hl} (replaced by zero past the row end at staging)
    };
    // full chunk at (row, t0): every load unconditional
    auto load_full = [&](Regs &R, int64_t row, int64_t t0) {
        const v4f_s *g4 = reinterpret_cast<const v4f_s *>(p.gz + row * p.ld + t0);
        const v4f_s *x4 = reinterpret_cast<const v4f_s *>(p.x + row * p.ld + t0);
#pragma unroll
        for (int i = 0; i < NV; ++i) {
            const v4f_s u = __builtin_nontemporal_load(g4 + lane + 64 * i);
            R.g[i] = make_float4(u.x, u.y, u.z, u.w);
        }
#pragma unroll
        for (int i = 0; i < NV; ++i) {
            const v4f_s u = __builtin_nontemporal_load(x4 + lane + 64 * i);
            R.x[i] = make_float4(u.x, u.y, u.z, u.w);
        }
        if (HS > 0) {
            const int64_t m = t0 + C + hl;
            R.gh = p.gz[row * p.ld + (m < p.n ? m : p.n - 1)];
        }
    };
    // The samples outside full chunks, a chunk at a time: "end" r is what row r has
    // left.  Packed: the rows one after the other, HS zeros after each, cut into
    // chunks; end r is chunk r of that.
    const bool packed = p.pack != 0;
    const int stride = (int)p.n + HS, lead = (int)p.ld - stride;   // packed: of the rows (both fit)
    const uint32_t inv = packed ? ((1u << 20) + stride - 1) / stride : 0;
    struct End {
        int64_t at;      // first sample of the chunk's first row, or of the rest of the row
        int skip;        // samples of that row before the chunk
        int lim, rows;   // samples of a row, rows from this one on
    };
    auto end_of = [&](int64_t r) {
        if (!packed) return End{r * p.ld + p.tpr * C, 0, (int)(p.n - p.tpr * C), 1};
        const int64_t v = r * C;
        const int64_t row = v >> 32 ? v / stride : (int64_t)((uint32_t)v / (uint32_t)stride);
        const int64_t more = p.rows - row;
        return End{row * p.ld, (int)(v - row * stride), (int)p.n, (int)(more < 1024 ? more : 1024)};
    };
    // places of samples j(0), j(1), .. of an end relative to its `at`, -1 where there
    // is none
    auto end_at = [&](const End &e, auto j, auto &at) {
        constexpr int M = sizeof(at) / sizeof(int);
        if (packed) {
#pragma unroll
            for (int i = 0; i < M; ++i) {
                const int t = e.skip + j(i);
                const int q = (int)(((uint32_t)t * inv) >> 20);   // t / stride (t below 2^10)
                at[i] = t - q * stride < e.lim && q < e.rows ? t + q * lead : -1;
            }
        } else {
#pragma unroll
            for (int i = 0; i < M; ++i) at[i] = j(i) < e.lim ? j(i) : -1;
        }
    };
    auto load_part = [&](Regs &R, const End &e) {
        const float2 *gr = p.gz + e.at, *xr = p.x + e.at;
        int at[S];
        end_at(e, [&](int i) { return 2 * (lane + 64 * (i / 2)) + i % 2; }, at);
        const auto get = [&](const float2 *v, int i) { return at[i] >= 0 ? v[(uint32_t)at[i]] : make_float2(0.f, 0.f); };
#pragma unroll
        for (int i = 0; i < NV; ++i) {
            const float2 a = get(gr, 2 * i), b = get(gr, 2 * i + 1);
            R.g[i] = make_float4(a.x, a.y, b.x, b.y);
            const float2 c = get(xr, 2 * i), d = get(xr, 2 * i + 1);
            R.x[i] = make_float4(c.x, c.y, d.x, d.y);
        }
        R.gh = make_float2(0.f, 0.f);
        if (HS > 0 && packed) {
            int ah[1];
            end_at(e, [&](int) { return C + hl; }, ah);
            if (ah[0] >= 0) R.gh = gr[(uint32_t)ah[0]];
        }
    };
    auto stage = [&](const Regs &R, bool halo) {
        wave_lds_order();   // the previous chunk's LDS reads are done
#pragma unroll
        for (int i = 0; i < NV; ++i) {
            const int j = 2 * (lane + 64 * i);
            G[slot(j)] = make_float2(R.g[i].x, R.g[i].y);
            G[slot(j) + 1] = make_float2(R.g[i].z, R.g[i].w);
            X[slot(j)] = make_float2(R.x[i].x, R.x[i].y);
            X[slot(j) + 1] = make_float2(R.x[i].z, R.x[i].w);
        }
        if (HS > 0 && lane < HS) G[slot(C + lane)] = halo ? R.gh : make_float2(0.f, 0.f);
        wave_lds_order();
    };
    // the lane's halo sample of a full chunk at t0 is inside the row
    auto in_row = [&](int64_t t0) { return t0 + C + lane < p.n; };
    // gradients of a staged chunk: a full one at e.at, or an end
    auto compute = [&](const End &e, auto full_tag) {
        constexpr bool FULL = decltype(full_tag)::value;
        // An opaque zero keeps the table reads inside the loop (hoisted, the
        // whole table would occupy registers next to the accumulators).
        int z = 0;
        asm volatile("" : "+v"(z));
        const float4 *M4 = reinterpret_cast<const float4 *>(mt + z);
        float ga[W], gb[W];
#pragma unroll
        for (int w = 0; w < W; ++w) {
            const float2 g = G[slot(lane * S + w) + K0 + K0 / S];   // sample K0 on
            ga[w] = g.x;
            gb[w] = g.y;
        }
        float va[S], vb[S], sq[S];
#pragma unroll
        for (int i = 0; i < S; ++i) {
            const float2 v = X[slot(lane * S + i)];
            va[i] = v.x;
            vb[i] = v.y;
            sq[i] = __builtin_fmaf(v.x, v.x, v.y * v.y);
        }
        float Pa[S], Pb[S], Q[S];
        float pws[HORNER && DC ? NI : 1][S];   // s^j of every level
        float pw[S], pwl[S];                   // s^j, 2 j s^(j-1)
        if constexpr (HORNER && DC) {
#pragma unroll
            for (int j = 1; j < NI; ++j)
#pragma unroll
                for (int i = 0; i < S; ++i) pws[j][i] = j == 1 ? sq[i] : pws[j - 1][i] * sq[i];
        }
#pragma unroll
        for (int i = 0; i < S; ++i) {
            Pa[i] = Pb[i] = Q[i] = 0.f;
            pw[i] = 1.f;
            pwl[i] = 0.f;
        }
#pragma unroll
        for (int jj = 0; jj < NI; ++jj) {
            const int j = HORNER ? NI - 1 - jj : jj;
            float Ua[S], Ub[S], ba[S], bb[S];
#pragma unroll
            for (int i = 0; i < S; ++i) {
                Ua[i] = Ub[i] = 0.f;
                if constexpr (DC) {
                    const float w = HORNER && j > 0 ? pws[HORNER ? j : 0][i] : pw[i];
                    ba[i] = w * va[i];
                    bb[i] = w * vb[i];
                }
            }
#pragma unroll
            for (int k = 0; k < L; ++k) {
                float4 m;   // [[m.x, m.y], [m.z, m.w]]
                if constexpr (DX) m = M4[k * NI + j];
#pragma unroll
                for (int i = 0; i < S; ++i) {
                    const float a = ga[i + k], b = gb[i + k];
                    if constexpr (DX) {
                        Ua[i] = __builtin_fmaf(m.x, a, Ua[i]);
                        Ua[i] = __builtin_fmaf(m.z, b, Ua[i]);
                        Ub[i] = __builtin_fmaf(m.y, a, Ub[i]);
                        Ub[i] = __builtin_fmaf(m.w, b, Ub[i]);
                    }
                    if constexpr (DC) {
                        float *u = &acc[4 * (k * NI + j)];
                        u[0] = __builtin_fmaf(a, ba[i], u[0]);
                        u[1] = __builtin_fmaf(a, bb[i], u[1]);
                        u[2] = __builtin_fmaf(b, ba[i], u[2]);
                        u[3] = __builtin_fmaf(b, bb[i], u[3]);
                    }
                }
            }
#pragma unroll
            for (int i = 0; i < S; ++i) {
                if constexpr (HORNER) {
                    Pa[i] = j == NI - 1 ? Ua[i] : __builtin_fmaf(Pa[i], sq[i], Ua[i]);
                    Pb[i] = j == NI - 1 ? Ub[i] : __builtin_fmaf(Pb[i], sq[i], Ub[i]);
                    if (j > 0) {   // the factor 2 of Q comes at the end
                        const float d = (float)j * __builtin_fmaf(va[i], Ua[i], vb[i] * Ub[i]);
                        Q[i] = j == NI - 1 ? d : __builtin_fmaf(Q[i], sq[i], d);
                    }
                } else {
                    if constexpr (DX) {
                        // level 0 has s^0 = 1: P starts at U_0
                        Pa[i] = j == 0 ? Ua[i] : __builtin_fmaf(pw[i], Ua[i], Pa[i]);
                        Pb[i] = j == 0 ? Ub[i] : __builtin_fmaf(pw[i], Ub[i], Pb[i]);
                        if (j > 0) {
                            const float d = __builtin_fmaf(va[i], Ua[i], vb[i] * Ub[i]);
                            Q[i] = j == 1 ? pwl[i] * d : __builtin_fmaf(pwl[i], d, Q[i]);
                        }
                        pwl[i] = (float)(2 * (j + 1)) * pw[i];   // 2 (j + 1) s^j: Q carries the factor 2 of dx
                    }
                    pw[i] *= sq[i];
                }
            }
            // One power level at a time: the empty asm statements consume this
            // level's results, so the instruction selector cannot sink its
            // multiply-adds past the barrier (it did, which kept every
            // level's table entries live at once); only this level's L
            // table entries are in registers.
            if constexpr (DC) {
#pragma unroll
                for (int k = 0; k < L; ++k)
#pragma unroll
                    for (int q = 0; q < 4; ++q) asm volatile("" ::"v"(acc[4 * (k * NI + j) + q]));
            }
            if constexpr (DX) {
#pragma unroll
                for (int i = 0; i < S; ++i) asm volatile("" ::"v"(Pa[i]), "v"(Pb[i]), "v"(Q[i]));
            }
            __builtin_amdgcn_sched_barrier(0);
        }
        if constexpr (DC && K0 == 0) {
#pragma unroll
            for (int i = 0; i < S; ++i) {
                acc[E - 2] += ga[i];
                acc[E - 1] += gb[i];
            }
        }
        if constexpr (DX) {
            float dxa[S], dxb[S];
#pragma unroll
            for (int i = 0; i < S; ++i) {
                const float q = HORNER ? 2.f * Q[i] : Q[i];
                dxa[i] = __builtin_fmaf(q, va[i], Pa[i]);
                dxb[i] = __builtin_fmaf(q, vb[i], Pb[i]);
            }
            if constexpr (FULL) {
                // back through LDS so every store instruction writes 1 KiB
                wave_lds_order();
#pragma unroll
                for (int i = 0; i < S; ++i) G[slot(lane * S + i)] = make_float2(dxa[i], dxb[i]);
                wave_lds_order();
                v4f_s *o4 = reinterpret_cast<v4f_s *>(p.gx + e.at);
#pragma unroll
                for (int i = 0; i < NV; ++i) {
                    const int j = 2 * (lane + 64 * i);
                    const float2 u = G[slot(j)], w = G[slot(j) + 1];
                    const v4f_s v = {u.x, u.y, w.x, w.y};
                    __builtin_nontemporal_store(v, o4 + lane + 64 * i);
                }
            } else {
                int at[S];
                end_at(e, [&](int i) { return lane * S + i; }, at);
                float2 *o = p.gx + e.at;
#pragma unroll
                for (int i = 0; i < S; ++i)
                    if (at[i] >= 0) o[(uint32_t)at[i]] = make_float2(dxa[i], dxb[i]);
            }
        }
    };

    int held = 0;                                // chunks in the FP32 sums
    const int64_t tpr = p.tpr;                   // full chunks per row
    const int64_t total = p.rows * tpr;
    const int64_t nw = (int64_t)nb * WAVES;
    const int64_t gw = (int64_t)xcd_remap(blockIdx.x, nb) * WAVES + wv;
    if (gw < total) {
        const int64_t left = (total - 1 - gw) / nw + 1;
        // (row, chunk in row) advanced by nw chunks per step without a division
        const int64_t dq = nw / tpr, dr = nw - dq * tpr;
        int64_t row = gw / tpr, tix = gw - row * tpr;
        Regs R;
        load_full(R, row, tix * C);
        stage(R, in_row(tix * C));
        for (int64_t i = 0; i + 1 < left; ++i) {
            const int64_t cur = row * p.ld + tix * C;
            row += dq;
            tix += dr;
            if (tix >= tpr) {
                tix -= tpr;
                ++row;
            }
            load_full(R, row, tix * C);
            compute(End{cur, 0, 0, 0}, BwdTag<true>{});
            stage(R, in_row(tix * C));
            if (++held == p.flush) {
                flush();
                held = 0;
            }
        }
        compute(End{row * p.ld + tix * C, 0, 0, 0}, BwdTag<true>{});
        ++held;
    }
    // the ends continue the round-robin order (chunk c to wave c mod nw)
    const int64_t ends = packed ? (p.rows * (int64_t)stride - HS + C - 1) / C : p.n > tpr * C ? p.rows : 0;
    for (int64_t r = (gw + nw - total % nw) % nw; r < ends; r += nw) {
        Regs R;
        const End e = end_of(r);
        load_part(R, e);
        stage(R, true);
        if (held == p.flush) {
            flush();
            held = 0;
        }
        compute(e, BwdTag<false>{});
        ++held;
    }

    if constexpr (DC) {
        // wave FP64 totals -> block -> one FP32 partial per block, fixed order
        flush();
#pragma unroll
        for (int g = 0; g < NGT; ++g)
            if (64 * g + lane < E) red[wv * E + 64 * g + lane] = tot[g];
        __syncthreads();
        for (int e = tid; e < E; e += kBlock) {
            double t = 0.0;
#pragma unroll
            for (int w = 0; w < WAVES; ++w) t += red[w * E + e];
            const int at = e < NM ? 4 * NI * K0 + e : p.E - 2 + (e - NM);
            p.partials[(int64_t)blockIdx.x * p.E + at] = (float)t;
        }
    }
}

// The coefficient gradient of short "fine" inputs (below kBwdShort samples), taps K0
// .. K0 + L - 1: the rows one after the other, a sample per lane, so that a lane's
// FP32 sums cover one sample per 2^18 of the input before they go to FP64; a chunk
// of four would round more (32 rows of 20001 samples, six taps: relative error 0.61e-7,
// in bwd_kernel 0.77e-7).  A tap past the row's end adds nothing, whatever x holds.
// Bound by the wave sums in FP64, each longer than a 64-sample step (23 us there, 154
// with one thread per sample and a pass over the rows per sixteen entries).
template <int NI, int L, int K0>
__global__ void __launch_bounds__(kBlock) bwd_dc_short_kernel(BwdParams p)
{
    constexpr int WAVES = kBlock / 64, NM = 4 * L * NI, E = NM + (K0 == 0 ? 2 : 0), NGT = (E + 63) / 64;
    __shared__ double red[WAVES * E];
    const int tid = threadIdx.x, lane = tid & 63;
    const int wv = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int total = (int)(p.rows * p.n), n = (int)p.n;
    const int nw = (int)gridDim.x * WAVES;
    float acc[E];
    double tot[NGT];
#pragma unroll
    for (int e = 0; e < E; ++e) acc[e] = 0.f;
#pragma unroll
    for (int g = 0; g < NGT; ++g) tot[g] = 0.0;
    struct In {
        float2 v, g[L];
        int taps;   // of this pass inside the row
    };
    const auto load = [&](int c) {
        In r;
        const int i = 64 * c + lane, q = i < total ? i : total - 1;
        const int row = (int)((uint32_t)q / (uint32_t)n), m = q - row * n;
        const int64_t at = row * p.ld + m;
        r.v = p.x[at];
        r.taps = i < total ? n - m - K0 : 0;
#pragma unroll
        for (int k = 0; k < L; ++k) r.g[k] = p.gz[at + (m + K0 + k < n ? K0 + k : 0)];
        return r;
    };
    const int chunks = (total + 63) / 64;
    int held = 0;
    int c = (int)blockIdx.x * WAVES + wv;
    if (c < chunks) {
        In r = load(c);
        while (true) {
            const int next = c + nw;
            const In a = r;
            if (next < chunks) r = load(next);
            float ba[NI], bb[NI];
            const float s = __builtin_fmaf(a.v.x, a.v.x, a.v.y * a.v.y);
            float w = 1.f;
#pragma unroll
            for (int j = 0; j < NI; ++j) {
                ba[j] = w * a.v.x;
                bb[j] = w * a.v.y;
                w *= s;
            }
#pragma unroll
            for (int k = 0; k < L; ++k) {
                if (k < a.taps) {
#pragma unroll
                    for (int j = 0; j < NI; ++j) {
                        float *e = acc + 4 * (k * NI + j);
                        e[0] = __builtin_fmaf(a.g[k].x, ba[j], e[0]);
                        e[1] = __builtin_fmaf(a.g[k].x, bb[j], e[1]);
                        e[2] = __builtin_fmaf(a.g[k].y, ba[j], e[2]);
                        e[3] = __builtin_fmaf(a.g[k].y, bb[j], e[3]);
                    }
                    if (K0 == 0 && k == 0) {
                        acc[E - 2] += a.g[0].x;
                        acc[E - 1] += a.g[0].y;
                    }
                }
            }
            if (++held == p.flush || next >= chunks) {
                wave_sums_into<double, E>(acc, tot, lane);
#pragma unroll
                for (int e = 0; e < E; ++e) acc[e] = 0.f;
                held = 0;
            }
            if (next >= chunks) break;
            c = next;
        }
    }
    // as bwd_kernel: wave FP64 totals -> block -> one FP32 partial per block
#pragma unroll
    for (int g = 0; g < NGT; ++g)
        if (64 * g + lane < E) red[wv * E + 64 * g + lane] = tot[g];
    __syncthreads();
    for (int e = tid; e < E; e += kBlock) {
        double t = 0.0;
#pragma unroll
        for (int w = 0; w < WAVES; ++w) t += red[w * E + e];
        const int at = e < NM ? 4 * NI * K0 + e : p.E - 2 + (e - NM);
        p.partials[(int64_t)blockIdx.x * p.E + at] = (float)t;
    }
}

template <int NI, int L, int K0 = 0>
hipError_t launch_bwd_short(const BwdParams &p, hipStream_t stream, int grid)
{
    hipLaunchKernelGGL((bwd_dc_short_kernel<NI, L, K0>), dim3((uint32_t)grid), dim3(kBlock), 0, stream, p);
    return hipGetLastError();
}

template <int NI, int L, bool DX, bool DC, int K0 = 0>
hipError_t launch_bwd(const BwdParams &p, hipStream_t stream, int grid)
{
    hipLaunchKernelGGL((bwd_kernel<NI, L, DX, DC, K0>), dim3((uint32_t)grid), dim3(kBlock), 0, stream, p);
    return hipGetLastError();
}

template <int NI, int L>
void register_bwd_one(BwdTable &t)
{
    t.fn[NI - 1][L - 1][0] = &launch_bwd<NI, L, true, false>;
    t.kern[NI - 1][L - 1][0] = (const void *)&bwd_kernel<NI, L, true, false>;
    if constexpr (L <= kSpecL) {
        t.fn[NI - 1][L - 1][1] = &launch_bwd<NI, L, false, true>;
        t.fn[NI - 1][L - 1][2] = &launch_bwd<NI, L, true, true>;
        t.kern[NI - 1][L - 1][1] = (const void *)&bwd_kernel<NI, L, false, true>;
        t.kern[NI - 1][L - 1][2] = (const void *)&bwd_kernel<NI, L, true, true>;
        t.fn[NI - 1][L - 1][3] = &launch_bwd_short<NI, L>;
        t.kern[NI - 1][L - 1][3] = (const void *)&bwd_dc_short_kernel<NI, L, 0>;
        t.tail[NI - 1][L - 1][0] = &launch_bwd<NI, L, false, true, kSpecL>;
        t.tail[NI - 1][L - 1][1] = &launch_bwd_short<NI, L, kSpecL>;
    }
}

}  // namespace dpd
