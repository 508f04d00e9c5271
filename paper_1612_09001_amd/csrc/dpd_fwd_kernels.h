// Forward kernels of the APH predistorter (Eq. 1 / Algorithm 1) for gfx950.
//
// One pass per sample does all three steps of Algorithm 1 -- basis
// (polynomial), filtering and accumulation + c -- in registers.  The paper's
// own fused single kernel (section 3.2.2) keeps intermediates out of global
// memory too; it fetches the L-1 preceding basis values with warp shuffles and
// spends (L-1)/32 of the lanes on redundant samples (section 3.3.2).  Here
// a block instead stages its tile plus an (L-1)-sample halo once (LDS or
// direct cached loads), and each thread produces S consecutive outputs from a
// register window of S+L-1 samples, so no lane is redundant.
//
// Arithmetic per output.  With s = |x|^2 and v = (Re x, Im x), the main and
// conjugate taps of order 2j+1 combine into one real 2x2 matrix M_{j,k}
// (h w + hbar conj(w) is real-linear in w), so
//     z_n = c + sum_k W_k(s_{n-k}) v_{n-k},   W_k(s) = sum_j M_{j,k} s^j,
// and W_k is evaluated by Horner in s: 4*NI fused multiply-adds per tap and
// output, the minimum for 4*NI*L independent real coefficients.  No sqrt or
// transcendental is needed for odd orders.
#pragma once

#include "dpd_internal.h"

namespace dpd {

typedef float v4f __attribute__((ext_vector_type(4)));
// Two samples at a time from any sample's address: the hardware's 16-byte
// global loads and stores need 4-byte alignment only, so rows that start at an
// odd sample run the same instructions (a 1 KiB access then touches nine cache
// lines instead of eight).
typedef float v4f_s __attribute__((ext_vector_type(4), aligned(8)));

// Coefficient tables are read through the constant address space: uniform,
// read-only loads from it become scalar loads (SGPR operands of the FMAs).
typedef const float __attribute__((address_space(4))) cfloat;
__device__ __forceinline__ const cfloat *as_const(const float *p)
{
    return (const cfloat *)p;
}

// Global-address-space views, for pointers the compiler cannot trace back to
// a kernel argument (so loads and stores become global_*, not flat_*, and
// only count against the vector-memory counter).
typedef float v2f __attribute__((ext_vector_type(2)));
typedef const v2f __attribute__((address_space(1))) gcv2f;
typedef const v4f __attribute__((address_space(1))) gcv4f;
typedef v2f __attribute__((address_space(1))) gv2f;
typedef v4f __attribute__((address_space(1))) gv4f;

// Consecutive tiles share a halo; keep neighbours on one XCD (one L2) by
// mapping dispatch order (round-robin over the 8 XCDs) to contiguous ranges.
__device__ __forceinline__ uint32_t xcd_remap(uint32_t b, uint32_t G)
{
    const uint32_t q = G >> 3, r = G & 7u;
    const uint32_t x = b & 7u, l = b >> 3;
    return x < r ? x * (q + 1) + l : r * (q + 1) + (x - r) * q + l;
}

// Sample m of a row; zero before the start unless a history is given
// (hist[L-1+m] for -(L-1) <= m < 0).
template <int L>
__device__ __forceinline__ float2 sample_or_hist(const float2 *__restrict__ x, int64_t m, int64_t n,
                                                 const float2 *__restrict__ hist)
{
    if (m >= 0) return m < n ? x[m] : make_float2(0.f, 0.f);
    if (hist != nullptr && m >= -(int64_t)(L - 1)) return hist[(L - 1) + m];
    return make_float2(0.f, 0.f);
}

// S outputs from a window of S+L-1 samples; window index w = i + (L-1) - k
// holds x_{n_i - k}.  `top` holds M_{NI-1,k} (4 floats per tap) in VGPRs; the
// remaining levels are read through the uniform pointer M (scalar loads).
template <int NI, int L, int S>
__device__ __forceinline__ void fir_outputs(const float (&a)[S + L - 1], const float (&b)[S + L - 1],
                                            const float (&s)[S + L - 1], const float (&top)[4 * L],
                                            const cfloat *M, float (&zr)[S], float (&zi)[S])
{
    constexpr int T = 4 * (NI - 1);   // scalar coefficients per tap
    // An opaque zero offset keeps the scalar loads inside the caller's chunk
    // loop: hoisted, the whole table would not fit the scalar registers and
    // would be spilled to VGPR lanes and read back with one v_readlane each.
    int z = 0;
    asm volatile("" : "+s"(z));
    const cfloat *Mz = M + z;
    const float cr = Mz[4 * L * NI], ci = Mz[4 * L * NI + 1];
#pragma unroll
    for (int i = 0; i < S; ++i) {
        zr[i] = cr;
        zi[i] = ci;
    }
    // tap k's coefficients are in c while tap k + 1's load
    float c[T > 0 ? T : 1];
#pragma unroll
    for (int e = 0; e < T; ++e) c[e] = Mz[e];
#pragma unroll
    for (int k = 0; k < L; ++k) {
        float cn[T > 0 ? T : 1];
        if (k + 1 < L) {
#pragma unroll
            for (int e = 0; e < T; ++e) cn[e] = Mz[4 * NI * (k + 1) + e];
        }
#pragma unroll
        for (int i = 0; i < S; ++i) {
            const int w = i + (L - 1) - k;
            float w00 = top[4 * k + 0], w01 = top[4 * k + 1];
            float w10 = top[4 * k + 2], w11 = top[4 * k + 3];
#pragma unroll
            for (int j = NI - 2; j >= 0; --j) {
                w00 = __builtin_fmaf(w00, s[w], c[4 * j + 0]);
                w01 = __builtin_fmaf(w01, s[w], c[4 * j + 1]);
                w10 = __builtin_fmaf(w10, s[w], c[4 * j + 2]);
                w11 = __builtin_fmaf(w11, s[w], c[4 * j + 3]);
            }
            zr[i] = __builtin_fmaf(w00, a[w], zr[i]);
            zr[i] = __builtin_fmaf(w01, b[w], zr[i]);
            zi[i] = __builtin_fmaf(w10, a[w], zi[i]);
            zi[i] = __builtin_fmaf(w11, b[w], zi[i]);
        }
        if (k + 1 < L) {
#pragma unroll
            for (int e = 0; e < T; ++e) c[e] = cn[e];
        }
    }
}

// Same FIR with every coefficient in registers (coef: the whole table,
// 4*L*NI + 2 floats): no scalar operands, so no extra moves or scalar
// register pressure.  Used when the table is small enough to keep resident.
template <int NI, int L, int S>
__device__ __forceinline__ void fir_outputs_reg(const float (&a)[S + L - 1], const float (&b)[S + L - 1],
                                                const float (&s)[S + L - 1],
                                                const float (&coef)[4 * L * NI + 2], float (&zr)[S],
                                                float (&zi)[S])
{
#pragma unroll
    for (int i = 0; i < S; ++i) {
        zr[i] = coef[4 * L * NI];
        zi[i] = coef[4 * L * NI + 1];
    }
#pragma unroll
    for (int k = 0; k < L; ++k) {
        const float *Mk = coef + 4 * NI * k;
#pragma unroll
        for (int i = 0; i < S; ++i) {
            const int w = i + (L - 1) - k;
            float w00 = Mk[4 * (NI - 1) + 0], w01 = Mk[4 * (NI - 1) + 1];
            float w10 = Mk[4 * (NI - 1) + 2], w11 = Mk[4 * (NI - 1) + 3];
#pragma unroll
            for (int j = NI - 2; j >= 0; --j) {
                w00 = __builtin_fmaf(w00, s[w], Mk[4 * j + 0]);
                w01 = __builtin_fmaf(w01, s[w], Mk[4 * j + 1]);
                w10 = __builtin_fmaf(w10, s[w], Mk[4 * j + 2]);
                w11 = __builtin_fmaf(w11, s[w], Mk[4 * j + 3]);
            }
            zr[i] = __builtin_fmaf(w00, a[w], zr[i]);
            zr[i] = __builtin_fmaf(w01, b[w], zr[i]);
            zi[i] = __builtin_fmaf(w10, a[w], zi[i]);
            zi[i] = __builtin_fmaf(w11, b[w], zi[i]);
        }
    }
}

// fir_outputs with the table in LDS (CS): each tap's 4*NI floats are read as
// broadcast 16-byte LDS loads one tap ahead of their use.  Scheduling
// barriers between taps keep the compiler from hoisting every tap's reads to
// the top (which would hold the whole table in registers).
template <int NI>
__device__ __forceinline__ void lds_tap_load(const float *CS, int k, float (&Mk)[4 * NI])
{
    const float4 *ck = reinterpret_cast<const float4 *>(CS + 4 * NI * k);
#pragma unroll
    for (int j = 0; j < NI; ++j) {
        const float4 u = ck[j];
        Mk[4 * j + 0] = u.x;
        Mk[4 * j + 1] = u.y;
        Mk[4 * j + 2] = u.z;
        Mk[4 * j + 3] = u.w;
    }
}

template <int NI, int L, int S>
__device__ __forceinline__ void fir_outputs_lds(const float (&a)[S + L - 1], const float (&b)[S + L - 1],
                                                const float (&s)[S + L - 1], const float *CS,
                                                float (&zr)[S], float (&zi)[S])
{
    const float2 c = *reinterpret_cast<const float2 *>(CS + 4 * L * NI);
#pragma unroll
    for (int i = 0; i < S; ++i) {
        zr[i] = c.x;
        zi[i] = c.y;
    }
    float Mk[4 * NI];
    lds_tap_load<NI>(CS, 0, Mk);
    int zo = 0;   // opaque zero of the next tap's address
#pragma unroll
    for (int k = 0; k < L; ++k) {
        float Mn[4 * NI];
        if (k + 1 < L) lds_tap_load<NI>(CS + zo, k + 1, Mn);
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int i = 0; i < S; ++i) {
            const int w = i + (L - 1) - k;
            float w00 = Mk[4 * (NI - 1) + 0], w01 = Mk[4 * (NI - 1) + 1];
            float w10 = Mk[4 * (NI - 1) + 2], w11 = Mk[4 * (NI - 1) + 3];
#pragma unroll
            for (int j = NI - 2; j >= 0; --j) {
                w00 = __builtin_fmaf(w00, s[w], Mk[4 * j + 0]);
                w01 = __builtin_fmaf(w01, s[w], Mk[4 * j + 1]);
                w10 = __builtin_fmaf(w10, s[w], Mk[4 * j + 2]);
                w11 = __builtin_fmaf(w11, s[w], Mk[4 * j + 3]);
            }
            zr[i] = __builtin_fmaf(w00, a[w], zr[i]);
            zr[i] = __builtin_fmaf(w01, b[w], zr[i]);
            zi[i] = __builtin_fmaf(w10, a[w], zi[i]);
            zi[i] = __builtin_fmaf(w11, b[w], zi[i]);
        }
        if (k + 2 < L) {
            // the reads of tap k + 2 wait for this tap's results: the selector
            // would move every tap's reads to the top, where the whole table
            // takes registers
#pragma unroll
            for (int i = 0; i < S; ++i) asm volatile("" : "+v"(zo) : "v"(zr[i]), "v"(zi[i]));
        }
        __builtin_amdgcn_sched_barrier(0);
        if (k + 1 < L) {
#pragma unroll
            for (int e = 0; e < 4 * NI; ++e) Mk[e] = Mn[e];
        }
    }
}

// fir_outputs with half of the table as scalar operands (M, the first column of
// each matrix) and half in VGPRs (from LDS, CS).  An FMA with a scalar operand
// cannot issue together with another wave's, FMAs of VGPRs alone draw more power
// and lower the clock (16 FMAs by each of two waves: 66 cycles all scalar, 46 to
// 49 all VGPR, 42 half and half), and half the table halves the LDS reads.  Each
// tap's entries are read when its turn comes: at four waves per SIMD the others
// cover the wait, and one buffer of them is what lets four fit (126 registers at NI
// = 5, L = 8, S = 8, against 156 with two buffers in VGPRs).
typedef float cvec4 __attribute__((ext_vector_type(4), aligned(4)));
typedef const __attribute__((address_space(4))) cvec4 ccvec4;

template <int NI, int L, int S>
__device__ __forceinline__ void fir_outputs_split(const float (&a)[S + L - 1], const float (&b)[S + L - 1],
                                                  const float (&s)[S + L - 1], const float *CS, const cfloat *M,
                                                  float (&zr)[S], float (&zi)[S])
{
    const float2 c = *reinterpret_cast<const float2 *>(CS + 4 * L * NI);
#pragma unroll
    for (int i = 0; i < S; ++i) {
        zr[i] = c.x;
        zi[i] = c.y;
    }
    // opaque zeros of the next tap's addresses
    int zv = 0, zs = 0;
    asm volatile("" : "+v"(zv));
    asm volatile("" : "+s"(zs));
#pragma unroll
    for (int k = 0; k < L; ++k) {
        float v0[NI], v1[NI], s0[NI], s1[NI];   // columns 1 and 0 of M_{j,k}
#pragma unroll
        for (int j = 0; j < NI; ++j) {
            const int e = 4 * (NI * k + j);
            v0[j] = CS[zv + e + 1];
            v1[j] = CS[zv + e + 3];
            const cvec4 u = *(ccvec4 *)(M + zs + e);
            s0[j] = u.x;
            s1[j] = u.z;
        }
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int i = 0; i < S; ++i) {
            const int w = i + (L - 1) - k;
            float w00 = s0[NI - 1], w01 = v0[NI - 1], w10 = s1[NI - 1], w11 = v1[NI - 1];
#pragma unroll
            for (int j = NI - 2; j >= 0; --j) {
                w00 = __builtin_fmaf(w00, s[w], s0[j]);
                w01 = __builtin_fmaf(w01, s[w], v0[j]);
                w10 = __builtin_fmaf(w10, s[w], s1[j]);
                w11 = __builtin_fmaf(w11, s[w], v1[j]);
            }
            zr[i] = __builtin_fmaf(w00, a[w], zr[i]);
            zr[i] = __builtin_fmaf(w01, b[w], zr[i]);
            zi[i] = __builtin_fmaf(w10, a[w], zi[i]);
            zi[i] = __builtin_fmaf(w11, b[w], zi[i]);
        }
        if (k + 1 < L) {
            // the reads of the next tap wait for this one's results (as in
            // fir_outputs_lds)
#pragma unroll
            for (int i = 0; i < S; ++i) asm volatile("" : "+v"(zv) : "v"(zr[i]), "v"(zi[i]));
            asm volatile("" : "+s"(zs) : "v"(zr[0]));
        }
        __builtin_amdgcn_sched_barrier(0);
    }
}

// Coefficient tables up to this many floats stay in registers in the
// streaming kernel (larger ones are read tap by tap, see fir_outputs_split).
constexpr int kRegCoefMax = 96;

template <int W>
__device__ __forceinline__ void split_window(const float2 (&win)[W], float (&a)[W], float (&b)[W],
                                             float (&s)[W])
{
#pragma unroll
    for (int w = 0; w < W; ++w) {
        a[w] = win[w].x;
        b[w] = win[w].y;
        s[w] = __builtin_fmaf(a[w], a[w], b[w] * b[w]);
    }
}

// Store S consecutive outputs starting at sample m0 (< n) of a row.
template <int S>
__device__ __forceinline__ void store_outputs(float2 *__restrict__ z, int64_t m0, int64_t n,
                                              bool full, const float (&zr)[S], const float (&zi)[S])
{
    if (full) {
        v4f_s *z4 = reinterpret_cast<v4f_s *>(z + m0);
#pragma unroll
        for (int i = 0; i < S / 2; ++i) {
            v4f_s v = {zr[2 * i], zi[2 * i], zr[2 * i + 1], zi[2 * i + 1]};
            __builtin_nontemporal_store(v, z4 + i);
        }
    } else {
#pragma unroll
        for (int i = 0; i < S; ++i)
            if (m0 + i < n) z[m0 + i] = make_float2(zr[i], zi[i]);
    }
}

// One-shot kernel (stage_lds = 0): each block computes one tile of kBlock*S
// outputs; every thread loads its own S+L-1 window with 16-byte loads (the
// halo part re-reads its neighbour's samples, which the vector L1 / L2 serve).
// S = 4: half of the table as scalar operands, half from LDS (fir_outputs_split;
// 2^22 samples at NI = 5: L = 12 25.7 us against 28.1 with all but the top Horner
// level scalar, L = 16 32.1 against 36.5; 2^23 at NI = L = 4 the same).  Otherwise
// the top level sits in VGPRs (an FMA takes one scalar operand) and the lower
// ones are scalar loads.  S = 2, the form of short calls, whose time is the chain
// of memory latencies: top level straight from scalar loads beside the window's,
// no barrier (3.06 us for 2^16 samples at NI = L = 4 against 3.13).  Larger S:
// through LDS, whose barrier starts the block's loads together (2^23 samples:
// 23.6 us against 25.4).
// PACK, for short rows: a tile is kBlock windows of S outputs, the windows of one
// row after those of the row before, so that no thread is left past a row's end
// and only a row's first and last windows are loaded sample by sample.
template <int NI, int L, int S, bool PACK>
__global__ void __launch_bounds__(kBlock) fwd_tile_kernel(FwdParams p)
{
    static_assert(S % 2 == 0, "S must be even (16-byte stores)");
    constexpr int T = kBlock * S;
    constexpr int HP = (L - 1 + 1) & ~1;   // halo rounded up to an even count
    constexpr int W = S + L - 1;
    constexpr int WL = HP + S;              // loaded samples (even)
    constexpr bool DIRECT = S == 2;
    constexpr bool SPLIT = S == 4;
    constexpr int NC = SPLIT ? 4 * L * NI + 2 : 4 * L;   // table floats in LDS
    __shared__ __align__(16) float ctab[DIRECT ? 1 : NC];
    const int tid = threadIdx.x;
    float top[4 * L];
    if constexpr (!DIRECT) {
        for (int e = tid; e < NC; e += kBlock)
            ctab[e] = p.M[SPLIT ? e : (e >> 2) * 4 * NI + 4 * (NI - 1) + (e & 3)];
        __syncthreads();
        if constexpr (!SPLIT) {
#pragma unroll
            for (int e = 0; e < 4 * L; ++e) top[e] = ctab[e];
        }
    }

    for (int64_t step = xcd_remap(blockIdx.x, gridDim.x); step < p.total_tiles; step += gridDim.x) {
        // a 64-bit division is a hundred instructions before the first load
        const int64_t at = PACK ? step * kBlock : step;   // window, tile
        int64_t row = (PACK ? at >> 32 : at >> 31) ? at / p.tiles_per_row
                                                   : (int64_t)((uint32_t)at / (uint32_t)p.tiles_per_row);
        int64_t m0;   // first output of this thread
        bool full;
        if constexpr (PACK) {
            const uint32_t w = (uint32_t)(at - row * p.tiles_per_row) + tid, q = w / (uint32_t)p.tiles_per_row;
            row += q;
            m0 = (int64_t)(w - q * (uint32_t)p.tiles_per_row) * S;
            if (row >= p.rows) return;   // the last tile: no barrier follows (no history)
            full = m0 + S <= p.n;
        } else {
            const int64_t t0 = (at - row * p.tiles_per_row) * (int64_t)T;
            full = t0 + T <= p.n;
            m0 = t0 + (int64_t)tid * S;
        }
        const float2 *__restrict__ x = p.in + row * p.ld;
        float2 *__restrict__ z = p.out + row * p.ld;
        const float2 *hist = !PACK && row == 0 ? p.hist : nullptr;

        float2 raw[WL];
        const int64_t lo = m0 - HP;
        if (full && lo >= 0) {
            const v4f_s *x4 = reinterpret_cast<const v4f_s *>(x + lo);
#pragma unroll
            for (int i = 0; i < WL / 2; ++i) {
                const v4f_s v = x4[i];
                raw[2 * i] = make_float2(v.x, v.y);
                raw[2 * i + 1] = make_float2(v.z, v.w);
            }
        } else {
#pragma unroll
            for (int i = 0; i < WL; ++i) raw[i] = sample_or_hist<L>(x, lo + i, p.n, hist);
        }
        float2 win[W];
#pragma unroll
        for (int w = 0; w < W; ++w) win[w] = raw[HP - (L - 1) + w];
        float a[W], b[W], s[W];
        split_window<W>(win, a, b, s);
        float zr[S], zi[S];
        const cfloat *M = as_const(p.M);
        if constexpr (DIRECT) {
#pragma unroll
            for (int e = 0; e < 4 * L; ++e) {
                top[e] = M[(e >> 2) * 4 * NI + 4 * (NI - 1) + (e & 3)];
                asm("" : "+v"(top[e]));
            }
        }
        if constexpr (SPLIT)
            fir_outputs_split<NI, L, S>(a, b, s, ctab, M, zr, zi);
        else
            fir_outputs<NI, L, S>(a, b, s, top, M, zr, zi);
        if (m0 < p.n) store_outputs<S>(z, m0, p.n, full, zr, zi);
        if (!PACK && L > 1 && p.hist != nullptr && step == 0) {
            // a carried history is read by this block alone; replace it once
            // every thread has
            __syncthreads();
            if (tid < L - 1) {
                const int64_t m = p.n - (L - 1) + tid;
                const float2 v = m >= 0 ? p.in[m] : p.hist[L - 1 + m];
                raw[0] = v;
            }
            __syncthreads();
            if (tid < L - 1) p.hist[tid] = raw[0];
        }
    }
}

// Compiler-only ordering point for LDS and global traffic between the lanes of one
// wave.  A wave's memory instructions of a kind execute in program order, so no
// wait is needed; this only stops the compiler from moving accesses across it.
__device__ __forceinline__ void wave_lds_order()
{
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// Wave priority of a persistent wave with `left` of `all` chunks to go: more for
// waves that are behind.  The waves of a SIMD are served oldest first, so without
// it one runs ahead and the last works alone at the end, where a single wave
// issues half of what two do.  2^26 samples at NI = 5, L = 8: 294 -> 282 us with
// three blocks per CU; with four and fir_outputs_split 271 (NI = 4, L = 8: 262 ->
// 235; NI = 4, L = 6: 225 -> 198; L = 16: 538 -> 485, three blocks).
__device__ __forceinline__ void progress_prio(int64_t left, int64_t all)
{
    if (2 * left > all) {
        if (4 * left > 3 * all)
            __builtin_amdgcn_s_setprio(3);
        else
            __builtin_amdgcn_s_setprio(2);
    } else if (4 * left > all) {
        __builtin_amdgcn_s_setprio(1);
    } else {
        __builtin_amdgcn_s_setprio(0);
    }
}

// Streaming kernel (stage_lds = 1).  Persistent grid of waves; at every step
// the waves of the grid work on adjacent chunks of C = 64*S samples (wave g
// takes chunks g, g + nw, g + 2 nw, ... of the flattened rows), so the whole
// chip sweeps memory in order.  Per chunk:
//   * the next chunk is already in flight (register prefetch); every
//     load instruction is a nontemporal read of 1 KiB of contiguous memory
//     (lane l, part i -> the 16 bytes at sample 2*(l + 64 i)); the L-1 halo
//     samples before the chunk are read by the first L-1 lanes, one each (a
//     vector load, in order with the chunk's; zeros at a row start, the
//     caller's history before row 0);
//   * samples and |x|^2 go to a wave-private LDS buffer laid out with one pad
//     slot after every S samples (odd lane stride: conflict-free window reads);
//     each lane reads its S+L-1 consecutive-sample window back, filters and
//     stores 16-byte outputs.
// The loop body has no divergent global accesses and no conditional loads, so
// the compiler's counter waits stay exact.  When C does not divide n, the last
// chunk of a row is the row's last C samples: the samples it shares with the
// chunk before come out the same there (each output is computed by itself, in
// one order), and the two waves store the same bits.  Only rows shorter than
// C + L - 1 samples take the guarded code after the loop for their end (a last
// chunk starting inside the first L - 1 samples would need part of the
// history).  No block-wide barrier after the coefficient staging.
// A carried history (dpd_apply_hist) is read only by the wave of row 0's first
// chunk, wave 0, which replaces it by the last L - 1 inputs once it has read it.
template <int S>
struct ChunkRegs {
    float4 v[S / 2];
    float2 h;   // raw halo sample for this lane's slot (selected at use)
};

// LDS slot of window sample d (relative to the chunk start, d >= -(L-1)).
template <int L, int S>
struct PadLayout {
    static constexpr int HG = (L - 1 + S - 1) / S;          // pad groups before the chunk
    static constexpr int OFF = HG * (S + 1);                // slot of sample 0
    static constexpr int SLOTS = OFF + 64 * (S + 1);
    __device__ static constexpr int slot(int d)
    {
        return OFF + d + (d >= 0 ? d / S : -((-d + S - 1) / S));
    }
};

// Blocks per CU the registers are held to: four where the table is read tap by tap
// and the window is small enough (NI = 5, L = 8 would take one register more than
// 128; larger filters would spill).
template <int NI, int L>
constexpr int fwd_stream_blocks()
{
    return 4 * L * NI + 2 > kRegCoefMax && L <= kSpecL && NI + L <= 14 ? 4 : 1;
}

template <int NI, int L, int S>
__global__ void __launch_bounds__(kBlock, (fwd_stream_blocks<NI, L>())) fwd_stream_kernel(FwdParams p)
{
    static_assert(S % 2 == 0, "S must be even (16-byte loads and stores)");
    constexpr int C = 64 * S;
    constexpr int W = S + L - 1;
    constexpr int NV = S / 2;
    constexpr int WAVES = kBlock / 64;
    using PL = PadLayout<L, S>;
    constexpr int HS = L - 1;                        // halo samples
    constexpr int NC = 4 * L * NI + 2;               // coefficient table floats
    constexpr bool REG = NC <= kRegCoefMax;          // whole table in registers
    __shared__ __align__(16) float ctab[NC];
    __shared__ __align__(16) float2 xs[WAVES][PL::SLOTS];
    __shared__ __align__(16) float ss[WAVES][PL::SLOTS];

    const int tid = threadIdx.x, lane = tid & 63;
    const int wv = __builtin_amdgcn_readfirstlane(tid >> 6);   // uniform per wave
    for (int e = tid; e < NC; e += kBlock) ctab[e] = p.M[e];
    __syncthreads();
    float coef[REG ? NC : 1];
    if constexpr (REG) {
#pragma unroll
        for (int e = 0; e < NC; ++e) coef[e] = ctab[e];
    }

    float2 *X = xs[wv];
    float *SX = ss[wv];
    const int64_t rows = p.total_tiles / p.tiles_per_row;
    // chunks per row of the main loop, the last one moved back to the row's end
    const bool whole = p.n % C == 0 || p.n >= C + HS;
    const int64_t tpr = whole ? (p.n + C - 1) / C : p.n / C;
    const int64_t t_end = p.n - C;
    const auto start = [&](int64_t k) { return k * C < t_end ? k * C : t_end; };
    const int64_t total = rows * tpr;
    const int64_t nw = (int64_t)gridDim.x * WAVES;
    const int64_t gw = (int64_t)xcd_remap(blockIdx.x, gridDim.x) * WAVES + wv;
    // halo sample this lane fetches: d = hl - HS in [-(L-1), -1]
    const int hl = HS > 0 ? (lane < HS ? lane : HS - 1) : 0;
    float2 hist_v = make_float2(0.f, 0.f);
    if (HS > 0 && p.hist != nullptr && gw == 0) {
        // every lane reads before any lane replaces: for n < L - 1 the sample that
        // a lane keeps is another lane's to overwrite
        hist_v = p.hist[hl];
        const int64_t m = p.n - HS + hl;
        const float2 v = *(m >= 0 ? p.in + m : p.hist + (HS + m));
        wave_lds_order();
        if (lane < HS) p.hist[lane] = v;
    }

    // raw sample for halo sample hl - HS of the chunk starting at t0 (lane hl
    // selects its own sample; the compiler makes it one per-lane load).  At a
    // row start (t0 < HS) nothing is read; the value is replaced at use.
    auto halo_raw = [&](int64_t row, int64_t t0) {
        float2 r = make_float2(0.f, 0.f);
        if (HS > 0 && t0 >= HS) {
            const cfloat *hp = as_const(reinterpret_cast<const float *>(p.in + row * p.ld + t0 - HS));
            r = make_float2(hp[0], hp[1]);
#pragma unroll
            for (int k = 1; k < (HS > 0 ? HS : 1); ++k)
                if (hl == k) r = make_float2(hp[2 * k], hp[2 * k + 1]);
        }
        return r;
    };
    // The same for a full chunk (row length >= C > HS): always read, from the
    // row start when t0 < HS, so the loop issues the same loads on every trip.
    auto halo_raw_full = [&](int64_t row, int64_t t0) {
        const int64_t off = t0 >= HS ? t0 - HS : 0;
        const cfloat *hp = as_const(reinterpret_cast<const float *>(p.in + row * p.ld + off));
        float2 r = make_float2(hp[0], hp[1]);
#pragma unroll
        for (int k = 1; k < (HS > 0 ? HS : 1); ++k)
            if (hl == k) r = make_float2(hp[2 * k], hp[2 * k + 1]);
        return r;
    };

    // samples -> LDS, windows -> registers, filter
    auto filter_chunk = [&](const ChunkRegs<S> &buf, int64_t row, int64_t t0, float (&zr)[S],
                            float (&zi)[S]) {
        wave_lds_order();
        if (HS > 0 && lane < HS) {
            float2 h = buf.h;
            if (t0 - HS + lane < 0) h = row == 0 ? hist_v : make_float2(0.f, 0.f);
            const int q = PL::slot(lane - HS);
            X[q] = h;
            SX[q] = __builtin_fmaf(h.x, h.x, h.y * h.y);
        }
#pragma unroll
        for (int i = 0; i < NV; ++i) {
            const float4 v = buf.v[i];
            const int j = 2 * (lane + 64 * i);           // even, same pad group as j + 1
            const int q = PL::OFF + j + j / S;
            X[q] = make_float2(v.x, v.y);
            X[q + 1] = make_float2(v.z, v.w);
            SX[q] = __builtin_fmaf(v.x, v.x, v.y * v.y);
            SX[q + 1] = __builtin_fmaf(v.z, v.z, v.w * v.w);
        }
        wave_lds_order();
        float a[W], b[W], s[W];
        const int lb = lane * (S + 1);
#pragma unroll
        for (int w = 0; w < W; ++w) {
            const int q = lb + PL::slot(w - (L - 1));
            const float2 v = X[q];
            a[w] = v.x;
            b[w] = v.y;
            s[w] = SX[q];
        }
        if constexpr (REG)
            fir_outputs_reg<NI, L, S>(a, b, s, coef, zr, zi);
        else
            fir_outputs_split<NI, L, S>(a, b, s, ctab, as_const(p.M), zr, zi);
    };

    // Store the S outputs of every lane of a full chunk.  S = 2: each lane's
    // 16 bytes are adjacent to its neighbour's, so the store instruction already
    // writes 1 KiB contiguously.  S > 2: the outputs go back through the wave's
    // LDS buffer and leave in the load order (lane l, part i -> samples
    // 2*(l + 64 i)), so every store writes whole cache lines.
    auto store_chunk = [&](float2 *zrow, int64_t t0, const float (&zr)[S], const float (&zi)[S]) {
        if constexpr (S == 2) {
            store_outputs<S>(zrow, t0 + lane * S, p.n, true, zr, zi);
        } else {
            wave_lds_order();
            const int lb = lane * (S + 1) + PL::OFF;
#pragma unroll
            for (int i = 0; i < S; ++i) X[lb + i] = make_float2(zr[i], zi[i]);
            wave_lds_order();
            v4f_s *z4 = reinterpret_cast<v4f_s *>(zrow + t0);
#pragma unroll
            for (int i = 0; i < NV; ++i) {
                const int j = 2 * (lane + 64 * i);
                const int q = PL::OFF + j + j / S;
                const float2 u = X[q], w = X[q + 1];
                const v4f_s v = {u.x, u.y, w.x, w.y};
                __builtin_nontemporal_store(v, z4 + lane + 64 * i);
            }
        }
    };

    // ---- main loop over whole chunks gw, gw + nw, ...
    if (gw < total) {
        // chunk c <-> (row, k); advancing by nw chunks without dividing
        const int64_t dr = nw / tpr, dk = nw - (nw / tpr) * tpr;
        struct Cur {
            int64_t row, k;
        };
        auto next = [&](Cur u) {
            u.row += dr;
            u.k += dk;
            if (u.k >= tpr) {
                u.k -= tpr;
                ++u.row;
            }
            return u;
        };
        int64_t left = (total - 1 - gw) / nw + 1;    // chunks of this wave
        const int64_t all = left;
        // The prefetch issues at raised wave priority, so a wave reaching it
        // is not held behind the other waves' filter work on the SIMD
        // (measured: 47.8 -> 47.2 us at the 2^24 headline, outputs unchanged).
        auto load_full = [&](ChunkRegs<S> &buf, const Cur &u) {
            __builtin_amdgcn_s_setprio(3);
            const int64_t t0 = start(u.k);
            const v4f_s *x4 = reinterpret_cast<const v4f_s *>(p.in + u.row * p.ld + t0);
#pragma unroll
            for (int i = 0; i < NV; ++i) {
                // read once: nontemporal (streaming) loads
                const v4f_s t = __builtin_nontemporal_load(x4 + lane + 64 * i);
                buf.v[i] = make_float4(t.x, t.y, t.z, t.w);
            }
            buf.h = halo_raw_full(u.row, t0);
            progress_prio(left, all);
        };
        auto step = [&](const ChunkRegs<S> &buf, const Cur &u) {
            float zr[S], zi[S];
            const int64_t t0 = start(u.k);
            filter_chunk(buf, u.row, t0, zr, zi);
            store_chunk(p.out + u.row * p.ld, t0, zr, zi);
        };
        // Two chunks per trip with the next one always in flight; the loop
        // body is straight-line code (exact counter waits) and the last one
        // or two chunks are peeled off, so nothing is read past the run.
        Cur cur;
        cur.row = gw / tpr;
        cur.k = gw - cur.row * tpr;
        ChunkRegs<S> A, B;
        load_full(A, cur);
        for (; left >= 3; left -= 2) {
            const Cur c1 = next(cur);
            load_full(B, c1);
            step(A, cur);
            const Cur c2 = next(c1);
            load_full(A, c2);
            step(B, c1);
            cur = c2;
        }
        if (left == 2) {
            const Cur c1 = next(cur);
            load_full(B, c1);
            step(A, cur);
            step(B, c1);
        } else {
            step(A, cur);
        }
    }

    // ---- the end of rows too short for a moved last chunk
    if (tpr * C < p.n) {
        for (int64_t rw = gw; rw < rows; rw += nw) {
            const int64_t t0 = tpr * C;
            const float2 *x = p.in + rw * p.ld;
            ChunkRegs<S> buf;
#pragma unroll
            for (int i = 0; i < NV; ++i) {
                const int64_t m = t0 + 2 * (lane + 64 * i);
                const float2 u = m < p.n ? x[m] : make_float2(0.f, 0.f);
                const float2 w = m + 1 < p.n ? x[m + 1] : make_float2(0.f, 0.f);
                buf.v[i] = make_float4(u.x, u.y, w.x, w.y);
            }
            buf.h = halo_raw(rw, t0);
            float zr[S], zi[S];
            filter_chunk(buf, rw, t0, zr, zi);
            const int64_t m0 = t0 + (int64_t)lane * S;
            float2 *z = p.out + rw * p.ld;
#pragma unroll
            for (int i = 0; i < S; ++i)
                if (m0 + i < p.n) z[m0 + i] = make_float2(zr[i], zi[i]);
        }
    }
}


int num_cus();

template <int NI, int L, int S, bool STREAM, bool PACK = false>
hipError_t launch_fwd(const FwdParams &p, hipStream_t stream, int grid_mult)
{
    int64_t grid;
    if constexpr (STREAM) {
        // persistent: grid_mult blocks per CU, never more than one chunk per wave
        // never more blocks than can be resident at once (a second round of a
        // persistent grid would double the tail)
        static const int occ = [] {
            int o = 0;
            if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&o, fwd_stream_kernel<NI, L, S>, kBlock,
                                                             0) != hipSuccess || o < 1)
                o = 1;
            return o;
        }();
        const int64_t want = (int64_t)num_cus() * (grid_mult < occ ? grid_mult : occ);
        const int64_t need = (p.total_tiles + kBlock / 64 - 1) / (kBlock / 64);   // >= 1 wave per chunk
        grid = need < want ? need : want;
        hipLaunchKernelGGL((fwd_stream_kernel<NI, L, S>), dim3((uint32_t)grid),
                           dim3(kBlock), 0,
                           stream, p);
    } else {
        const int64_t cap = 1 << 20;
        grid = p.total_tiles < cap ? p.total_tiles : cap;
        hipLaunchKernelGGL((fwd_tile_kernel<NI, L, S, PACK>), dim3((uint32_t)grid), dim3(kBlock), 0,
                           stream, p);
    }
    return hipGetLastError();
}

// Up to kSpecL taps: every launch shape.  More taps: one-shot at S = 2 and S = 4,
// streaming at S = 8.
template <int NI, int L>
void register_fwd_one(FwdTable &t)
{
    t.rows[NI - 1][L - 1][0] = &launch_fwd<NI, L, 2, false, true>;
    t.rows[NI - 1][L - 1][1] = &launch_fwd<NI, L, 4, false, true>;
    if constexpr (L > kSpecL) {
        for (int v = 0; v < kNumFwdVariants; ++v)
            t.fn[NI - 1][L - 1][v] = (v & 1)  ? &launch_fwd<NI, L, 8, true>
                                     : v == 0 ? &launch_fwd<NI, L, 2, false>
                                              : &launch_fwd<NI, L, 4, false>;
    } else {
    t.fn[NI - 1][L - 1][0] = &launch_fwd<NI, L, 2, false>;
    t.fn[NI - 1][L - 1][1] = &launch_fwd<NI, L, 2, true>;
    t.fn[NI - 1][L - 1][2] = &launch_fwd<NI, L, 4, false>;
    t.fn[NI - 1][L - 1][3] = &launch_fwd<NI, L, 4, true>;
    t.fn[NI - 1][L - 1][4] = &launch_fwd<NI, L, 8, false>;
    t.fn[NI - 1][L - 1][5] = &launch_fwd<NI, L, 8, true>;
    }
}

}  // namespace dpd
