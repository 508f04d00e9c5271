// Host side of the backward pass (dpd_backward, dpd_backward_ws_size) and the
// FP64 finalisation.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstring>
#include <mutex>

#include "dpd.h"
#include "dpd_bwd_kernels.h"
#include "dpd_plan.h"

#define DPD_EXPORT extern "C" __attribute__((visibility("default")))

namespace dpd {

int num_cus();

static BwdTable g_bwd;
static std::once_flag g_bwd_once;

static const BwdTable &bwd_table()
{
    std::call_once(g_bwd_once, [] {
        std::memset(&g_bwd, 0, sizeof(g_bwd));
        register_bwd_ni1(g_bwd);
        register_bwd_ni2(g_bwd);
        register_bwd_ni3(g_bwd);
        register_bwd_ni4(g_bwd);
        register_bwd_ni5(g_bwd);
        register_bwd_ni6(g_bwd);
        register_bwd_ni7(g_bwd);
        register_bwd_ni8(g_bwd);
    });
    return g_bwd;
}

// Resident blocks per CU of a specialised backward kernel (cached).
static int bwd_occupancy(int NI, int L, int want)
{
    static int cache[kSpecNI][kMaxL][4] = {};
    static std::mutex mu;
    std::lock_guard<std::mutex> lk(mu);
    int &o = cache[NI - 1][L - 1][want];
    if (o == 0) {
        int v = 0;
        if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&v, bwd_table().kern[NI - 1][L - 1][want],
                                                         kBlock, 0) != hipSuccess || v < 1)
            v = 1;
        o = v;
    }
    return o;
}

// Coefficient-gradient finalisation: block q sums, in FP64, the partials of
// the four entries of table matrix q = k*NI + j (block L*NI: the two entries
// of c) over all nblk producer blocks -- thread t takes producers t, t + 256,
// ... in order, then the DPP lane sum of each wave and the four waves in
// order, so the result is bitwise reproducible -- and applies the chain rule
// through M = [[hr+gr, gi-hi], [hi+gi, hr-gr]] to the main and conjugate
// coefficients of order 2j+1, tap k (section 2.2 layout):
//   u1 = dE/dm00, u4 = dE/dm01, u3 = dE/dm10, u2 = dE/dm11
//   grad h    = (u1 + u2) + j (u3 - u4)
//   grad hbar = (u1 - u2) + j (u3 + u4)
//   grad c    = sum G
__global__ void __launch_bounds__(kBlock) bwd_finalize(const float *__restrict__ partials, int nblk,
                                                       CoefMap map, float2 *__restrict__ gcoef)
{
    __shared__ double red[kBlock / 64][4];
    double u[4];
    dcoef_block_sums(partials, nblk, map, blockIdx.x, red, u);
    if (threadIdx.x != 0) return;
    int idx[2];
    float2 g[2];
    const int c = dcoef_block_grads(map, blockIdx.x, u, idx, g);
    for (int i = 0; i < c; ++i) gcoef[idx[i]] = g[i];
}

// dE/dx alone of a memoryless linear plan (NI = L = 1: an I/Q stage), G M^T, on rows
// shorter than a chunk: one sample per thread and step, so that no lane idles past
// a row's end (262144 rows of 63 samples 93 us in bwd_kernel, 73 here; 65536 of 255 97
// and 73).  The bits of bwd_kernel's dE/dx.
constexpr int kLinearU = 4;   // samples per thread
__global__ void __launch_bounds__(kBlock) bwd_dx_linear_kernel(BwdParams p)
{
    float M[4];
#pragma unroll
    for (int e = 0; e < 4; ++e) M[e] = table_entry(p.M, p.raw, p.map, e);
    const int64_t total = p.rows * p.n, per = (int64_t)kBlock * kLinearU;
    for (int64_t at = blockIdx.x * per; at < total; at += gridDim.x * per) {
        float2 g[kLinearU], v[kLinearU];
        int64_t to[kLinearU];
#pragma unroll
        for (int u = 0; u < kLinearU; ++u) {
            const int64_t i = at + u * kBlock + threadIdx.x;
            const int64_t row = total >> 31 ? i / p.n : (int64_t)((uint32_t)i / (uint32_t)p.n);
            to[u] = i < total ? row * p.ld + (i - row * p.n) : -1;
            g[u] = v[u] = make_float2(0.f, 0.f);
            if (to[u] >= 0) {
                g[u] = p.gz[to[u]];
                v[u] = p.x[to[u]];
            }
        }
#pragma unroll
        for (int u = 0; u < kLinearU; ++u) {
            const float a = __builtin_fmaf(M[2], g[u].y, M[0] * g[u].x), b = __builtin_fmaf(M[3], g[u].y, M[1] * g[u].x);
            // + 0 v as in bwd_kernel: not finite where x is not
            if (to[u] >= 0) p.gx[to[u]] = make_float2(__builtin_fmaf(0.f, v[u].x, a), __builtin_fmaf(0.f, v[u].y, b));
        }
    }
}

static int64_t grid_cap() { return (int64_t)num_cus() * 8; }

size_t bwd_ws_bytes(const CoefMap &map)
{
    const int64_t E = 4 * map.L * map.NI + 2;
    return (size_t)(grid_cap() * E * (int64_t)sizeof(float) + 256);
}

hipError_t launch_bwd_finalize(const float *partials, int nblk, const CoefMap &map, float2 *grad_coeffs,
                               hipStream_t st)
{
    hipLaunchKernelGGL(bwd_finalize, dim3((uint32_t)(map.L * map.NI + 1)), dim3(kBlock), 0, st, partials, nblk,
                       map, grad_coeffs);
    return hipGetLastError();
}

}  // namespace dpd

using namespace dpd;

DPD_EXPORT dpd_status dpd_backward_ws_size(const dpd_plan *plan, int64_t rows, int64_t n, size_t *bytes)
{
    if (plan == nullptr || bytes == nullptr || rows < 0 || n < 0) return DPD_EINVAL;
    *bytes = bwd_ws_bytes(plan->map);
    return DPD_OK;
}

static dpd_status backward_impl(dpd_plan *plan, void *stream, const void *coeffs_dev, const void *x,
                                const void *grad_z, void *grad_x, void *grad_coeffs, int64_t rows,
                                int64_t n, int64_t ld, void *ws, size_t ws_bytes)
{
    if (plan == nullptr) return DPD_EINVAL;
    if (rows == 1 && ld < n) ld = n;
    if (n < 0 || rows < 0 || (rows > 1 && ld < n)) return DPD_EINVAL;
    const CoefMap &map = plan->map;
    const hipStream_t st = (hipStream_t)stream;
    const bool want_dx = grad_x != nullptr, want_dc = grad_coeffs != nullptr;
    const bool empty = n == 0 || rows == 0;
    if (!empty && (x == nullptr || grad_z == nullptr)) return DPD_EINVAL;
    for (const void *q : {x, grad_z, (const void *)grad_x, (const void *)grad_coeffs, coeffs_dev})
        if ((uintptr_t)q % 8 != 0) return DPD_EINVAL;
    if (want_dc && (ws == nullptr || ws_bytes < bwd_ws_bytes(map) || (uintptr_t)ws % 4 != 0))
        return DPD_EINVAL;
    if (want_dx && !empty) {
        const size_t span = (size_t)(((rows - 1) * ld + n) * 8);
        auto ov = [&](const void *a, const void *b) {
            const uintptr_t p = (uintptr_t)a, q = (uintptr_t)b;
            return p < q + span && q < p + span;
        };
        if (ov(grad_x, x) || ov(grad_x, grad_z)) return DPD_EINVAL;
    }
    if (!want_dx && !want_dc) return DPD_OK;

    BwdParams p;
    p.x = (const float2 *)x;
    p.gz = (const float2 *)grad_z;
    p.gx = (float2 *)grad_x;
    p.partials = (float *)ws;
    p.E = 4 * map.L * map.NI + 2;
    p.n = n;
    p.ld = ld;
    p.rows = rows;
    // only dx reads the coefficients: dE/dcoeffs is the correlation of grad_z
    // with the basis of x alone
    p.M = plan->d_table;
    p.raw = (const float2 *)coeffs_dev;
    p.map = map;
    const bool even = (uintptr_t)x % 16 == 0 && (uintptr_t)grad_z % 16 == 0 && (uintptr_t)grad_x % 16 == 0 &&
                      (rows == 1 || ld % 2 == 0);
    p.fine = !even || map.L > kSpecL;
    p.flush = p.fine ? (int32_t)bwd_flush_fine(rows * n) : kBwdFlush;
    int nblk = 0;
    if (!empty) {
        const int64_t C = 64 * kBwdS;
        p.tpr = n / C;
        // Rows that fit a chunk more than twice are taken several at a time (65536 rows of
        // 33 samples at NI = L = 4, both gradients: 31 us, a chunk each 76; longer ones
        // would straddle chunks: 65536 x 254 124 and 100).
        p.pack = 2 * (n + map.L - 1) <= 240 && ld <= (int64_t)1 << 20;
        const int64_t chunks = p.pack ? (rows * (n + map.L - 1) + C - 1) / C : rows * ((n + C - 1) / C);
        const BwdTable &t = bwd_table();
        const auto grid_of = [&](int L, int want) {
            const int64_t cap = (int64_t)num_cus() * std::min(8, bwd_occupancy(map.NI, L, want));
            return (int)std::max<int64_t>(1, std::min(cap, want == 3 ? (rows * n + kBlock - 1) / kBlock : (chunks + 3) / 4));
        };
        // the kernel of the coefficient gradient alone (bwd_dc_short_kernel says why)
        const int dc = p.fine && rows * n < kBwdShort ? 3 : 1;
        hipError_t e = hipSuccess;
        // Both gradients of a filter whose registers leave one block per CU: on
        // long inputs two kernels of two and more blocks are faster, though they
        // read the samples twice (NI = 4, L = 8, 2^24 samples: 198 us and 161, 7 * 2^20
        // 92 and 82; NI = 5, L = 8: 242 and 213, 112 and 103).  Short ones pay for the
        // second launch (2^20 samples: 22 us and 25, 26 and 29; at 2^21 both are equal, at
        // 2^22, on this side of the line, two would be 4 to 13 % faster).
        // Likewise where only the kernel of dx alone sums by Horner, and where that of
        // dcoef is another one.
        const bool apart = want_dx && want_dc && map.L <= kSpecL &&
                           ((rows * n >= (int64_t)6 << 20 && bwd_occupancy(map.NI, map.L, 2) == 1) ||
                            (p.fine && !bwd_horner(map.NI, true, true)) || dc == 3);
        if (want_dx && !want_dc && map.NI * map.L == 1 && n < 64 * kBwdS) {
            const int64_t per = (int64_t)kBlock * kLinearU;
            hipLaunchKernelGGL(bwd_dx_linear_kernel, dim3((uint32_t)std::min<int64_t>((rows * n + per - 1) / per, 1 << 20)),
                               dim3(kBlock), 0, st, p);
            e = hipGetLastError();
        } else if (apart) {
            e = t.fn[map.NI - 1][map.L - 1][0](p, st, grid_of(map.L, 0));
            nblk = grid_of(map.L, dc);
            if (e == hipSuccess) e = t.fn[map.NI - 1][map.L - 1][dc](p, st, nblk);
        } else if (map.L <= kSpecL) {
            const int want = want_dx && want_dc ? 2 : (want_dc ? dc : 0);
            nblk = grid_of(map.L, want);
            e = t.fn[map.NI - 1][map.L - 1][want](p, st, nblk);
        } else {
            if (want_dx) e = t.fn[map.NI - 1][map.L - 1][0](p, st, grid_of(map.L, 0));
            if (want_dc) {
                // two passes over the taps, the same blocks in both
                nblk = grid_of(kSpecL, dc);
                if (e == hipSuccess) e = t.fn[map.NI - 1][kSpecL - 1][dc](p, st, nblk);
                if (e == hipSuccess) e = t.tail[map.NI - 1][map.L - kSpecL - 1][dc == 3](p, st, nblk);
            }
        }
        if (e != hipSuccess) return hip_fail(e);
    }
    if (want_dc) {
        hipLaunchKernelGGL(bwd_finalize, dim3((uint32_t)(map.L * map.NI + 1)), dim3(kBlock), 0, st,
                           (const float *)ws, nblk, map, (float2 *)grad_coeffs);
        hipError_t e = hipGetLastError();
        if (e != hipSuccess) return hip_fail(e);
    }
    return DPD_OK;
}

DPD_EXPORT dpd_status dpd_backward(dpd_plan *plan, void *stream, const void *coeffs_dev, const void *x,
                                   const void *grad_z, void *grad_x, void *grad_coeffs, int64_t rows,
                                   int64_t n, int64_t ld, void *ws, size_t ws_bytes)
{
    return backward_impl(plan, stream, coeffs_dev, x, grad_z, grad_x, grad_coeffs, rows, n, ld, ws, ws_bytes);
}

// ------------------------------------------------------------ no-allocation --
// Fixed device scratch for dpd_backward_noalloc: the per-block FP32 partials of
// the coefficient gradient (at most kMaxBwdScratch bytes; every plan on a
// 256-CU device needs <= 2048 blocks x 514 entries x 4 bytes + 256).  Each GPU
// holds its own copy of the array for the life of the process.  In host code
// the name `scratch` is only a host-side stand-in: its device address comes
// from hipGetSymbolAddress, once per device.
constexpr size_t kMaxBwdScratch = (size_t)17 << 18;   // 4.25 MiB
static __device__ __align__(256) unsigned char scratch[kMaxBwdScratch];

constexpr int kMaxScratchDevices = 64;
static std::mutex g_scratch_mu;
static void *g_scratch_addr[kMaxScratchDevices] = {};

// Device address of `scratch` on the current device (looked up on the first
// call on that device, with that device current).
static dpd_status scratch_address(void **out)
{
    int dev = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return hip_fail(e);
    if (dev < 0 || dev >= kMaxScratchDevices) return DPD_EUNSUPPORTED;
    std::lock_guard<std::mutex> lock(g_scratch_mu);
    if (g_scratch_addr[dev] == nullptr) {
        void *p = nullptr;
        e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
        if (e != hipSuccess) return hip_fail(e);
        if (p == nullptr) return DPD_EHIP;
        g_scratch_addr[dev] = p;
    }
    *out = g_scratch_addr[dev];
    return DPD_OK;
}

DPD_EXPORT dpd_status dpd_backward_noalloc(dpd_plan *plan, void *stream, const void *coeffs_dev, const void *x,
                                           const void *grad_z, void *grad_x, void *grad_coeffs, int64_t rows,
                                           int64_t n, int64_t ld)
{
    if (plan == nullptr) return DPD_EINVAL;
    if (grad_coeffs == nullptr)   // no coefficient gradient: no scratch is used
        return backward_impl(plan, stream, coeffs_dev, x, grad_z, grad_x, nullptr, rows, n, ld, nullptr, 0);
    if (bwd_ws_bytes(plan->map) > kMaxBwdScratch) return DPD_EUNSUPPORTED;
    void *ws = nullptr;
    dpd_status st = scratch_address(&ws);
    if (st != DPD_OK) return st;
    return backward_impl(plan, stream, coeffs_dev, x, grad_z, grad_x, grad_coeffs, rows, n, ld, ws,
                         kMaxBwdScratch);
}
