// Host side of the coefficient-learning step: the forward pass
// (dpd_transmit_loss_grad), the backward pass (dpd_transmit_backward) and the
// whole step (dpd_learn_step) over the kernels of dpd_learn_kernels.h, and the
// finalisation of loss, gradient and Adam.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <cstring>
#include <mutex>

#include "dpd.h"
#include "dpd_learn_kernels.h"
#include "dpd_plan.h"

#define DPD_EXPORT extern "C" __attribute__((visibility("default")))

namespace dpd {

int num_cus();

static const LnTable &ln_table()
{
    static const LnTable t = [] {
        LnTable r;
        std::memset(&r, 0, sizeof(r));
        register_learn_ni1(r);
        register_learn_ni2(r);
        register_learn_ni3(r);
        register_learn_ni4(r);
        register_learn_ni5(r);
        return r;
    }();
    return t;
}

// How a pass walks the rows.  Four samples per lane: half the registers of a chunk's
// windows and half its chain (64 rows of 2^18 samples, four against eight: one pass
// 145 us and 139 at NI = 4, L = 6, 165 and 199 at L = 8, where eight spills; the
// backward pass 97 and 100, 107 and 116; 4 x 4096: 15.6 and 18.2, 11.6 and 13.2).
// Eight, which reads a lane's window again half as often, where one block per CU
// has room for it (NI = 5, L = 8: one pass 255 and 270 us, backward 149 and 158) and
// waves have more than a chunk or two (4 x 4096: 18.6 and 23.2), and in the forward
// pass on rows of any length, whose sums no other pass has to match.
static int ln_walk(int mode, int64_t rows, int64_t n, int E)
{
    if (n % 256 != 0) return mode == kLnBwd ? kLn4Any : kLn8Any;
    return ln_blocks(kLnBoth, E) == 1 && n % 512 == 0 && rows * n > (int64_t)1 << 19 ? kLn8 : kLn4;
}

// One pass over the data; *nblk receives the number of blocks (and gradient
// partials), *nloss that of loss partials.  One round of resident blocks, on rows of
// whole 256s the same in every mode -- the blocks per CU that the kernels with a
// gradient are built for -- so that the partial sums, and with them loss and
// gradient, come out the same whether the step runs as one pass or two; the forward
// pass has twice as many where a run has two parts (ln_parts).  Arguments already
// validated.
static hipError_t ln_run(int mode, const dpd_plan *P, const dpd_plan *A, const dpd_plan *B, hipStream_t hs,
                         const void *coeffs_dev, const void *x, const void *z, const void *grad_y, void *grad_z,
                         int64_t rows, int64_t n, int64_t ld, float scale, float *lpart, float *gpart, int32_t *step,
                         bool fine, int *nblk, int *nloss)
{
    *nblk = *nloss = 0;
    const int64_t N = rows * n;
    LnParams p;
    p.M = P->d_table;
    p.raw = (const float2 *)coeffs_dev;
    p.map = P->map;
    p.A = A->d_table;
    p.B = B->d_table;
    p.x = (const float2 *)x;
    p.z = (float2 *)const_cast<void *>(z);
    p.gy = (float2 *)const_cast<void *>(grad_y);
    p.gz = (float2 *)grad_z;
    p.lpart = lpart;
    p.gpart = gpart;
    p.rows = rows;
    p.n = n;
    p.ld = rows > 1 ? ld : n;
    const int NI = P->map.NI, L = P->map.L, E = 4 * L * NI + 2;
    const int walk = ln_walk(mode, rows, n, E), S = ln_s(walk), C = 64 * S;
    p.tpr = (n + C - 1) / C;
    p.scale = scale;
    p.gscale = (float)(2.0 * scale / (double)N);
    p.fine = fine;
    p.flush = fine ? (int32_t)std::min<int64_t>(std::max<int64_t>(N >> 18, S + 1), 64) : kLnFlush;
    p.step = step;
    const bool parts = ln_parts(E, walk);
    const int64_t cap = std::min<int64_t>(kLossBlocks / (parts ? 2 : 1), (int64_t)num_cus() * ln_blocks(n % 256 == 0 ? kLnBoth : mode, E));
    const int blocks = (int)std::max<int64_t>(1, std::min<int64_t>(cap, (rows * p.tpr + kBlock / 64 - 1) / (kBlock / 64)));
    const int grid = mode == kLnFwd && parts ? 2 * blocks : blocks;
    const hipError_t e = ln_table().fn[NI - 1][L - 1][walk][mode](p, hs, grid);
    if (e == hipSuccess) {
        *nblk = grid;
        *nloss = parts ? 2 * blocks : blocks;
    }
    return e;
}

dpd_status check_transmit_forward(const dpd_plan *P, const dpd_plan *A, const dpd_plan *B, const void *x,
                                  const void *z, const void *grad_y, int64_t rows, int64_t n, int64_t ld,
                                  float scale)
{
    if (P == nullptr || A == nullptr || B == nullptr) return DPD_EINVAL;
    if (A->map.L != 1) return DPD_EINVAL;
    if (rows < 0 || n < 0 || (rows > 1 && ld < n)) return DPD_EINVAL;
    if (!std::isfinite(scale)) return DPD_EINVAL;
    if (A->map.NI != 1 || B->map.NI != kLnNIB || B->map.L != kLnLB || P->map.NI > kLnMaxNI ||
        P->map.L > kLnMaxL)
        return DPD_EUNSUPPORTED;
    if (rows * n > 0) {
        if (x == nullptr || z == nullptr || grad_y == nullptr) return DPD_EINVAL;
        for (const void *q : {x, z, grad_y})
            if ((uintptr_t)q % 8 != 0) return DPD_EINVAL;
        const size_t span = (size_t)(((rows - 1) * (rows > 1 ? ld : n) + n) * (int64_t)sizeof(float2));
        const auto lap = [&](const void *a, const void *b) {
            const uintptr_t u = (uintptr_t)a, v = (uintptr_t)b;
            return u < v + span && v < u + span;
        };
        if (lap(z, x) || lap(grad_y, x) || lap(z, grad_y)) return DPD_EINVAL;
    }
    return DPD_OK;
}


__global__ void step_advance(int32_t *step) { *step += 1; }

static bool ln_stages_ok(const dpd_plan *P, const dpd_plan *A, const dpd_plan *B)
{
    return A->map.NI == 1 && B->map.NI == kLnNIB && B->map.L == kLnLB && P->map.NI <= kLnMaxNI && P->map.L <= kLnMaxL;
}

// The shapes that dpd_learn_step takes and that dpd_transmit_backward takes
// without a dE/dz buffer (the kernels take any).
static bool one_call_shapes(const void *x, const void *z, const void *grad_y, const void *grad_z, int64_t n, int64_t rs)
{
    return (uintptr_t)x % 16 == 0 && (uintptr_t)z % 16 == 0 && (uintptr_t)grad_y % 16 == 0 &&
           (uintptr_t)grad_z % 16 == 0 && rs % 2 == 0 && n % 256 == 0;
}

// Learning-step finalisation in one launch: blocks 0 .. L NI sum the
// coefficient-gradient partials of their table entry in FP64 (as dpd_backward
// does), write the gradients (grad_coeffs may be NULL) and apply Adam to the
// coefficients they belong to (as dpd_adam_step does: each coefficient has
// exactly one entry); block L NI + 1 sums the loss partials.
__global__ void __launch_bounds__(kBlock) learn_finalize(const float *__restrict__ dc, int nblk, CoefMap map,
                                                         const float *__restrict__ lp, int nloss, double inv_n,
                                                         float *__restrict__ loss, float2 *__restrict__ gcoef,
                                                         float *__restrict__ params, float *__restrict__ m,
                                                         float *__restrict__ v, float lr, float b1, float b2,
                                                         float eps, float bc1, float bc2,
                                                         const int32_t *__restrict__ step)
{
    __shared__ double red[kBlock / 64][4];
    if (step != nullptr) {
        // Adam's bias corrections from the device-side step count
        const double t = (double)*step;
        bc1 = (float)(1.0 - pow((double)b1, t));
        bc2 = (float)(1.0 - pow((double)b2, t));
    }
    __shared__ double lred[kBlock / 64];
    const int q = blockIdx.x;
    if (q == map.L * map.NI + 1) {
        const double u = loss_block_total(lp, nloss, lred);
        if (threadIdx.x == 0 && loss != nullptr) *loss = (float)(u * inv_n);
        return;
    }
    double u[4];
    dcoef_block_sums(dc, nblk, map, q, red, u);
    if (threadIdx.x != 0) return;
    int idx[2];
    float2 g[2];
    const int c = dcoef_block_grads(map, q, u, idx, g);
    for (int i = 0; i < c; ++i) {
        if (gcoef != nullptr) gcoef[idx[i]] = g[i];
        const int r = 2 * idx[i];
        adam_one(params[r], g[i].x, m[r], v[r], lr, b1, b2, eps, bc1, bc2);
        adam_one(params[r + 1], g[i].y, m[r + 1], v[r + 1], lr, b1, b2, eps, bc1, bc2);
    }
}

// Workspace of dpd_learn_step: the loss partials, then (256-byte aligned) the
// coefficient-gradient partials.
static size_t learn_loss_bytes() { return ((size_t)kLossBlocks * sizeof(float) + 255) & ~(size_t)255; }

}  // namespace dpd

using namespace dpd;

DPD_EXPORT dpd_status dpd_transmit_loss_grad(dpd_plan *P, const dpd_plan *A, const dpd_plan *B, void *stream,
                                             const void *coeffs_dev, const void *x, void *z, int64_t rows, int64_t n,
                                             int64_t ld, float scale, float *loss_dev, void *grad_y, void *ws,
                                             size_t ws_bytes)
{
    const dpd_status st = check_transmit_forward(P, A, B, x, z, grad_y, rows, n, ld, scale);
    if (st != DPD_OK) return st;
    if (ws == nullptr || ws_bytes < kLossBlocks * sizeof(float) || (uintptr_t)ws % 4 != 0) return DPD_EINVAL;
    if (coeffs_dev != nullptr && (uintptr_t)coeffs_dev % 8 != 0) return DPD_EINVAL;
    const int64_t N = rows * n;
    const hipStream_t hs = (hipStream_t)stream;
    int nblk = 0, nloss = 0;
    hipError_t e = hipSuccess;
    if (N > 0)
        e = ln_run(kLnFwd, P, A, B, hs, coeffs_dev, x, z, grad_y, nullptr, rows, n, ld, scale, (float *)ws, nullptr,
                   nullptr, false, &nblk, &nloss);
    if (e != hipSuccess) return hip_fail(e);
    if (loss_dev != nullptr) {
        e = launch_loss_finalize((const float *)ws, nloss, N > 0 ? 1.0 / (double)N : 0.0, loss_dev, hs);
        if (e != hipSuccess) return hip_fail(e);
    }
    return DPD_OK;
}

DPD_EXPORT dpd_status dpd_transmit_backward(const dpd_plan *P, const dpd_plan *A, const dpd_plan *B, void *stream,
                                            const void *x, const void *z, const void *grad_y, void *grad_z,
                                            void *grad_coeffs, int64_t rows, int64_t n, int64_t ld, void *ws,
                                            size_t ws_bytes)
{
    if (P == nullptr || A == nullptr || B == nullptr || grad_coeffs == nullptr) return DPD_EINVAL;
    if (A->map.L != 1) return DPD_EINVAL;
    if (rows < 0 || n < 0 || (rows > 1 && ld < n)) return DPD_EINVAL;
    if (ws == nullptr || ws_bytes < bwd_ws_bytes(P->map) || (uintptr_t)ws % 4 != 0) return DPD_EINVAL;
    if ((uintptr_t)grad_coeffs % 8 != 0) return DPD_EINVAL;
    const int64_t N = rows * n;
    const int64_t rs = rows > 1 ? ld : n;
    if (N > 0) {
        if (x == nullptr || z == nullptr || grad_y == nullptr) return DPD_EINVAL;
        for (const void *q : {x, z, grad_y, (const void *)grad_z})
            if ((uintptr_t)q % 8 != 0) return DPD_EINVAL;
        if (grad_z != nullptr) {
            const size_t span = (size_t)(((rows - 1) * rs + n) * (int64_t)sizeof(float2));
            const auto lap = [&](const void *a, const void *b) {
                const uintptr_t u = (uintptr_t)a, v = (uintptr_t)b;
                return u < v + span && v < u + span;
            };
            if (lap(grad_z, x) || lap(grad_z, z) || lap(grad_z, grad_y)) return DPD_EINVAL;
        }
    }
    const hipStream_t hs = (hipStream_t)stream;
    // without a dE/dz buffer: only the shapes that never needed one
    if (N > 0 && grad_z == nullptr && !(ln_stages_ok(P, A, B) && one_call_shapes(x, z, grad_y, grad_z, n, rs)))
        return DPD_EUNSUPPORTED;
    const bool fine = (uintptr_t)x % 16 != 0 || (uintptr_t)grad_z % 16 != 0 || (rows > 1 && ld % 2 != 0);
    if (!ln_stages_ok(P, A, B) || (N > 0 && fine && N < kBwdShort)) {
        // other stages, and short inputs whose gradient bwd_dc_short_kernel sums: the
        // two passes, dE/dz through the caller's grad_z
        dpd_status st = dpd_cascade_backward(A, B, stream, z, grad_y, grad_z, rows, n, ld);
        if (st != DPD_OK) return st;
        return dpd_backward(const_cast<dpd_plan *>(P), stream, nullptr, x, grad_z, nullptr, grad_coeffs, rows, n,
                            ld, ws, ws_bytes);
    }
    int nblk = 0, nloss = 0;
    hipError_t e = hipSuccess;
    if (N > 0)
        e = ln_run(kLnBwd, P, A, B, hs, nullptr, x, z, grad_y, grad_z, rows, n, ld, 0.f, nullptr, (float *)ws, nullptr,
                   fine, &nblk, &nloss);
    if (e != hipSuccess) return hip_fail(e);
    e = launch_bwd_finalize((const float *)ws, nblk, P->map, (float2 *)grad_coeffs, hs);
    return e == hipSuccess ? DPD_OK : hip_fail(e);
}

DPD_EXPORT dpd_status dpd_learn_step_ws_size(const dpd_plan *P, size_t *bytes)
{
    if (P == nullptr || bytes == nullptr) return DPD_EINVAL;
    *bytes = learn_loss_bytes() + bwd_ws_bytes(P->map);
    return DPD_OK;
}

// The learning step with the Adam step count from the host (step >= 1) or,
// with step_dev, from a device counter the call advances.
static dpd_status learn_step(dpd_plan *P, const dpd_plan *A, const dpd_plan *B, void *stream, void *coeffs_dev,
                             float *adam_m, float *adam_v, int32_t step, int32_t *step_dev, float lr, float beta1,
                             float beta2, float eps, const void *x, void *z, void *grad_y, int64_t rows, int64_t n,
                             int64_t ld, float scale, float *loss_dev, void *grad_coeffs, void *ws, size_t ws_bytes)
{
    dpd_status st = check_transmit_forward(P, A, B, x, z, grad_y, rows, n, ld, scale);
    if (st != DPD_OK) return st;
    if (coeffs_dev == nullptr || adam_m == nullptr || adam_v == nullptr) return DPD_EINVAL;
    if (step_dev == nullptr ? step < 1 : (uintptr_t)step_dev % 4 != 0) return DPD_EINVAL;
    if ((uintptr_t)coeffs_dev % 8 != 0 || (uintptr_t)adam_m % 4 != 0 || (uintptr_t)adam_v % 4 != 0 ||
        (uintptr_t)grad_coeffs % 8 != 0)
        return DPD_EINVAL;
    if (!std::isfinite(lr) || !std::isfinite(beta1) || !std::isfinite(beta2) || !std::isfinite(eps))
        return DPD_EINVAL;
    const size_t need = learn_loss_bytes() + bwd_ws_bytes(P->map);
    if (ws == nullptr || ws_bytes < need || (uintptr_t)ws % 4 != 0) return DPD_EINVAL;
    // the K coefficients, their Adam moments and the gradient output must not overlap
    const size_t kb = (size_t)P->K * sizeof(float2);
    const auto lap = [kb](const void *a, const void *b) {
        const uintptr_t u = (uintptr_t)a, v = (uintptr_t)b;
        return a != nullptr && b != nullptr && u < v + kb && v < u + kb;
    };
    if (lap(coeffs_dev, adam_m) || lap(coeffs_dev, adam_v) || lap(adam_m, adam_v) || lap(grad_coeffs, coeffs_dev) ||
        lap(grad_coeffs, adam_m) || lap(grad_coeffs, adam_v))
        return DPD_EINVAL;
    if (step_dev != nullptr) {
        // nor the step counter any of them
        const auto in = [kb](const void *base, const void *q) {
            const uintptr_t u = (uintptr_t)base, v = (uintptr_t)q;
            return base != nullptr && v + sizeof(int32_t) > u && v < u + kb;
        };
        if (in(coeffs_dev, step_dev) || in(adam_m, step_dev) || in(adam_v, step_dev) || in(grad_coeffs, step_dev))
            return DPD_EINVAL;
    }
    const int64_t rs = rows > 1 ? ld : n;
    if (!ln_stages_ok(P, A, B) || !one_call_shapes(x, z, grad_y, nullptr, n, rs)) return DPD_EUNSUPPORTED;
    const hipStream_t hs = (hipStream_t)stream;
    const int64_t N = rows * n;
    float *lp = (float *)ws;
    float *dc = (float *)((char *)ws + learn_loss_bytes());
    int nblk = 0, nloss = 0;
    hipError_t e;
    if (N > 0) {
        e = ln_run(kLnBoth, P, A, B, hs, coeffs_dev, x, z, grad_y, nullptr, rows, n, ld, scale, lp, dc, step_dev,
                   false, &nblk, &nloss);
    } else {
        if (step_dev != nullptr) hipLaunchKernelGGL(step_advance, dim3(1), dim3(1), 0, hs, step_dev);
        e = hipGetLastError();
    }
    if (e != hipSuccess) return hip_fail(e);
    const float bc1 = step_dev ? 0.f : (float)(1.0 - std::pow((double)beta1, step));
    const float bc2 = step_dev ? 0.f : (float)(1.0 - std::pow((double)beta2, step));
    hipLaunchKernelGGL(learn_finalize, dim3((uint32_t)(P->map.L * P->map.NI + 2)), dim3(kBlock), 0, hs, dc, nblk,
                       P->map, lp, nloss, N > 0 ? 1.0 / (double)N : 0.0, loss_dev, (float2 *)grad_coeffs,
                       (float *)coeffs_dev, adam_m, adam_v, lr, beta1, beta2, eps, bc1, bc2,
                       (const int32_t *)step_dev);
    e = hipGetLastError();
    return e == hipSuccess ? DPD_OK : hip_fail(e);
}

DPD_EXPORT dpd_status dpd_learn_step(dpd_plan *P, const dpd_plan *A, const dpd_plan *B, void *stream,
                                     void *coeffs_dev, float *adam_m, float *adam_v, int32_t step, float lr,
                                     float beta1, float beta2, float eps, const void *x, void *z, void *grad_y,
                                     int64_t rows, int64_t n, int64_t ld, float scale, float *loss_dev,
                                     void *grad_coeffs, void *ws, size_t ws_bytes)
{
    return learn_step(P, A, B, stream, coeffs_dev, adam_m, adam_v, step, nullptr, lr, beta1, beta2, eps, x, z,
                      grad_y, rows, n, ld, scale, loss_dev, grad_coeffs, ws, ws_bytes);
}

DPD_EXPORT dpd_status dpd_learn_step_dev(dpd_plan *P, const dpd_plan *A, const dpd_plan *B, void *stream,
                                         void *coeffs_dev, float *adam_m, float *adam_v, int32_t *step_dev, float lr,
                                         float beta1, float beta2, float eps, const void *x, void *z, void *grad_y,
                                         int64_t rows, int64_t n, int64_t ld, float scale, float *loss_dev,
                                         void *grad_coeffs, void *ws, size_t ws_bytes)
{
    if (step_dev == nullptr) return DPD_EINVAL;
    return learn_step(P, A, B, stream, coeffs_dev, adam_m, adam_v, 0, step_dev, lr, beta1, beta2, eps, x, z, grad_y,
                      rows, n, ld, scale, loss_dev, grad_coeffs, ws, ws_bytes);
}
