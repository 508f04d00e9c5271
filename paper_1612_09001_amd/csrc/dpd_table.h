// One entry of a plan's precombined table, formed in a kernel from the raw
// coefficients: kernels that take device coefficients build the table in LDS
// themselves instead of waiting for a launch that writes it to memory.
#pragma once

#include "dpd_internal.h"

namespace dpd {

// Entry e (4 L NI matrix floats, then c): read from the table M, or with raw
// coefficients (K complex, section 2.2 layout) formed with the arithmetic of
// the table kernel (hr+gr, gi-hi, hi+gi, hr-gr), so both give the same bits.
__device__ __forceinline__ float table_entry(const float *M, const float2 *raw, const CoefMap &map, int e)
{
    if (raw == nullptr) return M[e];
    const int L = map.L, NI = map.NI;
    if (e >= 4 * L * NI) {
        const float2 c = raw[(map.n_main + map.n_conj) * L];
        return e == 4 * L * NI ? c.x : c.y;
    }
    const int k = e / (4 * NI), r = e - k * 4 * NI, j = r >> 2, q = r & 3;
    float2 h = make_float2(0.f, 0.f), g = make_float2(0.f, 0.f);
    if (map.main_idx[j] >= 0) h = raw[map.main_idx[j] * L + k];
    if (map.conj_idx[j] >= 0) g = raw[(map.n_main + map.conj_idx[j]) * L + k];
    return q == 0 ? h.x + g.x : q == 1 ? g.y - h.y : q == 2 ? h.y + g.y : h.x - g.x;
}

}  // namespace dpd
