// Instantiates the learning-step kernels for NI = DPD_NI (set on the compiler
// command line) and every L in 1..kLnMaxL.
#include "dpd_learn_kernels.h"

#ifndef DPD_NI
#error "compile with -DDPD_NI=<1..5>"
#endif

#define DPD_CAT2(a, b) a##b
#define DPD_CAT(a, b) DPD_CAT2(a, b)

namespace dpd {

void DPD_CAT(register_learn_ni, DPD_NI)(LnTable &t)
{
    register_learn_one<DPD_NI, 1>(t);
    register_learn_one<DPD_NI, 2>(t);
    register_learn_one<DPD_NI, 3>(t);
    register_learn_one<DPD_NI, 4>(t);
    register_learn_one<DPD_NI, 5>(t);
    register_learn_one<DPD_NI, 6>(t);
    register_learn_one<DPD_NI, 7>(t);
    register_learn_one<DPD_NI, 8>(t);
}

}  // namespace dpd
