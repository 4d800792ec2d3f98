// kernels_mr_unit.hip -- one compilation unit of the compile-time mixed-radix
// kernels (kernels_mr.h): the lengths kMrLen[i] with i mod PF_MR_UNITS ==
// PF_MR_UNIT, in the precision PF_MR_T.  build.py compiles this file once per
// unit and precision, in parallel.
#include <utility>

#include "kernels_mr.h"

#ifndef PF_MR_UNIT
#define PF_MR_UNIT 0
#endif
#ifndef PF_MR_T
#define PF_MR_T float
#endif
#ifndef PF_MR_NAME
#define PF_MR_NAME mr_pick_float_0
#endif

namespace pf {

namespace {

constexpr int kMine = (kMrCount - PF_MR_UNIT + PF_MR_UNITS - 1) / PF_MR_UNITS;  // lengths of this unit

template <int... K>
const void *pick(int index, int what, std::integer_sequence<int, K...>) {
    const void *r = nullptr;
    ((index == K * PF_MR_UNITS + PF_MR_UNIT
          ? (void)(r = mr_kernel_at<PF_MR_T, K * PF_MR_UNITS + PF_MR_UNIT>(what)) : (void)0), ...);
    return r;
}

}  // namespace

const void *PF_MR_NAME(int index, int what) { return pick(index, what, std::make_integer_sequence<int, kMine>()); }

}  // namespace pf
