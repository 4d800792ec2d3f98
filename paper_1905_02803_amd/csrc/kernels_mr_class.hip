// kernels_mr_class.hip -- the batched kernels of one class of lengths
// (kernels_mr.h, kMrClass) in one precision.  build.py compiles this file once
// per class and precision, in parallel.
#include "kernels_mr.h"

#ifndef PF_MR_CLASS
#define PF_MR_CLASS 0
#endif
#ifndef PF_MR_T
#define PF_MR_T float
#endif
#ifndef PF_MR_NAME
#define PF_MR_NAME mr_class_float_0
#endif

namespace pf {

const void *PF_MR_NAME(int what) {
    switch (what) {
        case MR_C2C: return reinterpret_cast<const void *>(&k_mr_c2c_class<PF_MR_CLASS, PF_MR_T>);
        case MR_R2C: return reinterpret_cast<const void *>(&k_mr_x_class<PF_MR_CLASS, 1, PF_MR_T>);
        case MR_C2R: return reinterpret_cast<const void *>(&k_mr_x_class<PF_MR_CLASS, 0, PF_MR_T>);
    }
    return nullptr;
}

}  // namespace pf
