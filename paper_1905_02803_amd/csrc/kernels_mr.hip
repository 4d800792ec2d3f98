// kernels_mr.hip -- host side of the compile-time mixed-radix passes
// (kernels_mr.h): which lengths have them, their launch shapes, launches.
#include <cstring>

#include "kernels_mr.h"

namespace pf {

// the compilation units (kernels_mr_unit.hip), PF_MR_UNITS per precision
#define PF_MR_EACH_UNIT(X, T) X(T, 0) X(T, 1) X(T, 2) X(T, 3) X(T, 4) X(T, 5) X(T, 6) X(T, 7)
static_assert(PF_MR_UNITS == 8, "PF_MR_EACH_UNIT names every unit");
#define PF_MR_DECLARE(T, U) const void *mr_pick_##T##_##U(int index, int what);
PF_MR_EACH_UNIT(PF_MR_DECLARE, float)
PF_MR_EACH_UNIT(PF_MR_DECLARE, double)
#undef PF_MR_DECLARE

namespace {

struct MrSizes {  // launch shape of one length in one precision
    int c2c_threads, x_threads, x_pairs;
    size_t c2c_lds, x_lds;
};

template <typename T, int I>
constexpr MrSizes sizes_at() {  // the kernels' own tile constants, so that host and device sizes agree
    using S = MrShape<T, kMrLen[I].n1, kMrLen[I].n2>;
    return MrSizes{S::CTHREADS, S::XTHREADS, S::XP, (size_t)S::CLDS, (size_t)S::XLDS};
}
template <typename T, int... I>
const MrSizes &sizes_of(int index, std::integer_sequence<int, I...>) {
    static constexpr MrSizes all[] = {sizes_at<T, I>()...};
    return all[index];
}
const MrSizes &sizes(int index, int prec) {
    constexpr auto seq = std::make_integer_sequence<int, kMrCount>();
    return prec ? sizes_of<double>(index, seq) : sizes_of<float>(index, seq);
}

const void *mr_kernel(int n, int prec, int what) {
    const int i = mr_index(n);
    if (i < 0) return nullptr;
#define PF_MR_REF(T, U) mr_pick_##T##_##U,
    static const mr_pick_fn f32[] = {PF_MR_EACH_UNIT(PF_MR_REF, float)};
    static const mr_pick_fn f64[] = {PF_MR_EACH_UNIT(PF_MR_REF, double)};
#undef PF_MR_REF
    return (prec ? f64 : f32)[i % PF_MR_UNITS](i, what);
}

int what_of(int kind) {
    return kind == PASS_C2C_MR ? MR_C2C : kind == PASS_R2C_MR ? MR_R2C : kind == PASS_C2R_MR ? MR_C2R : -1;
}

hipError_t mr_go(int kind, int n, int prec, unsigned blocks, unsigned threads, size_t lds, MrArgs &m, hipStream_t s) {
    const int what = what_of(kind);
    const void *k = what < 0 ? nullptr : mr_kernel(n, prec, what);
    if (!k) return hipErrorInvalidValue;
    if (blocks == 0) return hipSuccess;
    void *args[] = {&m};
    return hipLaunchKernel(k, dim3(blocks), dim3(threads), args, lds, s);
}

}  // namespace

bool mr_supported(int n, int prec) { return (prec == 0 || prec == 1) && mr_index(n) >= 0; }

int mr_threads_of(int n, int prec, int xpass) {
    const int i = mr_index(n);
    return i < 0 ? 0 : xpass ? sizes(i, prec).x_threads : sizes(i, prec).c2c_threads;
}

int mr_x_pairs(int n, int prec) {
    const int i = mr_index(n);
    return i < 0 ? 0 : sizes(i, prec).x_pairs;
}

size_t mr_lds_bytes(int n, int prec, int xpass) {
    const int i = mr_index(n);
    return i < 0 ? 0 : xpass ? sizes(i, prec).x_lds : sizes(i, prec).c2c_lds;
}

hipError_t mr_prepare(int n, int prec, int xpass) {
    const size_t lds = mr_lds_bytes(n, prec, xpass);
    if (lds <= 64 * 1024) return hipSuccess;  // the default limit
    hipError_t e = hipSuccess;
    for (int what : {MR_C2C, MR_R2C, MR_C2R}) {
        if ((what != MR_C2C) != (xpass != 0) || e != hipSuccess) continue;
        const void *k = mr_kernel(n, prec, what);
        e = k ? hipFuncSetAttribute(k, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds) : hipErrorInvalidValue;
    }
    return e;
}

hipError_t mr_launch(const PassDesc &d, hipStream_t s) {
    MrArgs m;
    std::memset(&m, 0, sizeof(m));
    m.one = d.a;
    m.dir = d.dir;
    return mr_go(d.kind, d.a.fft.n, d.prec, d.blocks, d.threads, d.lds, m, s);
}

hipError_t mr_launch_batch(const BatchLaunch &L, hipStream_t s) {
    MrArgs m;
    std::memset(&m, 0, sizeof(m));
    m.b = L.b;
    m.dir = L.dir;
    if (m.b.count < 1) return hipErrorInvalidValue;
    return mr_go(L.kind, L.n, L.prec, L.blocks, L.threads, L.lds, m, s);
}

}  // namespace pf
