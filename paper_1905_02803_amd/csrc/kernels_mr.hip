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

// the batched kernels of the classes of lengths (kernels_mr_class.hip)
static_assert(kMrClasses == 6, "every class is named below");
#define PF_MR_EACH_CLASS(X, T) X(T, 0) X(T, 1) X(T, 2) X(T, 3) X(T, 4) X(T, 5)
#define PF_MR_DECLARE(T, U) const void *mr_class_##T##_##U(int what);
PF_MR_EACH_CLASS(PF_MR_DECLARE, float)
PF_MR_EACH_CLASS(PF_MR_DECLARE, double)
#undef PF_MR_DECLARE

namespace {

template <typename T, int... C>
unsigned class_threads(int cls, bool x, std::integer_sequence<int, C...>) {
    static constexpr int c2c[] = {mr_class_c2c_threads<T>(C)...}, xs[] = {mr_class_x_threads<T, C>()...};
    return (unsigned)(x ? xs[cls] : c2c[cls]);
}

const void *class_kernel(int cls, int prec, int what) {
#define PF_MR_REF(T, U) mr_class_##T##_##U,
    typedef const void *(*fn)(int);
    static const fn f32[] = {PF_MR_EACH_CLASS(PF_MR_REF, float)};
    static const fn f64[] = {PF_MR_EACH_CLASS(PF_MR_REF, double)};
#undef PF_MR_REF
    return (prec ? f64 : f32)[cls](what);
}

struct MrSizes {  // launch shapes of one length in one precision: C2C, X, spectral step
    int threads[3], x_pairs, span;
    size_t lds[3];
};

template <typename T, int I>
constexpr MrSizes sizes_at() {  // the kernels' own tile constants, so that host and device sizes agree
    using S = MrShape<T, MrPlan<T, I>>;
    using Z = MrShape<T, MrTwoStep<T, kMrLen[I].n1, kMrLen[I].n2>>;
    return MrSizes{{S::CTHREADS, S::XTHREADS, Z::CTHREADS}, S::XP, S::SPAN,
                   {(size_t)S::CLDS, (size_t)S::XLDS, (size_t)Z::CLDS}};
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

hipError_t mr_go(const void *k, dim3 grid, unsigned threads, size_t lds, MrArgs &m, hipStream_t s) {
    if (!k) return hipErrorInvalidValue;
    if (grid.x == 0 || grid.y == 0) return hipSuccess;
    void *args[] = {&m};
    return hipLaunchKernel(k, grid, dim3(threads), args, lds, s);
}

// One side of a C2C pass: rows (columns contiguous; the workspace's, one block of
// columns apart, or the user's) or lines (points contiguous).
void pack_side(const Side &d, int cols, unsigned *sa, unsigned *sb, unsigned *ss, bool *lines) {
    *lines = d.sp == 1 && d.sc != 1;
    *sa = (unsigned)d.sa;
    *sb = (unsigned)(d.cpb == 1 ? d.sblk : cols * d.sc);
    *ss = (unsigned)(*lines ? d.sc : d.sp);
}

static_assert(sizeof(MrArgs) <= sizeof(PassArgs), "packed records fit the slots of the table");

MrArgs pack(int kind, int dir, int prec, const PassArgs &a) {
    MrArgs m;
    std::memset(&m, 0, sizeof(m));
    m.in = a.in;
    m.out = a.out;
    m.tw = a.tw;
    if (kind == PASS_C2C_MR) {
        bool il, ol;
        const int cols = prec ? 8 : 16;
        pack_side(a.in_s, cols, &m.c.isa, &m.c.isb, &m.c.iss, &il);
        pack_side(a.out_s, cols, &m.c.osa, &m.c.osb, &m.c.oss, &ol);
        m.C = a.C;
        m.CB = (int)a.CB;
        m.flags = (dir > 0 ? MR_BACKWARD : 0u) | (il ? MR_IN_LINES : 0u) | (ol ? MR_OUT_LINES : 0u);
    } else {
        m.x.zrows = (unsigned)a.zrows, m.x.kbrows = (unsigned)a.kbrows, m.x.y0 = (unsigned)a.y0;
        m.x.ny = (unsigned)a.ny, m.x.lines = (unsigned)a.lines;
    }
    const int i = mr_index(a.fft.n), cls = i < 0 ? -1 : mr_class(i);
    if (cls >= 0) m.count = i - kMrClass[cls].first;  // read from batch entries alone
    return m;
}

}  // namespace

bool mr_supported(int n, int prec) { return (prec == 0 || prec == 1) && mr_index(n) >= 0; }

int mr_threads_of(int n, int prec, int form) {
    const int i = mr_index(n);
    return i < 0 ? 0 : sizes(i, prec).threads[form];
}

int mr_span(int n, int prec) {
    const int i = mr_index(n);
    return i < 0 ? 0 : sizes(i, prec).span;
}

int mr_x_pairs(int n, int prec) {
    const int i = mr_index(n);
    return i < 0 ? 0 : sizes(i, prec).x_pairs;
}

size_t mr_lds_bytes(int n, int prec, int form) {
    const int i = mr_index(n);
    return i < 0 ? 0 : sizes(i, prec).lds[form];
}

hipError_t mr_prepare(int n, int prec, int form) {
    const size_t lds = mr_lds_bytes(n, prec, form);
    if (lds <= 64 * 1024) return hipSuccess;  // the default limit
    for (int what : {MR_C2C, MR_R2C, MR_C2R, MR_SPEC}) {
        if (form != (what == MR_C2C ? MR_FORM_C2C : what == MR_SPEC ? MR_FORM_SPEC : MR_FORM_X)) continue;
        const void *k = mr_kernel(n, prec, what);
        if (!k) return hipErrorInvalidValue;
        const hipError_t e = hipFuncSetAttribute(k, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}

// A length above 324 whose transforms have this many workgroups in all fills the chip
// by itself and runs its own kernel (12 FP32 grids of 336 .. 480 points 9.14 ms a pair,
// 9.87 as classes); below, a launch per length costs more than the classes' shared
// shape (64 FP32 grids with one edge of 336 .. 1024, the others of 16 .. 32, 1.29
// ms, 0.53 as classes, 0.84 as one launch of the runtime-radix kernels; 256 or 512
// in place of 1024: 0.54, 0.53; 2048: the same).
constexpr long long kMrOwnLaunch = 1024;

int mr_batch_class(int n, long long blocks) {
    const int i = mr_index(n), cls = i < 0 ? -1 : mr_class(i);
    return cls >= kMrLongClass && blocks >= kMrOwnLaunch ? -1 : cls;
}

hipError_t mr_prepare_batch(const BatchLaunch &L) {
    const int what = what_of(L.kind);
    if (L.cls < 0 || what < 0 || L.lds <= 64 * 1024) return hipSuccess;
    return hipFuncSetAttribute(class_kernel(L.cls, L.prec, what), hipFuncAttributeMaxDynamicSharedMemorySize,
                               (int)L.lds);
}

size_t mr_entry_bytes() { return sizeof(MrArgs); }

void mr_entry(int kind, int dir, int prec, const PassArgs &a, void *dst) {
    const MrArgs m = pack(kind, dir, prec, a);
    std::memcpy(dst, &m, sizeof(m));
}

hipError_t mr_launch(const PassDesc &d, hipStream_t s) {
    MrArgs m = pack(d.kind, d.dir, d.prec, d.a);
    dim3 grid = d.kind == PASS_C2C_MR ? dim3((unsigned)d.a.CB, (unsigned)d.a.A) : dim3(d.blocks);
    if (d.a.xcd) {
        grid = dim3(grid.x * grid.y);
        m.flags |= MR_XCD;
        m.count = (int)grid.x;
    } else if (d.kind == PASS_C2C_MR && d.a.tile_order) {
        grid = dim3(grid.y, grid.x);
        m.flags |= MR_OUTER_FAST;
    }
    if (d.nt_out) m.flags |= MR_NT_STORES;
    const int what = what_of(d.kind);
    return mr_go(what < 0 ? nullptr : mr_kernel(d.a.fft.n, d.prec, what), grid, d.threads, d.lds, m, s);
}

hipError_t mr_spec_launch(const PassArgs &a, int prec, int adj, int nx, hipStream_t s) {
    const int n = a.fft.n;
    MrArgs m;
    std::memset(&m, 0, sizeof(m));
    m.in = a.in;
    m.out = a.out;
    m.tw = a.tw;
    m.s.sa = (unsigned)a.in_s.sa, m.s.sb = (unsigned)a.in_s.sblk, m.s.ss = (unsigned)a.in_s.sp;
    m.s.nx = (unsigned)nx, m.s.ny = (unsigned)a.A;
    m.flags = adj ? MR_BACKWARD : 0u;
    return mr_go(mr_kernel(n, prec, MR_SPEC), dim3((unsigned)a.CB, (unsigned)a.A), (unsigned)mr_threads_of(n, prec, MR_FORM_SPEC),
                 mr_lds_bytes(n, prec, MR_FORM_SPEC), m, s);
}

hipError_t mr_launch_batch(const BatchLaunch &L, hipStream_t s) {
    if (L.b.count < 1) return hipErrorInvalidValue;
    MrArgs m;
    std::memset(&m, 0, sizeof(m));
    m.in = L.b.user_in;
    m.out = L.b.user_out;
    m.b.table = reinterpret_cast<const MrArgs *>(L.b.args);
    m.b.first = L.b.first;
    m.count = L.b.count;
    m.flags = MR_BATCH | (L.b.in_user ? MR_IN_USER : 0u) | (L.b.out_user ? MR_OUT_USER : 0u);
    const int what = what_of(L.kind);
    if (what < 0) return hipErrorInvalidValue;
    if (L.cls < 0) return mr_go(mr_kernel(L.n, L.prec, what), dim3(L.blocks), L.threads, L.lds, m, s);
    constexpr auto seq = std::make_integer_sequence<int, kMrClasses>();
    const bool x = what != MR_C2C;
    const unsigned threads = L.prec ? class_threads<double>(L.cls, x, seq) : class_threads<float>(L.cls, x, seq);
    return mr_go(class_kernel(L.cls, L.prec, what), dim3(L.blocks), threads, L.lds, m, s);
}

}  // namespace pf
