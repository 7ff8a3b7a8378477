// Launchers of the fine-level kernels that evaluate the operator per cell.
#include "kernels_cell.hpp"

namespace dgmg {

// Cells per workgroup: 64 fill a wave's lanes; on a level with fewer than one
// such workgroup per CU, smaller groups spread the cells over more CUs (a
// lane's scattered loads of its cell then share an address unit with fewer
// others).  Measured per step, 16 / 32 / 64 cells: 1,728 3D Q2 cells 5.1 / 5.3
// / 5.8 us, 8,000 6.8 / 5.7 / 6.0 us, 64,000 34 / 22 / 15 us.  3D Q3 cells
// take four lanes each.
static int cells_per_group(int b, int n) {
    if (b == 64 || n <= 16 * 256) return 16;
    return n <= 32 * 256 ? 32 : 64;
}
unsigned cell_groups(int b, int n) {
    const int nc = cells_per_group(b, n);
    return (unsigned)((n + nc - 1) / nc);
}

// block size BV and cells per workgroup NC as constants
#define DISPATCH_CELL(bval, nval, ...)                                                        \
    if ((bval) == 64) { constexpr int BV = 64, NC = 16; __VA_ARGS__; }                        \
    else if (cells_per_group(bval, nval) == 16) { constexpr int NC = 16; DISPATCH_CELL_B(bval, __VA_ARGS__) } \
    else if (cells_per_group(bval, nval) == 32) { constexpr int NC = 32; DISPATCH_CELL_B(bval, __VA_ARGS__) } \
    else { constexpr int NC = 64; DISPATCH_CELL_B(bval, __VA_ARGS__) }
#define DISPATCH_CELL_B(bval, ...)                                                            \
    switch (bval) {                                                                           \
        case 4: { constexpr int BV = 4; __VA_ARGS__; } break;                                 \
        case 8: { constexpr int BV = 8; __VA_ARGS__; } break;                                 \
        case 9: { constexpr int BV = 9; __VA_ARGS__; } break;                                 \
        case 16: { constexpr int BV = 16; __VA_ARGS__; } break;                               \
        case 25: { constexpr int BV = 25; __VA_ARGS__; } break;                               \
        case 27: { constexpr int BV = 27; __VA_ARGS__; } break;                               \
        default: fail(DGMG_EUNSUPPORTED, "unsupported block size");                           \
    }

template <typename T>
void cell_apply(const LaunchEvents& ev, int b, const CellArgs<T>& L, const T* va, T* y, const T* w, double* partial,
                hipStream_t st) {
    const unsigned g = cell_groups(b, L.n);
    DISPATCH_CELL(b, L.n, klaunch(ev, k_apply_cell<T, BV, NC>, g, cell_threads<BV>(), st, L, va, y, w, partial));
}

template <typename T>
void cell_residual(const LaunchEvents& ev, int b, const CellArgs<T>& L, const T* va, const T* vb, const T* rhs, T* r,
                   T* d, T c1, T* xout, double* partial, const T* P, T* rp, const int32_t* ptype, const T* bj,
                   hipStream_t st) {
    const unsigned g = cell_groups(b, L.n);
    auto go = [&](auto vbc, auto bjc) {
        constexpr bool VB = decltype(vbc)::value, BJ = decltype(bjc)::value;
        DISPATCH_CELL(b, L.n, klaunch(ev, k_residual_cell<T, BV, NC, VB, BJ>, g, cell_threads<BV>(), st, L, va, vb, rhs,
                                      r, d, c1, xout, partial, P, rp, ptype, bj));
    };
    using Y = std::true_type;
    using Z = std::false_type;
    if (vb && bj) go(Y{}, Y{});
    else if (vb) go(Y{}, Z{});
    else if (bj) go(Z{}, Y{});
    else go(Z{}, Z{});
}

template <typename T>
void cell_step(const LaunchEvents& ev, int b, const CellArgs<T>& L, const T* d, T* x, T* r, T* dn, T cd, T cr,
               int assign, int last, const T* bj, hipStream_t st) {
    const unsigned g = cell_groups(b, L.n);
    auto go = [&](auto bjc) {
        constexpr bool BJ = decltype(bjc)::value;
        DISPATCH_CELL(b, L.n, klaunch(ev, k_cheb_step_cell<T, BV, NC, BJ>, g, cell_threads<BV>(), st, L, d, x, r, dn, cd,
                                      cr, assign, last, bj));
    };
    if (bj) go(std::true_type{});
    else go(std::false_type{});
}

#define INSTANTIATE(T)                                                                                              \
    template void cell_apply<T>(const LaunchEvents&, int, const CellArgs<T>&, const T*, T*, const T*, double*,      \
                                hipStream_t);                                                                       \
    template void cell_residual<T>(const LaunchEvents&, int, const CellArgs<T>&, const T*, const T*, const T*, T*,  \
                                   T*, T, T*, double*, const T*, T*, const int32_t*, const T*, hipStream_t);        \
    template void cell_step<T>(const LaunchEvents&, int, const CellArgs<T>&, const T*, T*, T*, T*, T, T, int, int,  \
                               const T*, hipStream_t);
INSTANTIATE(float)
INSTANTIATE(double)

}  // namespace dgmg
