// Launchers of the kernels that evaluate a level per cell; included by one
// translation unit per geometry.
#pragma once
#include "kernels_cell.hpp"

namespace dgmg {

// Cells per workgroup: 64 fill a wave's lanes; on a level of up to 16 cells per
// CU, groups of 16 spread them over more CUs (a lane's scattered loads of its
// cell then share an address unit with fewer others).  Measured per step, 16 / 64 cells: 1,728 3D Q2 boxes 5.1 / 5.8 us,
// 8,000 6.8 / 6.0 us, 64,000 34 / 15 us.  3D Q3 cells take four lanes each.
// bj: the kernel has the cell-block term, whose epilogue reads b values per row.
// b = 64: groups of 4 on small levels; 512 cells, 4 / 16 cells: FP64 8.7 / 14.5 us, FP32
// 6.3 / 8.7 us; 1,728 cells 15.2 / 15.3, 7.5 / 8.9; 4,096 cells 28.7 / 25.1, 17.1 / 14.9.
// Q4 boxes take a lane per row in groups of 8 (GEO_BOXR) up to these sizes; V-cycle of
// two levels by rows / by cells of 64, us: point Jacobi 2,304 cells 129 / 141 (FP32 106 / 119),
// 4,096 cells 134 / 145 (112 / 122), 6,400 cells 188 / 162 (147 / 135); cell-block
// 9,216 cells 304 / 337 (191 / 199), 12,544 cells 417 / 419, 16,384 cells 492 / 492 (300 / 300).
static int cells_per_group(int geo, int b, int n, bool bj) {
    if (geo == GEO_ROW) return 1;
    if (b == 64) return bj && n <= 8 * 256 ? 4 : 16;
    if (geo == GEO_BOX && b == 25) return n <= (bj ? 50 : 16) * 256 ? 8 : 64;
    return n <= 16 * 256 ? 16 : 64;
}

// block size BV, cells per workgroup NC and the kernels' geometry KG as constants
// (BJ: of the kernels with the cell-block term)
#define DISPATCH_CELL(bval, nc, ...)                                                          \
    if constexpr (GEO == GEO_ROW) {                                                           \
        if ((bval) == 64) { constexpr int BV = 64, NC = 1, KG = GEO; __VA_ARGS__; return; }             \
    } else if constexpr (GEO == GEO_BOX) {                                                    \
        if constexpr (BJ) {                                                                   \
            if ((bval) == 64 && (nc) == 4) { constexpr int BV = 64, NC = 4, KG = GEO; __VA_ARGS__; return; } \
        }                                                                                     \
        if ((bval) == 64) { constexpr int BV = 64, NC = 16, KG = GEO; __VA_ARGS__; return; }            \
        if ((bval) == 25 && (nc) == 8) {                                                      \
            constexpr int BV = 25, NC = 8, KG = GEO_BOXR;                                     \
            __VA_ARGS__;                                                                      \
            return;                                                                           \
        }                                                                                     \
        if ((bval) == 25) { constexpr int BV = 25, NC = 64, KG = GEO; __VA_ARGS__; return; }  \
    }                                                                                         \
    if constexpr (GEO != GEO_MAP && GEO != GEO_ROW) {                                         \
        if ((bval) == 4) { DISPATCH_NC(4, nc, __VA_ARGS__) return; }                          \
        if ((bval) == 8) { DISPATCH_NC(8, nc, __VA_ARGS__) return; }                          \
    }                                                                                         \
    if constexpr (GEO != GEO_HYB && GEO != GEO_ROW) {                                         \
        if ((bval) == 9) { DISPATCH_NC(9, nc, __VA_ARGS__) return; }                          \
    }                                                                                         \
    if constexpr (GEO != GEO_HYB && GEO != GEO_BLD && GEO != GEO_ROW) {                       \
        if ((bval) == 16) { DISPATCH_NC(16, nc, __VA_ARGS__) return; }                        \
        if constexpr (GEO != GEO_BOX) {                                                       \
            if ((bval) == 25) { DISPATCH_NC(25, nc, __VA_ARGS__) return; }                    \
        }                                                                                     \
        if ((bval) == 27) { DISPATCH_NC(27, nc, __VA_ARGS__) return; }                        \
    }                                                                                         \
    fail(DGMG_EUNSUPPORTED, "unsupported block size");
#define DISPATCH_NC(bval, nc, ...)                                                            \
    constexpr int BV = bval, KG = GEO;                                                        \
    if ((nc) == 16) { constexpr int NC = 16; __VA_ARGS__; }                                   \
    else { constexpr int NC = 64; __VA_ARGS__; }

template <typename T, int GEO>
void cell_apply(const LaunchEvents& ev, int b, const CellArgs<T>& L, const T* va, T* y, const T* w, double* partial,
                hipStream_t st) {
    constexpr bool BJ = false;
    const int nc = cells_per_group(GEO, b, L.n, BJ);
    const unsigned g = (unsigned)((L.n + nc - 1) / nc);
    DISPATCH_CELL(b, nc, klaunch(ev, k_apply_cell<T, BV, NC, KG>, g, cell_threads<BV, KG>(), st, L, va, y, w, partial));
}

template <typename T, int GEO>
void cell_residual(const LaunchEvents& ev, int b, const CellArgs<T>& L, const T* va, const T* vb, const T* rhs, T* r,
                   T* d, T c1, T* xout, double* partial, const T* P, T* rp, const int32_t* ptype, const T* bj,
                   hipStream_t st) {
    // as many partials as cell_groups says
    const int nc = cells_per_group(GEO, b, L.n, bj && !partial);
    const unsigned g = (unsigned)((L.n + nc - 1) / nc);
    auto go = [&](auto vbc, auto bjc) {
        constexpr bool VB = decltype(vbc)::value, BJ = decltype(bjc)::value;
        DISPATCH_CELL(b, nc, klaunch(ev, k_residual_cell<T, BV, NC, KG, VB, BJ>, g, cell_threads<BV, KG>(), st, L, va, vb, rhs,
                                      r, d, c1, xout, partial, P, rp, ptype, bj));
    };
    using Y = std::true_type;
    using Z = std::false_type;
    if (vb && bj) go(Y{}, Y{});
    else if (vb) go(Y{}, Z{});
    else if (bj) go(Z{}, Y{});
    else go(Z{}, Z{});
}

template <typename T, int GEO>
void cell_step(const LaunchEvents& ev, int b, const CellArgs<T>& L, const T* d, T* x, T* r, T* dn, T cd, T cr,
               int assign, int last, const T* bj, hipStream_t st) {
    const int nc = cells_per_group(GEO, b, L.n, bj != nullptr);
    const unsigned g = (unsigned)((L.n + nc - 1) / nc);
    auto go = [&](auto bjc) {
        constexpr bool BJ = decltype(bjc)::value;
        DISPATCH_CELL(b, nc, klaunch(ev, k_cheb_step_cell<T, BV, NC, KG, BJ>, g, cell_threads<BV, KG>(), st, L, d, x, r, dn, cd,
                                      cr, assign, last, bj));
    };
    if (bj) go(std::true_type{});
    else go(std::false_type{});
}

template <int GEO>
bool cell_rhs(int b, const CellArgs<double>& L, int bdf, double chi, double cU, double cM, const double* U,
              const double* Up, const double* iapp, const double* g, double* out, double* xout, hipStream_t st) {
    const unsigned n = (unsigned)((L.n + 63) / 64);
    auto go = [&](auto bc) {
        hipLaunchKernelGGL((k_rhs_cell<decltype(bc)::value, GEO>), dim3(n), dim3(256), 0, st, L, bdf, chi, cU, 1.0 / cM, U, Up,
                           iapp, g, out, xout);
        return true;
    };
    switch (b) {
        case 9: return go(std::integral_constant<int, 9>{});
        case 16: return go(std::integral_constant<int, 16>{});
        case 25: return go(std::integral_constant<int, 25>{});
        case 27: return go(std::integral_constant<int, 27>{});
    }
    return false;
}
#define DGMG_CELL_RHS(GEO)                                                                                          \
    template bool cell_rhs<GEO>(int, const CellArgs<double>&, int, double, double, double, const double*,           \
                                const double*, const double*, const double*, double*, double*, hipStream_t);

#define DGMG_CELL_LAUNCHERS(T, GEO)                                                                                              \
    template void cell_apply<T, GEO>(const LaunchEvents&, int, const CellArgs<T>&, const T*, T*, const T*, double*,      \
                                hipStream_t);                                                                       \
    template void cell_residual<T, GEO>(const LaunchEvents&, int, const CellArgs<T>&, const T*, const T*, const T*, T*,  \
                                   T*, T, T*, double*, const T*, T*, const int32_t*, const T*, hipStream_t);        \
    template void cell_step<T, GEO>(const LaunchEvents&, int, const CellArgs<T>&, const T*, T*, T*, T*, T, T, int, int,  \
                               const T*, hipStream_t);

}  // namespace dgmg
