// Fine levels evaluated per cell (kernels_cell.hpp): arguments and launchers.
#pragma once
#include <hip/hip_runtime.h>

#include <cstdint>

#include "kernels_common.hpp"
#include "launch.hpp"

namespace dgmg {

// Constants of the operator on identical axis-aligned boxes: 1D tables on
// [0,1] (Q = p + 1 Lobatto nodes, Q Gauss points) and the box geometry; D
// points to the per-cell packed (scaled) conductivity.
constexpr int kMfMaxQ = 5;
template <typename T>
struct MfConst {
    T Ig[kMfMaxQ * kMfMaxQ];   // Ig[g*Q + j] = l_j(gauss_g)
    T Gc[kMfMaxQ * kMfMaxQ];   // Gc[g*Q + h] = c_h'(gauss_g), c_h the Lagrange basis on the Gauss points
    T M1[kMfMaxQ * kMfMaxQ];   // M1[i*Q + j] = int l_i l_j
    T N1[kMfMaxQ * kMfMaxQ];   // N1[i*Q + j] = int l_i l_j'
    T Ed[2 * kMfMaxQ];         // Ed[e*Q + j] = l_j'(e), e = 0, 1 (l_j(e) is 0 or 1: Lobatto ends)
    T gw[kMfMaxQ];             // Gauss weights on [0,1]
    T hinv[3];                 // 1 / h_k
    T vol;                     // |K|
    T area[3];                 // |F| of a face normal to axis k
    T eta[3];                  // penalty factor of a face normal to axis k
    T cM;                      // mass coefficient of A_0
    const T* D;                // per cell: packed symmetric D (d(d+1)/2 values)
};
// How a level's cells are evaluated: identical boxes, bilinear / trilinear
// cells with their metric data at the Gauss points, stored blocks of a nodal
// level on a conforming grid of boxes, stored cell blocks (with the cell's
// own face terms) and metric data at the faces' Gauss points, whole stored
// blocks (agglomerates in a grid whose boxes overlap), or whole blocks of 64
// rows, a lane per row.  GEO_BOXR: the kernels that take a small level of boxes
// (GEO_BOX) with a lane per row.
enum { GEO_BOX = 0, GEO_MAP = 1, GEO_BLK = 2, GEO_HYB = 3, GEO_BLD = 4, GEO_ROW = 5, GEO_BOXR = 6 };

// entry (i, j) of a nodal face block along axis a: node i on the lower cell's
// upper face or node j on the upper cell's lower face
__host__ __device__ constexpr bool face_entry(int i, int j, int a, int q) {
    return node_coord(i, a, q) == q - 1 || node_coord(j, a, q) == 0;
}
// entries and 16-byte groups per cell (layout in kernels_cell.hpp)
template <int B, int GEO>
struct CellPack {
    static constexpr int D = dim_of<B>(), Q = ax_nodes_1d(B, D), QN = B / Q;
    static constexpr int NEC = GEO == GEO_MAP ? B * (D * (D + 1) / 2 + 1)
                               : GEO != GEO_BOX ? B * (B + 1) / 2 : 0;
    static constexpr int NEF = GEO == GEO_MAP || GEO == GEO_HYB ? QN * (2 * D + 1)
                               : GEO == GEO_BLD ? B * B
                               : GEO == GEO_BLK ? 2 * QN * B - QN * QN : 0;
    static constexpr int cell_groups(int w) { return (NEC + w - 1) / w; }
    static constexpr int face_groups(int w) { return (NEF + w - 1) / w; }
    static constexpr int groups(int w) { return cell_groups(w) + D * face_groups(w); }
};

template <typename T>
struct CellArgs {
    const int32_t* __restrict__ up;        // [d][n] upper neighbour (itself if none)
    const int32_t* __restrict__ lo;        // [d][n] lower neighbour (-1 if none)
    const T* __restrict__ dinv;
    int32_t n;
    const T* __restrict__ data;            // mapped and stored cells: their entries
    MfConst<T> mf;
};

// Workgroups of the cell kernels on a level of n cells with b x b blocks (the
// number of partial sums they write).
unsigned cell_groups(int geo, int b, int n);

// The cell forms of k_apply, k_residual and k_cheb_step (same arguments).
template <typename T, int GEO>
void cell_apply(const LaunchEvents& ev, int b, const CellArgs<T>& L, const T* va, T* y, const T* w, double* partial,
                hipStream_t st);
template <typename T, int GEO>
void cell_residual(const LaunchEvents& ev, int b, const CellArgs<T>& L, const T* va, const T* vb, const T* rhs, T* r,
                   T* d, T c1, T* xout, double* partial, const T* P, T* rp, const int32_t* ptype, const T* bj,
                   hipStream_t st);
template <typename T, int GEO>
void cell_step(const LaunchEvents& ev, int b, const CellArgs<T>& L, const T* d, T* x, T* r, T* dn, T cd, T cr,
               int assign, int last, const T* bj, hipStream_t st);

// The load vector (k_rhs) on boxes and mapped cells; false where the block size
// has no such kernel.  cM: mass coefficient of the level's operator.
template <int GEO>
bool cell_rhs(int b, const CellArgs<double>& L, int bdf, double chi, double cU, double cM, const double* U,
              const double* Up, const double* iapp, const double* g, double* out, double* xout, hipStream_t st);

// geometry GEO of a level as a constant
#define DISPATCH_GEO(gval, ...)                                                        \
    switch (gval) {                                                                    \
        case GEO_BOX: { constexpr int GEO = GEO_BOX; __VA_ARGS__; } break;             \
        case GEO_MAP: { constexpr int GEO = GEO_MAP; __VA_ARGS__; } break;             \
        case GEO_BLK: { constexpr int GEO = GEO_BLK; __VA_ARGS__; } break;             \
        case GEO_HYB: { constexpr int GEO = GEO_HYB; __VA_ARGS__; } break;             \
        case GEO_BLD: { constexpr int GEO = GEO_BLD; __VA_ARGS__; } break;             \
        default: { constexpr int GEO = GEO_ROW; __VA_ARGS__; } break;                  \
    }

}  // namespace dgmg
