// Level operators evaluated per cell: fine levels (section 3: cell and
// interior-face terms of a_h and the mass term of eq. fully_discrete) by sum
// factorisation on boxes and mapped cells, Q1 levels from cell blocks and face
// data, agglomerated levels from stored blocks.
//
// Mapping: a workgroup takes 64 or 16 consecutive cells, one per lane, and has a
// wave for the cell terms and one per axis, which evaluates both faces normal to
// it (stored blocks: one per face), each lane with its cell's B values in
// registers: every 1D pass is register arithmetic with wave-uniform (scalar
// register) table entries, so there is no LDS traffic or barrier between
// passes.  Each wave leaves its share of the B rows in LDS; after the only
// barrier the epilogue sums the shares in wave order, a lane per row, with
// coalesced vector accesses.  3D Q3 cells take four lanes each, agglomerates of
// 64 DoFs a workgroup, small levels of Q4 squares a lane per row.
//
// Boxes: on extents h the Q_p basis is a tensor product of 1D Lagrange
// polynomials on Gauss-Lobatto nodes, the Gauss-Legendre rule with p+1 points
// integrates every cell and face term exactly, and the only per-cell data is
// the (scaled) conductivity D_K.
//   cell:  nodal values to the Gauss points by D 1D passes, gradients there by
//          the collocation derivative G, the weighted fluxes, and the
//          transposed passes;
//   face:  the traces (Lobatto end layers) and normal derivatives of both
//          sides; the tangential integrals are the 1D matrices
//          M_ij = int l_i l_j and N_ij = int l_i l_j', applied to
//            q0 = -s/2 (k_a d_K + k_a^N d_N) + sigma (u_K - u_N),
//            q_t = -s/2 (k_t u_K + k_t^N u_N),  jc = -s/2 (u_K - u_N),
//          with k_c = D[a][c] / h_c and s = +1 on the cell's upper side.
// Bound: FP32 arithmetic of one lane per cell (about 3,800 multiply-adds per
// 3D Q2 cell, 140 per DoF) beside the vector streams; 64^3 Q2, FP32 Chebyshev
// step: 46 us, 4.4 TB/s on its 202 MB (a thread per DoF with every pass through
// LDS and eight barriers: 150 us, LDS busy 91%); FP64 130 us (286 us); 128^2 Q4
// FP64 7.6 us (17.2 us); 16^3 Q3 FP64 8.3 us (18.0 us).  The other forms' figures
// stand beside them.
// Included by cell_launch.hpp, in one translation unit per form (cell_*.hip).
#pragma once
#include <hip/hip_runtime.h>

#include <cstddef>
#include <cstdint>
#include <type_traits>

#include "cell.hpp"
#include "kernels_common.hpp"

namespace dgmg {

template <int D>
constexpr int npack() {
    return D * (D + 1) / 2;
}
// packed symmetric index of (a, b): 2D (xx, xy, yy); 3D (xx, xy, xz, yy, yz, zz)
template <int D>
constexpr int pk(int a, int b) {
    const int lo = a < b ? a : b, hi = a < b ? b : a;
    return D == 2 ? lo + hi : (lo == 0 ? hi : (lo == 1 ? 2 + hi : 5));
}

// threads per workgroup: a wave for the cell terms and one per axis, or per
// face where the faces' blocks are streamed
template <int B, int GEO>
constexpr int cell_threads() {
    return GEO == GEO_BOXR ? kWG : 64 * (1 + (GEO == GEO_BLK || GEO == GEO_BLD || GEO == GEO_ROW ? 2 : 1) * dim_of<B>());
}
template <typename T, int B, int NCELL, int GEO = GEO_BOX>
struct CellTile {
    static constexpr int D = dim_of<B>(), Q = ax_nodes_1d(B, D), QN = B / Q;
    static constexpr int NC = NCELL;                  // cells per workgroup, one per lane
    static constexpr int NT = cell_threads<B, GEO>();
    static constexpr int NS = GEO == GEO_BOXR ? 1 : NT / 64;   // shares of a row's product
    static constexpr int SB = GEO == GEO_ROW ? B : B | 1;   // odd LDS stride of a cell's rows
};

// vector of 16 bytes at the alignment of its elements (a cell's values start
// at a multiple of B elements)
template <typename T>
struct Vec16;
template <>
struct Vec16<float> {
    typedef float type __attribute__((ext_vector_type(4), aligned(4)));
};
template <>
struct Vec16<double> {
    typedef double type __attribute__((ext_vector_type(2), aligned(8)));
};

// the B values of cell c of va (+ vb)
template <typename T, int B, bool VB>
__device__ __forceinline__ void load_cell(const T* __restrict__ va, const T* __restrict__ vb, int c, T* x) {
    using V = typename Vec16<T>::type;
    constexpr int W = 16 / sizeof(T);
    const T* p = va + (size_t)c * B;
#pragma unroll
    for (int k = 0; k + W <= B; k += W) {
        const V v = *reinterpret_cast<const V*>(p + k);
#pragma unroll
        for (int q = 0; q < W; ++q) x[k + q] = v[q];
    }
#pragma unroll
    for (int k = B / W * W; k < B; ++k) x[k] = p[k];
    if constexpr (VB) {
        T y[B];
        load_cell<T, B, false>(vb, nullptr, c, y);
#pragma unroll
        for (int k = 0; k < B; ++k) x[k] += y[k];
    }
}

// Ends a stage of the box terms.  The FP64 tables of Q = 5 take 50 scalar
// registers each, and the scheduler, which hoists their loads, spilled them to
// vector lanes (1,022 lane accesses of 5,297 instructions in one step): no load
// crosses a stage.  128^2 Q4 boxes, FP64 step 8.3 -> 7.6 us; 256^2: step 21.0 -> 19.7,
// residual of a pending update 33.3 -> 31.1, product 15.7 -> 14.4 us.
template <typename T, int B>
__device__ __forceinline__ void stage_end() {
    if constexpr (B == 25 && sizeof(T) == 8) __builtin_amdgcn_sched_barrier(0);
}
constexpr int ipow(int q, int e) { return e == 0 ? 1 : q * ipow(q, e - 1); }

// u <- (1D matrix M along axis A of the Q^D array) u; TR: its transpose
template <typename T, int Q, int D, int A, bool TR>
__device__ __forceinline__ void line_pass(T* u, const T* M) {
    constexpr int S = ipow(Q, A), N = ipow(Q, D);
#pragma unroll
    for (int k = 0; k < N / Q; ++k) {
        const int base = (k / S) * S * Q + k % S;
        T t[Q];
#pragma unroll
        for (int g = 0; g < Q; ++g) {
            T s = 0;
#pragma unroll
            for (int j = 0; j < Q; ++j) s += (TR ? M[j * Q + g] : M[g * Q + j]) * u[base + j * S];
            t[g] = s;
        }
#pragma unroll
        for (int g = 0; g < Q; ++g) u[base + g * S] = t[g];
    }
}
template <typename T, int Q, int D, bool TR>
__device__ __forceinline__ void all_passes(T* u, const T* M) {
    if constexpr (D > 0) line_pass<T, Q, D, 0, TR>(u, M);
    if constexpr (D > 1) line_pass<T, Q, D, 1, TR>(u, M);
    if constexpr (D > 2) line_pass<T, Q, D, 2, TR>(u, M);
}

// Cell terms of cell c: cM w u and the fluxes w D grad u, tested.
template <typename T, int B, int NC, bool VB>
__device__ __forceinline__ void box_cell_terms(const CellArgs<T>& L, int c, const T* __restrict__ va,
                                           const T* __restrict__ vb, T* ys) {
    using Ct = CellTile<T, B, NC>;
    constexpr int D = Ct::D, Q = Ct::Q, NP = npack<D>();
    const MfConst<T>& C = L.mf;
    T u[B], y[B], Dk[NP];
    load_cell<T, B, VB>(va, vb, c, u);
    stage_end<T, B>();
#pragma unroll
    for (int k = 0; k < NP; ++k) Dk[k] = C.D[(size_t)c * NP + k];
#pragma unroll
    for (int a = 0; a < D; ++a)
#pragma unroll
        for (int b = a; b < D; ++b) Dk[pk<D>(a, b)] *= C.vol * C.hinv[a] * C.hinv[b];
    const T mass = C.vol * C.cM;
    all_passes<T, Q, D, false>(u, C.Ig);
    stage_end<T, B>();
#pragma unroll
    for (int g = 0; g < B; ++g) y[g] = 0;
#pragma unroll
    for (int g = 0; g < B; ++g) {
        const int gc[3] = {node_coord(g, 0, Q), node_coord(g, 1, Q), D == 3 ? node_coord(g, 2, Q) : 0};
        const T w = D == 3 ? C.gw[gc[0]] * C.gw[gc[1]] * C.gw[gc[2]] : C.gw[gc[0]] * C.gw[gc[1]];
        T gr[D];
#pragma unroll
        for (int a = 0; a < D; ++a) {
            T s = 0;
#pragma unroll
            for (int h = 0; h < Q; ++h) s += C.Gc[gc[a] * Q + h] * u[g + (h - gc[a]) * ipow(Q, a)];
            gr[a] = s;
        }
        y[g] += w * mass * u[g];
#pragma unroll
        for (int a = 0; a < D; ++a) {
            T f = 0;
#pragma unroll
            for (int b = 0; b < D; ++b) f += Dk[pk<D>(a, b)] * gr[b];
            f *= w;
#pragma unroll
            for (int h = 0; h < Q; ++h) y[g + (h - gc[a]) * ipow(Q, a)] += C.Gc[gc[a] * Q + h] * f;
        }
    }
    stage_end<T, B>();
    all_passes<T, Q, D, true>(y, C.Ig);
#pragma unroll
    for (int i = 0; i < B; ++i) ys[i] = y[i];
}

// Both faces of cell c normal to axis A.
template <typename T, int B, int NC, bool VB, int A>
__device__ __forceinline__ void box_face_terms(const CellArgs<T>& L, int c, const T* __restrict__ va,
                                           const T* __restrict__ vb, T* ys) {
    using Ct = CellTile<T, B, NC>;
    constexpr int D = Ct::D, Q = Ct::Q, QN = Ct::QN, NP = npack<D>();
    constexpr int SA = ipow(Q, A);                        // stride of the normal direction
    constexpr int t1 = A == 0 ? 1 : 0, t2 = D == 3 ? (A == 2 ? 1 : 2) : t1;
    constexpr int S1 = ipow(Q, t1), S2 = D == 3 ? ipow(Q, t2) : 0;
    const MfConst<T>& C = L.mf;
    const int lo = L.lo[(size_t)A * L.n + c], up = L.up[(size_t)A * L.n + c];
    const int nb[2] = {lo >= 0 ? lo : c, up};
    const bool has[2] = {lo >= 0, up != c};
    T xk[B], DK[D], DN[2][D];
    load_cell<T, B, VB>(va, vb, c, xk);
    stage_end<T, B>();
    const T daa = C.D[(size_t)c * NP + pk<D>(A, A)];
#pragma unroll
    for (int k = 0; k < D; ++k) {
        DK[k] = C.D[(size_t)c * NP + pk<D>(A, k)] * C.hinv[k];
        DN[0][k] = C.D[(size_t)nb[0] * NP + pk<D>(A, k)] * C.hinv[k];
        DN[1][k] = C.D[(size_t)nb[1] * NP + pk<D>(A, k)] * C.hinv[k];
    }
    T T0[2][QN], Tn[2][QN];
#pragma unroll
    for (int s = 0; s < 2; ++s) {
        T xn[B];
        load_cell<T, B, VB>(va, vb, nb[s], xn);
        stage_end<T, B>();
        const T ar = has[s] ? C.area[A] : T(0);
        const T hs = (s ? T(-0.5) : T(0.5)) * ar;         // -s/2, area folded in
        const T sig = C.eta[A] * T(0.5) * (daa + C.D[(size_t)nb[s] * NP + pk<D>(A, A)]) * ar;
        T q0[QN], q1[QN], q2[QN], jc[QN];
#pragma unroll
        for (int m = 0; m < QN; ++m) {
            const int J0 = (m % Q) * S1 + (m / Q) * S2;
            T dK = 0, dN = 0;
#pragma unroll
            for (int j = 0; j < Q; ++j) {
                dK += C.Ed[s * Q + j] * xk[J0 + j * SA];
                dN += C.Ed[(1 - s) * Q + j] * xn[J0 + j * SA];
            }
            const T uK = xk[J0 + s * (Q - 1) * SA], uN = xn[J0 + (1 - s) * (Q - 1) * SA];
            const T j = uK - uN;
            q0[m] = hs * (DK[A] * dK + DN[s][A] * dN) + sig * j;
            q1[m] = hs * (DK[t1] * uK + DN[s][t1] * uN);
            q2[m] = D == 3 ? hs * (DK[t2] * uK + DN[s][t2] * uN) : T(0);
            jc[m] = hs * j;
        }
        stage_end<T, B>();
        if constexpr (D == 2) {
            // one table at a time: M, then N (stage_end)
            T v[Q], w[Q];
#pragma unroll
            for (int i = 0; i < Q; ++i) {
                T a = 0, n = 0;
#pragma unroll
                for (int j = 0; j < Q; ++j) {
                    a += C.M1[i * Q + j] * q0[j];
                    n += C.M1[i * Q + j] * jc[j];
                }
                v[i] = a;
                Tn[s][i] = DK[A] * n;
            }
            stage_end<T, B>();
#pragma unroll
            for (int i = 0; i < Q; ++i) {
                T a = v[i], e = 0;
#pragma unroll
                for (int j = 0; j < Q; ++j) {
                    a += C.N1[i * Q + j] * q1[j];
                    e += C.N1[j * Q + i] * jc[j];
                }
                T0[s][i] = a + DK[t1] * e;
            }
            stage_end<T, B>();
        } else {
            // tangential direction t1, in place line by line: q0 <- M q0 + N q1
            // + k1 N^T jc, q2 <- M q2, jc <- M jc; then t2
#pragma unroll
            for (int m2 = 0; m2 < Q; ++m2) {
                T a[Q], b[Q], e[Q];
#pragma unroll
                for (int i = 0; i < Q; ++i) {
                    T v = 0, w = 0, x = 0, z = 0;
#pragma unroll
                    for (int j = 0; j < Q; ++j) {
                        const int m = j + Q * m2;
                        v += C.M1[i * Q + j] * q0[m] + C.N1[i * Q + j] * q1[m];
                        w += C.N1[j * Q + i] * jc[m];
                        x += C.M1[i * Q + j] * q2[m];
                        z += C.M1[i * Q + j] * jc[m];
                    }
                    a[i] = v + DK[t1] * w;
                    b[i] = x;
                    e[i] = z;
                }
#pragma unroll
                for (int i = 0; i < Q; ++i) {
                    q0[i + Q * m2] = a[i];
                    q2[i + Q * m2] = b[i];
                    jc[i + Q * m2] = e[i];
                }
            }
#pragma unroll
            for (int m1 = 0; m1 < Q; ++m1)
#pragma unroll
                for (int i = 0; i < Q; ++i) {
                    T v = 0, n = 0, w = 0;
#pragma unroll
                    for (int j = 0; j < Q; ++j) {
                        const int m = m1 + Q * j;
                        v += C.M1[i * Q + j] * q0[m] + C.N1[i * Q + j] * q2[m];
                        w += C.N1[j * Q + i] * jc[m];
                        n += C.M1[i * Q + j] * jc[m];
                    }
                    T0[s][m1 + Q * i] = v + DK[t2] * w;
                    Tn[s][m1 + Q * i] = DK[A] * n;
                }
        }
    }
    stage_end<T, B>();
    // test functions: the trace at the two end layers, the end derivative on every layer
#pragma unroll
    for (int m = 0; m < QN; ++m) {
        const int J0 = (m % Q) * S1 + (m / Q) * S2;
#pragma unroll
        for (int j = 0; j < Q; ++j) {
            T v = C.Ed[j] * Tn[0][m] + C.Ed[Q + j] * Tn[1][m];
            if (j == 0) v += T0[0][m];
            if (j == Q - 1) v += T0[1][m];
            ys[J0 + j * SA] = v;
        }
    }
}

// ---- per-cell data of mapped and stored cells
// Entries of cell c, 16 bytes (W values) per lane and load: group g at
// data + ((c / 64) NG + g) 64 W + (c % 64) W, so that the 64 lanes of
// consecutive cells read 1 KiB.  Groups 0 .. NGC - 1 belong to the cell, then
// NGF groups per axis to the face on its upper side.  The face on the lower
// side is read from the lower neighbour's groups.
template <typename T>
struct Vec16a;
template <>
struct Vec16a<float> {
    typedef float type __attribute__((ext_vector_type(4)));
};
template <>
struct Vec16a<double> {
    typedef double type __attribute__((ext_vector_type(2)));
};
template <typename T, int NE>
struct Stream {
    using V = typename Vec16a<T>::type;
    static constexpr int W = 16 / sizeof(T);
    const V* p;
    V v;
    __device__ __forceinline__ Stream(const T* base) : p(reinterpret_cast<const V*>(base)) {}
    // entry e (compile-time after unrolling), entries in ascending order
    __device__ __forceinline__ T get(int e) {
        if (e % W == 0) v = p[(size_t)(e / W) * 64];
        return v[e % W];
    }
};
// Groups requested ahead: 64^3 Q2's level of 32,768 boxes, FP32 step at 4 / 8 /
// 12 / 16 groups 44 / 49 / 42 / 42 us, FP64 94 / 97 / 102 / 102 us.
template <typename T>
constexpr int ring_groups() {
    return sizeof(T) == 4 ? 12 : 4;
}
// f(e, entry e) for the NE entries of a stored block in order, with R groups
// requested ahead of the one in use (the loads of the straight-line products
// would otherwise all be hoisted into hundreds of live registers).
template <typename T, int NE, int R, typename F>
__device__ __forceinline__ void stream_entries(const T* base, F&& f) {
    using V = typename Vec16a<T>::type;
    constexpr int W = 16 / sizeof(T), NG = (NE + W - 1) / W, RG = R < NG ? R : NG;
    const V* p = reinterpret_cast<const V*>(base);
    V ring[RG];
#pragma unroll
    for (int g = 0; g < RG; ++g) ring[g] = p[(size_t)g * 64];
    p += RG * 64;
#pragma unroll
    for (int g = 0; g < NG; ++g) {
        const V v = ring[g % RG];
        if (g + RG < NG) {
            int off = g * 64;
            asm volatile("" : "+v"(off) : "v"(v[0]));   // the next request follows this group's arrival
            ring[g % RG] = p[off];
        }
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int w = 0; w < W; ++w)
            if (g * W + w < NE) f(g * W + w, v[w]);
    }
}
// (row, column) of the stored entries in their order
template <int B>
struct TriList {
    unsigned char i[B * (B + 1) / 2] = {}, j[B * (B + 1) / 2] = {};
    constexpr TriList() {
        int e = 0;
        for (int a = 0; a < B; ++a)
            for (int b = a; b < B; ++b, ++e) {
                i[e] = (unsigned char)a;
                j[e] = (unsigned char)b;
            }
    }
};
template <int B, int A, int GEO>
struct FaceList {
    unsigned char i[CellPack<B, GEO>::NEF] = {}, j[CellPack<B, GEO>::NEF] = {};
    constexpr FaceList() {
        int e = 0;
        for (int a = 0; a < B; ++a)
            for (int b = 0; b < B; ++b)
                if (GEO == GEO_BLD || face_entry(a, b, A, CellPack<B, GEO>::Q)) {
                    i[e] = (unsigned char)a;
                    j[e++] = (unsigned char)b;
                }
    }
};
template <typename T, int B, int GEO>
__device__ __forceinline__ const T* cell_data(const CellArgs<T>& L, int c, int group) {
    using P = CellPack<B, GEO>;
    constexpr int W = 16 / sizeof(T), NG = P::groups(W);
    return L.data + (((size_t)(c >> 6) * NG + group) * 64 + (c & 63)) * W;
}

// ---- mapped cells (bilinear / trilinear geometry): per Gauss point the
// weighted metric tensor w J^-1 D J^-T and the mass weight
template <typename T, int B, int NC, bool VB>
__device__ __forceinline__ void map_cell_terms(const CellArgs<T>& L, int c, const T* __restrict__ va,
                                               const T* __restrict__ vb, T* ys) {
    using Ct = CellTile<T, B, NC>;
    constexpr int D = Ct::D, Q = Ct::Q, NP = npack<D>();
    const MfConst<T>& C = L.mf;
    T u[B], y[B];
    load_cell<T, B, VB>(va, vb, c, u);
    all_passes<T, Q, D, false>(u, C.Ig);
#pragma unroll
    for (int g = 0; g < B; ++g) y[g] = 0;
    Stream<T, B*(NP + 1)> K(cell_data<T, B, GEO_MAP>(L, c, 0));
#pragma unroll
    for (int g = 0; g < B; ++g) {
        const int gc[3] = {node_coord(g, 0, Q), node_coord(g, 1, Q), D == 3 ? node_coord(g, 2, Q) : 0};
        T k[NP + 1], gr[D];
#pragma unroll
        for (int q = 0; q <= NP; ++q) k[q] = K.get(g * (NP + 1) + q);
#pragma unroll
        for (int a = 0; a < D; ++a) {
            T s = 0;
#pragma unroll
            for (int h = 0; h < Q; ++h) s += C.Gc[gc[a] * Q + h] * u[g + (h - gc[a]) * ipow(Q, a)];
            gr[a] = s;
        }
        y[g] += k[NP] * u[g];
#pragma unroll
        for (int a = 0; a < D; ++a) {
            T f = 0;
#pragma unroll
            for (int b = 0; b < D; ++b) f += k[pk<D>(a, b)] * gr[b];
#pragma unroll
            for (int h = 0; h < Q; ++h) y[g + (h - gc[a]) * ipow(Q, a)] += C.Gc[gc[a] * Q + h] * f;
        }
    }
    all_passes<T, Q, D, true>(y, C.Ig);
#pragma unroll
    for (int i = 0; i < B; ++i) ys[i] = y[i];
}

// Both faces normal to A.  Per Gauss point of a face: p = -w/2 J_+^-1 D_+ n and
// m = -w/2 J_-^-1 D_- n as weights of the reference gradients (normal, t1, t2)
// of the lower (+) and upper (-) cell, and w sigma.  With j = u_own - u_nb, the
// value flux is (o + v)_t d_t u_own - v_t d_t j + o_n d_own + v_n d_nb + w sigma j
// up to the side's sign (o, v: the own and the neighbour's weights), and the
// conormal flux o j is tested against the reference gradient.
template <typename T, int B, int NC, bool VB, int A>
__device__ __forceinline__ void map_face_terms(const CellArgs<T>& L, int c, const T* __restrict__ va,
                                               const T* __restrict__ vb, T* ys) {
    using Ct = CellTile<T, B, NC>;
    constexpr int D = Ct::D, Q = Ct::Q, QN = Ct::QN;
    constexpr int SA = ipow(Q, A);
    constexpr int t1 = A == 0 ? 1 : 0, t2 = D == 3 ? (A == 2 ? 1 : 2) : t1;
    constexpr int S1 = ipow(Q, t1), S2 = D == 3 ? ipow(Q, t2) : 0;
    constexpr int NE = 2 * D + 1, W = 16 / sizeof(T);
    using P = CellPack<B, GEO_MAP>;
    const MfConst<T>& C = L.mf;
    const int lo = L.lo[(size_t)A * L.n + c], up = L.up[(size_t)A * L.n + c];
    const int nb[2] = {lo >= 0 ? lo : c, up};
    const bool has[2] = {lo >= 0, up != c};
    T xk[B], T0[2][QN], Tn[2][QN];
    load_cell<T, B, VB>(va, vb, c, xk);
#pragma unroll
    for (int s = 0; s < 2; ++s) {
        T xn[B];
        load_cell<T, B, VB>(va, vb, nb[s], xn);
        Stream<T, NE * QN> F(cell_data<T, B, GEO_MAP>(L, s ? c : nb[0], P::cell_groups(W) + A * P::face_groups(W)));
        T uK[QN], jp[QN], dK[QN], dN[QN], acc[QN], cn[QN];
#pragma unroll
        for (int m = 0; m < QN; ++m) {
            const int J0 = (m % Q) * S1 + (m / Q) * S2;
            T a = 0, b = 0;
#pragma unroll
            for (int j = 0; j < Q; ++j) {
                a += C.Ed[s * Q + j] * xk[J0 + j * SA];
                b += C.Ed[(1 - s) * Q + j] * xn[J0 + j * SA];
            }
            dK[m] = a;
            dN[m] = b;
            uK[m] = xk[J0 + s * (Q - 1) * SA];
            jp[m] = uK[m] - xn[J0 + (1 - s) * (Q - 1) * SA];
            acc[m] = 0;
        }
        all_passes<T, Q, D - 1, false>(uK, C.Ig);
        all_passes<T, Q, D - 1, false>(jp, C.Ig);
        all_passes<T, Q, D - 1, false>(dK, C.Ig);
        all_passes<T, Q, D - 1, false>(dN, C.Ig);
#pragma unroll
        for (int q = 0; q < QN; ++q) {
            const int q1 = q % Q, q2 = q / Q;
            T f[NE];
#pragma unroll
            for (int k = 0; k < NE; ++k) f[k] = F.get(q * NE + k);
            const T* o = s ? f : f + D;                   // own weights, then the neighbour's
            const T* v = s ? f + D : f;
            T val = o[0] * dK[q] + v[0] * dN[q] + (s ? f[2 * D] : -f[2 * D]) * jp[q];
            // the jump u_+ - u_- is j on the upper face, -j on the lower one;
            // the own test function enters with the same sign
            const T js = s ? jp[q] : -jp[q];
#pragma unroll
            for (int h = 0; h < Q; ++h) {
                const int m = h + Q * q2;
                val += C.Gc[q1 * Q + h] * ((o[1] + v[1]) * uK[m] - v[1] * jp[m]);
                acc[m] += C.Gc[q1 * Q + h] * (o[1] * js);
                if constexpr (D == 3) {
                    const int n = q1 + Q * h;
                    val += C.Gc[q2 * Q + h] * ((o[2] + v[2]) * uK[n] - v[2] * jp[n]);
                    acc[n] += C.Gc[q2 * Q + h] * (o[2] * js);
                }
            }
            acc[q] += s ? val : -val;
            cn[q] = o[0] * js;
        }
        all_passes<T, Q, D - 1, true>(acc, C.Ig);
        all_passes<T, Q, D - 1, true>(cn, C.Ig);
#pragma unroll
        for (int m = 0; m < QN; ++m) {
            T0[s][m] = has[s] ? acc[m] : T(0);
            Tn[s][m] = has[s] ? cn[m] : T(0);
        }
    }
#pragma unroll
    for (int m = 0; m < QN; ++m) {
        const int J0 = (m % Q) * S1 + (m / Q) * S2;
#pragma unroll
        for (int j = 0; j < Q; ++j) {
            T v = C.Ed[j] * Tn[0][m] + C.Ed[Q + j] * Tn[1][m];
            if (j == 0) v += T0[0][m];
            if (j == Q - 1) v += T0[1][m];
            ys[J0 + j * SA] = v;
        }
    }
}

// ---- stored blocks: the upper triangle of the cell block, and the face
// block's entries (i, j) with node i on the upper face or node j on the
// neighbour's lower face (the others vanish on a nodal level; GEO_BLD holds all
// of them).  Every entry is
// read coalesced, also by the cell above a face, whose transposed reads by a
// thread per row touched a line per lane: level 1 of the 64^3 Q2 cube (32,768
// boxes of 27 DoFs, 209 MB of entries), FP32 step 92 -> 42 us, FP64 260 -> 94.
template <typename T, int B, int NC, bool VB, int GEO>
__device__ __forceinline__ void blk_cell_terms(const CellArgs<T>& L, int c, const T* __restrict__ va,
                                               const T* __restrict__ vb, T* ys) {
    T x[B], y[B];
    load_cell<T, B, VB>(va, vb, c, x);
#pragma unroll
    for (int i = 0; i < B; ++i) y[i] = 0;
    constexpr TriList<B> tri;
    stream_entries<T, B*(B + 1) / 2, ring_groups<T>()>(cell_data<T, B, GEO>(L, c, 0), [&](int e, T a) {
        const int i = tri.i[e], j = tri.j[e];
        y[i] += a * x[j];
        if (j > i) y[j] += a * x[i];
    });
#pragma unroll
    for (int i = 0; i < B; ++i) ys[i] = y[i];
}
template <typename T, int B, bool VB, int GEO, int A, int S>
__device__ __forceinline__ void blk_face_terms(const CellArgs<T>& L, int c, const T* __restrict__ va,
                                               const T* __restrict__ vb, T* ys) {
    constexpr int W = 16 / sizeof(T);
    using P = CellPack<B, GEO>;
    constexpr FaceList<B, A, GEO> list;
    // no lower neighbour: the products are dropped with zero values (a missing
    // upper face has zero entries)
    const int v = (S ? L.up : L.lo)[(size_t)A * L.n + c], nb = v >= 0 ? v : c;
    T x[B], y[B];
    load_cell<T, B, VB>(va, vb, nb, x);
#pragma unroll
    for (int i = 0; i < B; ++i) {
        x[i] = v >= 0 ? x[i] : T(0);
        y[i] = 0;
    }
    stream_entries<T, P::NEF, ring_groups<T>()>(
        cell_data<T, B, GEO>(L, S ? c : nb, P::cell_groups(W) + A * P::face_groups(W)), [&](int e, T a) {
            const int i = list.i[e], j = list.j[e];
            if (S) y[i] += a * x[j];
            else y[j] += a * x[i];
        });
#pragma unroll
    for (int i = 0; i < B; ++i) ys[i] = y[i];
}

// ---- 3D Q3 agglomerates: a workgroup per cell, a wave per block, a lane per
// row.  Blocks are whole, W columns interleaved: entry (i, j) at
// (j / W) 64 W + i W + j % W of a cell's own block and then its upper faces'.  A
// wave with all seven blocks of its cell waited for a dozen memory round trips
// one after the other (512 cells, FP64 step: 24.5 us, 14.8 us here; 64 cells 19.3,
// 5.5 us).
// sum over the wave's lanes l of P_l[i mod 16], at lane i
template <typename T>
__device__ __forceinline__ T reduce_columns16(T* P, int i) {
#pragma unroll
    for (int h = 8; h > 0; h >>= 1) {
        const bool up = (i & h) != 0;
#pragma unroll
        for (int j = 0; j < h; ++j) {
            // values, not elements: a choice of elements would index P dynamically
            const T a = P[j], b = P[j + h], mine = up ? b : a, give = up ? a : b;
            P[j] = mine + __shfl_xor(give, h, 64);
        }
    }
    T s = P[0];
    s += __shfl_xor(s, 16, 64);
    return s + __shfl_xor(s, 32, 64);
}
template <typename T>
__device__ __forceinline__ T lane_value(T v, int j);
template <>
__device__ __forceinline__ float lane_value<float>(float v, int j) {
    return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), j));
}
template <>
__device__ __forceinline__ double lane_value<double>(double v, int j) {
    return __hiloint2double(__builtin_amdgcn_readlane(__double2hiint(v), j),
                            __builtin_amdgcn_readlane(__double2loint(v), j));
}
// wave w of cell c: 0 its own block, 1 + 2 a + s the face on side s of axis a
template <typename T, bool VB>
__device__ __forceinline__ T row_terms(const CellArgs<T>& L, int c, int w, int lane, const T* __restrict__ va,
                                       const T* __restrict__ vb) {
    using V = typename Vec16a<T>::type;
    constexpr int W = 16 / sizeof(T), NV = 64 / W, HV = NV / 2;
    const int a = (w - 1) >> 1, side = (w - 1) & 1;
    const int nb = w == 0 ? c : (side ? L.up : L.lo)[(size_t)a * L.n + c];
    if (nb < 0 || (w > 0 && nb == c)) return T(0);        // no neighbour (uniform)
    const bool low = w > 0 && !side;
    const V* F = reinterpret_cast<const V*>(L.data + ((size_t)(low ? nb : c) * 4 + (w ? 1 + a : 0)) * 4096) + lane;
    T x = va[(size_t)nb * 64 + lane];
    if constexpr (VB) x += vb[(size_t)nb * 64 + lane];
    T acc = 0;
#pragma unroll
    for (int h = 0; h < 2; ++h) {                          // half of the columns' loads in flight
        V f[HV];
#pragma unroll
        for (int k = 0; k < HV; ++k) f[k] = F[(size_t)(h * HV + k) * 64];
        if (!low) {
#pragma unroll
            for (int k = 0; k < HV; ++k)
#pragma unroll
                for (int q = 0; q < W; ++q) acc += f[k][q] * lane_value(x, (h * HV + k) * W + q);
        } else {
            // transposed: column j summed over the lanes' rows, 16 at a time
#pragma unroll
            for (int g = 0; g < 2; ++g) {
                T P[16];
#pragma unroll
                for (int j = 0; j < 16; ++j) P[j] = f[(g * 16 + j) / W][j % W] * x;
                const T r = reduce_columns16(P, lane);
                acc += (lane >> 4) == h * 2 + g ? r : T(0);
            }
        }
    }
    return acc;
}

// ---- Q1 cells: the stored cell block holds the cell's own face terms, and
// the neighbours' terms come from the faces' metric data (28 values per 3D
// face against 48 nonzeros of its block): map_face_terms with u_own = 0.
template <typename T, int B, bool VB, int A>
__device__ __forceinline__ void hyb_face_terms(const CellArgs<T>& L, int c, const T* __restrict__ va,
                                               const T* __restrict__ vb, T* ys) {
    using P = CellPack<B, GEO_HYB>;
    constexpr int D = P::D, Q = P::Q, QN = P::QN, SA = ipow(Q, A);
    constexpr int t1 = A == 0 ? 1 : 0, t2 = D == 3 ? (A == 2 ? 1 : 2) : t1;
    constexpr int S1 = ipow(Q, t1), S2 = D == 3 ? ipow(Q, t2) : 0;
    constexpr int NE = 2 * D + 1, W = 16 / sizeof(T);
    const MfConst<T>& C = L.mf;
    const int lo = L.lo[(size_t)A * L.n + c], up = L.up[(size_t)A * L.n + c];
    const int nb[2] = {lo >= 0 ? lo : c, up};
    const bool has[2] = {lo >= 0, up != c};
    T T0[2][QN], Tn[2][QN];
#pragma unroll
    for (int s = 0; s < 2; ++s) {
        T xn[B], un[QN], dn[QN], acc[QN], cn[QN];
        load_cell<T, B, VB>(va, vb, nb[s], xn);
        Stream<T, NE * QN> F(cell_data<T, B, GEO_HYB>(L, s ? c : nb[0], P::cell_groups(W) + A * P::face_groups(W)));
#pragma unroll
        for (int m = 0; m < QN; ++m) {
            const int J0 = (m % Q) * S1 + (m / Q) * S2;
            T b = 0;
#pragma unroll
            for (int j = 0; j < Q; ++j) b += C.Ed[(1 - s) * Q + j] * xn[J0 + j * SA];
            dn[m] = b;
            un[m] = xn[J0 + (1 - s) * (Q - 1) * SA];
            acc[m] = 0;
        }
        all_passes<T, Q, D - 1, false>(un, C.Ig);
        all_passes<T, Q, D - 1, false>(dn, C.Ig);
#pragma unroll
        for (int q = 0; q < QN; ++q) {
            const int q1 = q % Q, q2 = q / Q;
            T f[NE];
#pragma unroll
            for (int k = 0; k < NE; ++k) f[k] = F.get(q * NE + k);
            const T* o = s ? f : f + D;                   // own weights, then the neighbour's
            const T* v = s ? f + D : f;
            T val = v[0] * dn[q] - (s ? f[2 * D] : -f[2 * D]) * un[q];
            const T js = s ? -un[q] : un[q];
#pragma unroll
            for (int h = 0; h < Q; ++h) {
                const int m = h + Q * q2;
                val += C.Gc[q1 * Q + h] * (v[1] * un[m]);
                acc[m] += C.Gc[q1 * Q + h] * (o[1] * js);
                if constexpr (D == 3) {
                    const int n = q1 + Q * h;
                    val += C.Gc[q2 * Q + h] * (v[2] * un[n]);
                    acc[n] += C.Gc[q2 * Q + h] * (o[2] * js);
                }
            }
            acc[q] += s ? val : -val;
            cn[q] = o[0] * js;
        }
        all_passes<T, Q, D - 1, true>(acc, C.Ig);
        all_passes<T, Q, D - 1, true>(cn, C.Ig);
#pragma unroll
        for (int m = 0; m < QN; ++m) {
            T0[s][m] = has[s] ? acc[m] : T(0);
            Tn[s][m] = has[s] ? cn[m] : T(0);
        }
    }
#pragma unroll
    for (int m = 0; m < QN; ++m) {
        const int J0 = (m % Q) * S1 + (m / Q) * S2;
#pragma unroll
        for (int j = 0; j < Q; ++j) {
            T v = C.Ed[j] * Tn[0][m] + C.Ed[Q + j] * Tn[1][m];
            if (j == 0) v += T0[0][m];
            if (j == Q - 1) v += T0[1][m];
            ys[J0 + j * SA] = v;
        }
    }
}

template <typename T, int B, int NC, bool VB, int GEO>
__device__ __forceinline__ void cell_terms(const CellArgs<T>& L, int c, const T* __restrict__ va,
                                           const T* __restrict__ vb, T* ys) {
    if constexpr (GEO == GEO_BOX) box_cell_terms<T, B, NC, VB>(L, c, va, vb, ys);
    else if constexpr (GEO == GEO_HYB) blk_cell_terms<T, B, NC, VB, GEO>(L, c, va, vb, ys);
    else map_cell_terms<T, B, NC, VB>(L, c, va, vb, ys);
}
template <typename T, int B, int NC, bool VB, int GEO, int A>
__device__ __forceinline__ void face_terms(const CellArgs<T>& L, int c, const T* __restrict__ va,
                                           const T* __restrict__ vb, T* ys) {
    if constexpr (GEO == GEO_BOX) box_face_terms<T, B, NC, VB, A>(L, c, va, vb, ys);
    else if constexpr (GEO == GEO_HYB) hyb_face_terms<T, B, VB, A>(L, c, va, vb, ys);
    else map_face_terms<T, B, NC, VB, A>(L, c, va, vb, ys);
}

// ---- 3D Q3 cells: four lanes per cell
// A lane per cell would hold 64 values per array and issue 4,000 dependent
// instructions (19 us on a single cell in FP64, more than the launch of a
// whole small level).  Here lane l of a quad holds the 16 values with index l
// along one axis, passes along that axis read the other three lanes through
// DPP, and a wave takes 16 cells.
template <int J>
__device__ __forceinline__ float quad_lane(float v) {
    return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), J * 0x55, 0xf, 0xf, true));
}
template <int J>
__device__ __forceinline__ double quad_lane(double v) {
    const int lo = __builtin_amdgcn_update_dpp(0, __double2loint(v), J * 0x55, 0xf, 0xf, true);
    const int hi = __builtin_amdgcn_update_dpp(0, __double2hiint(v), J * 0x55, 0xf, 0xf, true);
    return __hiloint2double(hi, lo);
}
// sum_j c[j] v(lane j of the quad)
template <typename T>
__device__ __forceinline__ T quad_dot(const T* c, T v) {
    return c[0] * quad_lane<0>(v) + c[1] * quad_lane<1>(v) + c[2] * quad_lane<2>(v) + c[3] * quad_lane<3>(v);
}
template <typename T>
__device__ __forceinline__ T quad_pick(const T* a, int stride, int l) {
    // values, not elements: a choice of elements would become a choice of addresses
    const T v0 = a[0], v1 = a[stride], v2 = a[2 * stride], v3 = a[3 * stride];
    return l == 0 ? v0 : l == 1 ? v1 : l == 2 ? v2 : v3;
}
// row l of a 4 x 4 table, or column l
template <typename T>
__device__ __forceinline__ void quad_row(const T* M, int l, T* c) {
#pragma unroll
    for (int j = 0; j < 4; ++j) c[j] = quad_pick(M + j, 4, l);
}
template <typename T>
__device__ __forceinline__ void quad_col(const T* M, int l, T* c) {
#pragma unroll
    for (int j = 0; j < 4; ++j) c[j] = quad_pick(M + 4 * j, 1, l);
}

template <typename T, bool VB>
__device__ __forceinline__ void cell_terms_quad(const CellArgs<T>& L, int c, int l, const T* __restrict__ va,
                                                const T* __restrict__ vb, T* ys) {
    const MfConst<T>& C = L.mf;
    T u[16], y[16], f2[16], Dk[6], cI[4], cG[4];
    load_cell<T, 16, VB>(va, vb, c * 4 + l, u);
#pragma unroll
    for (int k = 0; k < 6; ++k) Dk[k] = C.D[(size_t)c * 6 + k];
#pragma unroll
    for (int a = 0; a < 3; ++a)
#pragma unroll
        for (int b = a; b < 3; ++b) Dk[pk<3>(a, b)] *= C.vol * C.hinv[a] * C.hinv[b];
    const T mass = C.vol * C.cM, wl = quad_pick(C.gw, 1, l);
    all_passes<T, 4, 2, false>(u, C.Ig);
    quad_row(C.Ig, l, cI);
    quad_row(C.Gc, l, cG);
#pragma unroll
    for (int g = 0; g < 16; ++g) u[g] = quad_dot(cI, u[g]);
#pragma unroll
    for (int g = 0; g < 16; ++g) y[g] = 0;
#pragma unroll
    for (int g = 0; g < 16; ++g) {
        const int g0 = g % 4, g1 = g / 4;
        const T w = C.gw[g0] * C.gw[g1] * wl;
        T gr[3] = {0, 0, quad_dot(cG, u[g])};
#pragma unroll
        for (int h = 0; h < 4; ++h) {
            gr[0] += C.Gc[g0 * 4 + h] * u[h + 4 * g1];
            gr[1] += C.Gc[g1 * 4 + h] * u[g0 + 4 * h];
        }
        T f[3];
#pragma unroll
        for (int a = 0; a < 3; ++a) f[a] = w * (Dk[pk<3>(a, 0)] * gr[0] + Dk[pk<3>(a, 1)] * gr[1] + Dk[pk<3>(a, 2)] * gr[2]);
        y[g] += w * mass * u[g];
#pragma unroll
        for (int h = 0; h < 4; ++h) {
            y[h + 4 * g1] += C.Gc[g0 * 4 + h] * f[0];
            y[g0 + 4 * h] += C.Gc[g1 * 4 + h] * f[1];
        }
        f2[g] = f[2];
    }
    quad_col(C.Ig, l, cI);
    quad_col(C.Gc, l, cG);
#pragma unroll
    for (int g = 0; g < 16; ++g) {
        y[g] += quad_dot(cG, f2[g]);
        y[g] = quad_dot(cI, y[g]);
    }
    all_passes<T, 4, 2, true>(y, C.Ig);
#pragma unroll
    for (int g = 0; g < 16; ++g) ys[l * 16 + g] = y[g];
}

// Both faces normal to axis A; lane l holds the nodes with index l along the
// second tangential axis.
template <typename T, bool VB, int A>
__device__ __forceinline__ void face_terms_quad(const CellArgs<T>& L, int c, int l, const T* __restrict__ va,
                                                const T* __restrict__ vb, T* ys) {
    constexpr int t1 = A == 0 ? 1 : 0, t2 = A == 2 ? 1 : 2;
    constexpr int SA = ipow(4, A), S1 = ipow(4, t1), S2 = ipow(4, t2);
    const MfConst<T>& C = L.mf;
    const int lo = L.lo[(size_t)A * L.n + c], up = L.up[(size_t)A * L.n + c];
    const int nb[2] = {lo >= 0 ? lo : c, up};
    const bool has[2] = {lo >= 0, up != c};
    // value (normal index j, first tangential index m) of a cell at x[at(j, m)]
    auto at = [](int j, int m) { return A == 0 ? j + 4 * m : m + 4 * j; };
    auto load = [&](int cell, T* x) {
        if constexpr (A < 2) {
            load_cell<T, 16, VB>(va, vb, cell * 4 + l, x);
        } else {
#pragma unroll
            for (int j = 0; j < 4; ++j) load_cell<T, 4, VB>(va, vb, cell * 16 + 4 * j + l, x + 4 * j);
        }
    };
    T xk[16], DK[3], daa = C.D[(size_t)c * 6 + pk<3>(A, A)];
    load(c, xk);
#pragma unroll
    for (int k = 0; k < 3; ++k) DK[k] = C.D[(size_t)c * 6 + pk<3>(A, k)] * C.hinv[k];
    T cM[4], cN[4], cT[4];
    quad_row(C.M1, l, cM);
    quad_row(C.N1, l, cN);
    quad_col(C.N1, l, cT);
    T T0[2][4], Tn[2][4];
#pragma unroll
    for (int s = 0; s < 2; ++s) {
        T xn[16], DN[3];
        load(nb[s], xn);
        const T dnn = C.D[(size_t)nb[s] * 6 + pk<3>(A, A)];
#pragma unroll
        for (int k = 0; k < 3; ++k) DN[k] = C.D[(size_t)nb[s] * 6 + pk<3>(A, k)] * C.hinv[k];
        const T ar = has[s] ? C.area[A] : T(0);
        const T hs = (s ? T(-0.5) : T(0.5)) * ar;
        const T sig = C.eta[A] * T(0.5) * (daa + dnn) * ar;
        T q0[4], q1[4], q2[4], jc[4];
#pragma unroll
        for (int m = 0; m < 4; ++m) {
            T dK = 0, dN = 0;
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                dK += C.Ed[s * 4 + j] * xk[at(j, m)];
                dN += C.Ed[(1 - s) * 4 + j] * xn[at(j, m)];
            }
            const T uK = xk[at(3 * s, m)], uN = xn[at(3 * (1 - s), m)], j = uK - uN;
            q0[m] = hs * (DK[A] * dK + DN[A] * dN) + sig * j;
            q1[m] = hs * (DK[t1] * uK + DN[t1] * uN);
            q2[m] = hs * (DK[t2] * uK + DN[t2] * uN);
            jc[m] = hs * j;
        }
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            T v = 0, w = 0, x = 0, z = 0;
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                v += C.M1[i * 4 + j] * q0[j] + C.N1[i * 4 + j] * q1[j];
                w += C.N1[j * 4 + i] * jc[j];
                x += C.M1[i * 4 + j] * q2[j];
                z += C.M1[i * 4 + j] * jc[j];
            }
            v += DK[t1] * w;
            T0[s][i] = quad_dot(cM, v) + quad_dot(cN, x) + DK[t2] * quad_dot(cT, z);
            Tn[s][i] = DK[A] * quad_dot(cM, z);
        }
    }
#pragma unroll
    for (int m = 0; m < 4; ++m)
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            T v = C.Ed[j] * Tn[0][m] + C.Ed[4 + j] * Tn[1][m];
            if (j == 0) v += T0[0][m];
            if (j == 3) v += T0[1][m];
            ys[m * S1 + l * S2 + j * SA] = v;
        }
}

// ---- Q4 squares, a lane per row: two cells per wave, every 1D pass through LDS
// within the wave, so that no barrier separates them.  A lane per cell has 1,200
// multiply-adds to do one after the other, which is all that a level of a few
// hundred cells takes; here a row has about 90, and the face terms run beside
// them: lanes 0 .. 19 of a cell take a node of a face each.  576 boxes, step: FP64
// 6.5 us by cells, 4.8 us here, FP32 5.4, 4.2 us; residual of a pending update 8.5, 4.9 us.
template <typename T, int B, int NC, bool VB>
__device__ __forceinline__ void box_rows(const CellArgs<T>& L, int cell0, const T* __restrict__ va,
                                         const T* __restrict__ vb, T* sh) {
    constexpr int Q = 5, CW = 64 / B, NF = 4 * Q, NTAB = 4 * Q * Q + 3 * Q;
    static_assert(B == Q * Q && Q == kMfMaxQ && NC == CW * kWG / 64, "whole tables, two cells per wave");
    // the 1D tables lie one after the other at the start of MfConst
    static_assert(offsetof(MfConst<T>, gw) == (4 * Q * Q + 2 * Q) * sizeof(T), "order of the tables");
    struct Cell {
        T p[3][B], fq[3][NF], ft[2][NF];
    };
    struct Wave {
        T tab[NTAB];
        Cell c[CW];
    };
    __shared__ Wave work[kWG / 64];
    const int lane = (int)threadIdx.x & 63, w = (int)threadIdx.x >> 6;
    const int lc = lane / B, i = lane - lc * B;
    if (lc >= CW) return;
    const MfConst<T>& C = L.mf;
    const T* tabs = reinterpret_cast<const T*>(&C);
    Wave& W = work[w];
    Cell& S = W.c[lc];
    const T *Ig = W.tab, *Gc = W.tab + B, *M1 = W.tab + 2 * B, *N1 = W.tab + 3 * B, *Ed = W.tab + 4 * B,
            *gw = W.tab + 4 * B + 2 * Q;
    const int c = min(cell0 + w * CW + lc, L.n - 1);
    const int ix = i % Q, iy = i / Q;
    // face item: node m of the face on side s of axis A
    const bool face = i < NF;
    const int f = face ? i / Q : 0, m = ix, A = f >> 1, s = f & 1;
    const int nv = (s ? L.up : L.lo)[(size_t)A * L.n + c], nb = nv >= 0 ? nv : c;
    auto value = [&](int cell, int k) {
        const size_t t = (size_t)cell * B + k;
        return VB ? va[t] + vb[t] : va[t];
    };
    const T u = value(c, i);
    T xn[Q], tv[(NTAB + CW * B - 1) / (CW * B)];
#pragma unroll
    for (int j = 0; j < Q; ++j) xn[j] = value(nb, A ? m + Q * j : j + Q * m);
#pragma unroll
    for (int k = 0; k < (NTAB + CW * B - 1) / (CW * B); ++k) tv[k] = tabs[min(lane + k * CW * B, NTAB - 1)];
    const T Dxx = C.D[(size_t)c * 3], Dxy = C.D[(size_t)c * 3 + 1], Dyy = C.D[(size_t)c * 3 + 2];
    const T nxx = C.D[(size_t)nb * 3], nxy = C.D[(size_t)nb * 3 + 1], nyy = C.D[(size_t)nb * 3 + 2];
#pragma unroll
    for (int k = 0; k < (NTAB + CW * B - 1) / (CW * B); ++k)
        if (lane + k * CW * B < NTAB) W.tab[lane + k * CW * B] = tv[k];
    S.p[0][i] = u;
    wave_lds_fence();
    // x pass; face nodes: traces and normal derivatives of both sides
    const T hA = A ? C.hinv[1] : C.hinv[0], hT = A ? C.hinv[0] : C.hinv[1];
    const T kA = (A ? Dyy : Dxx) * hA, kT = Dxy * hT;
    T a = 0;
#pragma unroll
    for (int j = 0; j < Q; ++j) a += Ig[ix * Q + j] * S.p[0][iy * Q + j];
    S.p[1][i] = a;
    if (face) {
        T dK = 0, dN = 0;
#pragma unroll
        for (int j = 0; j < Q; ++j) {
            dK += Ed[s * Q + j] * S.p[0][A ? m + Q * j : j + Q * m];
            dN += Ed[(1 - s) * Q + j] * xn[j];
        }
        const T uK = S.p[0][A ? m + Q * s * (Q - 1) : s * (Q - 1) + Q * m], uN = s ? xn[0] : xn[Q - 1];
        const T ar = (s ? nv != c : nv >= 0) ? (A ? C.area[1] : C.area[0]) : T(0);
        const T hs = (s ? T(-0.5) : T(0.5)) * ar;
        const T sig = (A ? C.eta[1] : C.eta[0]) * T(0.5) * (A ? Dyy + nyy : Dxx + nxx) * ar;
        const T j = uK - uN;
        S.fq[0][i] = hs * (kA * dK + (A ? nyy : nxx) * hA * dN) + sig * j;
        S.fq[1][i] = hs * (kT * uK + nxy * hT * uN);
        S.fq[2][i] = hs * j;
    }
    wave_lds_fence();
    // y pass; tangential integrals of the faces
    T g = 0;
#pragma unroll
    for (int j = 0; j < Q; ++j) g += Ig[iy * Q + j] * S.p[1][j * Q + ix];
    S.p[2][i] = g;
    if (face) {
        T v = 0, n = 0, t = 0;
#pragma unroll
        for (int j = 0; j < Q; ++j) {
            const T q0 = S.fq[0][f * Q + j], q1 = S.fq[1][f * Q + j], jc = S.fq[2][f * Q + j];
            v += M1[m * Q + j] * q0 + N1[m * Q + j] * q1;
            t += N1[j * Q + m] * jc;
            n += M1[m * Q + j] * jc;
        }
        S.ft[0][i] = v + kT * t;
        S.ft[1][i] = kA * n;
    }
    wave_lds_fence();
    // gradient and weighted fluxes at the Gauss point
    T gx = 0, gy = 0;
#pragma unroll
    for (int h = 0; h < Q; ++h) {
        gx += Gc[ix * Q + h] * S.p[2][iy * Q + h];
        gy += Gc[iy * Q + h] * S.p[2][h * Q + ix];
    }
    const T wq = gw[ix] * gw[iy] * C.vol, h0 = C.hinv[0], h1 = C.hinv[1];
    S.p[0][i] = wq * (Dxx * h0 * h0 * gx + Dxy * h0 * h1 * gy);
    S.p[1][i] = wq * (Dxy * h0 * h1 * gx + Dyy * h1 * h1 * gy);
    wave_lds_fence();
    T y = wq * C.cM * g;
#pragma unroll
    for (int h = 0; h < Q; ++h) y += Gc[h * Q + ix] * S.p[0][iy * Q + h] + Gc[h * Q + iy] * S.p[1][h * Q + ix];
    S.p[2][i] = y;
    wave_lds_fence();
    // transposed passes, and the faces' terms of the row's test function
    T b = 0;
#pragma unroll
    for (int h = 0; h < Q; ++h) b += Ig[h * Q + ix] * S.p[2][iy * Q + h];
    S.p[0][i] = b;
    wave_lds_fence();
    T r = 0;
#pragma unroll
    for (int h = 0; h < Q; ++h) r += Ig[h * Q + iy] * S.p[0][h * Q + ix];
#pragma unroll
    for (int q = 0; q < 2; ++q) {                        // axis
        const int n = q ? iy : ix, t = q ? ix : iy;      // normal and tangential index
        r += Ed[n] * S.ft[1][2 * q * Q + t] + Ed[Q + n] * S.ft[1][(2 * q + 1) * Q + t];
        if (n == 0) r += S.ft[0][2 * q * Q + t];
        if (n == Q - 1) r += S.ft[0][(2 * q + 1) * Q + t];
    }
    sh[(w * CW + lc) * CellTile<T, B, NC, GEO_BOXR>::SB + i] = r;
}

// Evaluates the workgroup's shares: sh[w * NC * SB + cell * SB + row].  Lanes past
// the last cell evaluate cell n - 1 and their rows are not read.  The caller
// synchronises before it reads the shares.
template <typename T, int B, int NC, bool VB, int GEO>
__device__ __forceinline__ void cell_product(const CellArgs<T>& L, int cell0, const T* __restrict__ va,
                                             const T* __restrict__ vb, T* sh) {
    using Ct = CellTile<T, B, NC, GEO>;
    static_assert(NC <= (B == 64 ? 16 : 64), "cells of a workgroup do not fit a wave");
    const int lane = (int)threadIdx.x & 63, w = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
    if constexpr (GEO == GEO_ROW) {
        static_assert(B == 64 && NC == 1, "a workgroup per cell of 64 rows");
        sh[w * 64 + lane] = row_terms<T, VB>(L, cell0, w, lane, va, vb);
        return;
    } else if constexpr (GEO == GEO_BOXR) {
        box_rows<T, B, NC, VB>(L, cell0, va, vb, sh);
        return;
    } else if constexpr (B == 64) {
        static_assert(GEO == GEO_BOX, "3D Q3 cells: boxes or agglomerates by rows");
        if (lane >= 4 * NC) return;   // whole quads
        const int c = min(cell0 + lane / 4, L.n - 1), l = lane & 3;
        T* ys = sh + (w * Ct::NC + lane / 4) * Ct::SB;
        if (w == 0) cell_terms_quad<T, VB>(L, c, l, va, vb, ys);
        else if (w == 1) face_terms_quad<T, VB, 0>(L, c, l, va, vb, ys);
        else if (w == 2) face_terms_quad<T, VB, 1>(L, c, l, va, vb, ys);
        else face_terms_quad<T, VB, 2>(L, c, l, va, vb, ys);
        return;
    }
    if (lane >= NC) return;
    const int c = min(cell0 + lane, L.n - 1);
    T* ys = sh + (w * Ct::NC + lane) * Ct::SB;
    if constexpr (GEO == GEO_BLK || GEO == GEO_BLD) {
        if (w == 0) blk_cell_terms<T, B, NC, VB, GEO>(L, c, va, vb, ys);
        else if (w == 1) blk_face_terms<T, B, VB, GEO, 0, 0>(L, c, va, vb, ys);
        else if (w == 2) blk_face_terms<T, B, VB, GEO, 0, 1>(L, c, va, vb, ys);
        else if (w == 3) blk_face_terms<T, B, VB, GEO, 1, 0>(L, c, va, vb, ys);
        else if (Ct::D == 2 || w == 4) blk_face_terms<T, B, VB, GEO, 1, 1>(L, c, va, vb, ys);
        else if constexpr (Ct::D == 3) {
            if (w == 5) blk_face_terms<T, B, VB, GEO, 2, 0>(L, c, va, vb, ys);
            else blk_face_terms<T, B, VB, GEO, 2, 1>(L, c, va, vb, ys);
        }
        return;
    }
    if (w == 0) cell_terms<T, B, NC, VB, GEO>(L, c, va, vb, ys);
    else if (w == 1) face_terms<T, B, NC, VB, GEO, 0>(L, c, va, vb, ys);
    else if (Ct::D == 2 || w == 2) face_terms<T, B, NC, VB, GEO, 1>(L, c, va, vb, ys);
    else if constexpr (Ct::D == 3) face_terms<T, B, NC, VB, GEO, 2>(L, c, va, vb, ys);
}
// row k = cell * SB + i of the product
template <typename T, int B, int NC, int GEO>
__device__ __forceinline__ T cell_row(const T* sh, int k) {
    using Ct = CellTile<T, B, NC, GEO>;
    T a = sh[k];
#pragma unroll
    for (int w = 1; w < Ct::NS; ++w) a += sh[w * Ct::NC * Ct::SB + k];
    return a;
}

#define DGMG_CELL_GROUP(T, B)                                                        \
    using Ct = CellTile<T, B, NC, GEO>;                                                       \
    __shared__ T sh[Ct::NS * Ct::NC * Ct::SB];                                       \
    const int cell0 = xcd_tile(blockIdx.x, gridDim.x) * Ct::NC;                      \
    const int rows = min(Ct::NC, L.n - cell0) * B;                                   \
    const size_t t0 = (size_t)cell0 * B;
// The epilogue takes a row per lane, all U rows of a thread at once, whose
// vector operands are requested together before the barrier: a loop that
// loaded row by row cost a memory latency per row, 7 of them on 3D Q2 cells.
template <int B, int NC, int GEO>
constexpr int cell_rows() {
    return (NC * B + cell_threads<B, GEO>() - 1) / cell_threads<B, GEO>();
}
#define DGMG_CELL_ROWS(B)                                                            \
    constexpr int U = cell_rows<B, NC, GEO>();                                       \
    static_assert(U <= 9, "rows of a thread held in registers");                     \
    auto row = [&](int u) { return (int)threadIdx.x + u * Ct::NT; };                 \
    auto at = [&](int e) { return e + (Ct::SB - B) * (e / B); };   // LDS index of row e

// The cell-block term's columns of the thread's U rows (row-major symmetric
// blocks: the lanes of a cell read consecutive words of a row), requested before
// the barrier where they fit in registers.  Boxes of 64 DoFs, 512 cells, step: FP64
// 8.7 -> 8.1 us, FP32 6.3 -> 6.0; boxes of 27 (7.5 -> 7.7 us) and mapped cells (25 DoFs FP64
// 7.5 -> 8.6) were slower with it.
template <typename T, int B, int NC, int GEO>
constexpr bool block_columns_early() {
    return (GEO == GEO_BOXR || (GEO == GEO_BOX && B == 64)) && cell_rows<B, NC, GEO>() * B * sizeof(T) <= 640;
}
template <typename T, int B, int NT, int U>
__device__ __forceinline__ void load_block_columns(const T* __restrict__ bj, int cell0, int rows, T (*dk)[B]) {
#pragma unroll
    for (int u = 0; u < U; ++u) {
        const int e = min((int)threadIdx.x + u * NT, rows - 1), lc = e / B;
        const T* Dc = bj + (size_t)(cell0 + lc) * B * B + (e - lc * B);
#pragma unroll
        for (int i = 0; i < B; ++i) dk[u][i] = Dc[(size_t)i * B];
    }
}

// y = A va; optional partial of dot(w, y).
template <typename T, int B, int NC, int GEO>
__global__ __launch_bounds__((cell_threads<B, GEO>())) void k_apply_cell(CellArgs<T> L, const T* __restrict__ va,
                                                                  T* __restrict__ y, const T* __restrict__ w,
                                                                  double* __restrict__ partial) {
    DGMG_CELL_GROUP(T, B)
    DGMG_CELL_ROWS(B)
    cell_product<T, B, NC, false, GEO>(L, cell0, va, nullptr, sh);
    T wv[U];
#pragma unroll
    for (int u = 0; u < U; ++u) wv[u] = w ? w[t0 + min(row(u), rows - 1)] : T(0);
    __syncthreads();
    double contrib = 0.0;
#pragma unroll
    for (int u = 0; u < U; ++u) {
        const int e = row(u);
        if (e >= rows) continue;
        const T a = cell_row<T, B, NC, GEO>(sh, at(e));
        y[t0 + e] = a;
        contrib += (double)wv[u] * (double)a;
    }
    if (partial) wg_sum_store<Ct::NT>(contrib, partial);
}

// Residual with the epilogues of k_residual.
template <typename T, int B, int NC, int GEO, bool VB, bool BJ>
__global__ __launch_bounds__((cell_threads<B, GEO>())) void k_residual_cell(
    CellArgs<T> L, const T* __restrict__ va, const T* __restrict__ vb, const T* __restrict__ rhs, T* __restrict__ r,
    T* __restrict__ d, T c1, T* __restrict__ xout, double* __restrict__ partial, const T* __restrict__ P,
    T* __restrict__ rp, const int32_t* __restrict__ ptype, const T* __restrict__ bj) {
    DGMG_CELL_GROUP(T, B)
    DGMG_CELL_ROWS(B)
    cell_product<T, B, NC, VB, GEO>(L, cell0, va, vb, sh);
    T bv[U], di[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
        const size_t t = t0 + min(row(u), rows - 1);
        bv[u] = rhs[t];
        di[u] = d && !BJ ? L.dinv[t] : T(0);
    }
    constexpr bool EARLY = BJ && block_columns_early<T, B, NC, GEO>();
    T dk[EARLY ? U : 1][B];
    if constexpr (EARLY) {
        if (d) load_block_columns<T, B, Ct::NT, U>(bj, cell0, rows, dk);
    }
    __syncthreads();
    double contrib = 0.0;
#pragma unroll
    for (int u = 0; u < U; ++u) {
        const int e = row(u);
        if (e >= rows) continue;
        const size_t t = t0 + e;
        const T rr = bv[u] - cell_row<T, B, NC, GEO>(sh, at(e));
        if (r) r[t] = rr;
        if (!BJ && d) d[t] = di[u] * rr * c1;
        if (xout) xout[t] = VB ? va[t] + vb[t] : va[t];
        contrib += (double)rr * (double)rr;
        sh[at(e)] = rr;                               // a row's first share is read by its own thread only
    }
    if ((BJ && d) || P) {
        __syncthreads();
        if constexpr (EARLY) {
            if (d) {
#pragma unroll
                for (int u = 0; u < U; ++u) {
                    const int e = row(u);
                    if (e >= rows) continue;
                    const T* rc = sh + e / B * Ct::SB;
                    T z = 0;
#pragma unroll
                    for (int i = 0; i < B; ++i) z += dk[u][i] * rc[i];
                    d[t0 + e] = c1 * z;
                }
            }
            if (!P) {
                if (partial) wg_sum_store<Ct::NT>(contrib, partial);
                return;
            }
        }
        // two rows of a thread at a time, their loads requested together
        for (int e0 = threadIdx.x; e0 < rows; e0 += 2 * Ct::NT) {
            T z[2] = {0, 0}, s[2] = {0, 0};
#pragma unroll
            for (int u = 0; u < 2; ++u) {
                const int e = min(e0 + u * Ct::NT, rows - 1), lc = e / B, j = e - lc * B, cell = cell0 + lc;
                const T* rc = sh + lc * Ct::SB;
                if constexpr (BJ && !EARLY) {
                    if (d) {
                        const T* Dc = bj + (size_t)cell * B * B + j;
#pragma unroll
                        for (int i = 0; i < B; ++i) z[u] += Dc[(size_t)i * B] * rc[i];
                    }
                }
                if (P) {
                    // column j of P_cell: a block of the type table or of the
                    // tile-interleaved restriction layout
                    constexpr int TC = Tile<T, B>::TC, TR = Tile<T, B>::TR;
                    const int ht = cell / TC, hl = cell - ht * TC;
                    const T* Pc = ptype ? P + (size_t)ptype[cell] * B * B + j : P + (size_t)ht * B * TR + hl * B + j;
                    const int ks = ptype ? B : TR;
#pragma unroll
                    for (int i = 0; i < B; ++i) s[u] += Pc[i * ks] * rc[i];
                }
            }
#pragma unroll
            for (int u = 0; u < 2; ++u) {
                const int e = e0 + u * Ct::NT;
                if (e >= rows) continue;
                if (BJ && !EARLY && d) d[t0 + e] = c1 * z[u];
                if (P) rp[t0 + e] = s[u];
            }
        }
    }
    if (partial) wg_sum_store<Ct::NT>(contrib, partial);
}

// One inner Chebyshev step, as k_cheb_step.
template <typename T, int B, int NC, int GEO, bool BJ>
__global__ __launch_bounds__((cell_threads<B, GEO>())) void k_cheb_step_cell(CellArgs<T> L, const T* __restrict__ d,
                                                                      T* __restrict__ x, T* __restrict__ r,
                                                                      T* __restrict__ dn, T cd, T cr, int assign,
                                                                      int last, const T* __restrict__ bj) {
    DGMG_CELL_GROUP(T, B)
    DGMG_CELL_ROWS(B)
    cell_product<T, B, NC, false, GEO>(L, cell0, d, nullptr, sh);
    T rv[U], dv[U], xv[U], di[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
        const size_t t = t0 + min(row(u), rows - 1);   // padded rows reread the last one
        rv[u] = r[t];
        dv[u] = d[t];
        xv[u] = assign ? T(0) : x[t];
        di[u] = BJ ? T(0) : L.dinv[t];
    }
    constexpr bool EARLY = BJ && block_columns_early<T, B, NC, GEO>();
    T dk[EARLY ? U : 1][B];
    if constexpr (EARLY) load_block_columns<T, B, Ct::NT, U>(bj, cell0, rows, dk);
    __syncthreads();
    if constexpr (BJ) {
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int e = row(u);
            if (e >= rows) continue;
            const T rr = rv[u] - cell_row<T, B, NC, GEO>(sh, at(e));
            if (!last) r[t0 + e] = rr;
            sh[at(e)] = rr;                           // a row's first share is read by its own thread only
        }
        __syncthreads();
    }
#pragma unroll
    for (int u = 0; u < U; ++u) {
        const int e = row(u);
        if (e >= rows) continue;
        const size_t t = t0 + e;
        T z;
        if constexpr (BJ) {
            const int lc = e / B;
            const T* Dc = bj + (size_t)(cell0 + lc) * B * B + (e - lc * B);
            const T* rc = sh + lc * Ct::SB;
            z = 0;
#pragma unroll
            for (int i = 0; i < B; ++i) z += (EARLY ? dk[EARLY ? u : 0][i] : Dc[(size_t)i * B]) * rc[i];
        } else {
            const T rr = rv[u] - cell_row<T, B, NC, GEO>(sh, at(e));
            if (!last) r[t] = rr;
            z = di[u] * rr;
        }
        const T x1 = assign ? dv[u] : xv[u] + dv[u];
        const T dnew = cd * dv[u] + cr * z;
        x[t] = last ? x1 + dnew : x1;
        if (!last) dn[t] = dnew;
    }
}

// Load vector of the step (k_rhs) on boxes and mapped cells: the mass block is
// evaluated at the Gauss points, M f = I^T (w (I f)), instead of read (b^2
// values per cell: 1.5 GB on the 64^3 Q2 cube).  The workgroup forms f row by
// row, its first wave takes a cell per lane, and the rows are written
// together.  Step of 64^3 Q2: 349 us, 79 us here.
template <int B, int GEO>
__global__ __launch_bounds__(256) void k_rhs_cell(CellArgs<double> L, int bdf, double chi, double cU, double inv_cM,
                                                  const double* U, const double* Up, const double* __restrict__ iapp,
                                                  const double* __restrict__ g, double* __restrict__ b, double* xout) {
    using Ct = CellTile<double, B, 64, GEO>;
    constexpr int D = Ct::D, Q = Ct::Q, R = (64 * B + 255) / 256;
    __shared__ double sh[64 * Ct::SB];
    const int cell0 = xcd_tile(blockIdx.x, gridDim.x) * 64;
    const int rows = min(64, L.n - cell0) * B;
    const size_t t0 = (size_t)cell0 * B;
    auto at = [&](int e) { return e + (Ct::SB - B) * (e / B); };
    double u[R];
#pragma unroll
    for (int k = 0; k < R; ++k) {
        const int e = min((int)threadIdx.x + k * 256, rows - 1);
        u[k] = U[t0 + e];
        const double hist = bdf == 2 ? 4.0 * u[k] - Up[t0 + e] : u[k];
        const double f = cU * hist + (iapp ? iapp[t0 + e] : 0.0) - chi * g[t0 + e];
        if ((int)threadIdx.x + k * 256 < rows) sh[at(e)] = f;
    }
    __syncthreads();
    if (threadIdx.x < 64 && (int)threadIdx.x * B < rows) {
        const MfConst<double>& C = L.mf;
        double* fc = sh + threadIdx.x * Ct::SB;
        double v[B];
#pragma unroll
        for (int i = 0; i < B; ++i) v[i] = fc[i];
        if constexpr (GEO == GEO_BOX) {
            line_pass<double, Q, D, 0, false>(v, C.M1);
            line_pass<double, Q, D, 1, false>(v, C.M1);
            if constexpr (D == 3) line_pass<double, Q, D, 2, false>(v, C.M1);
#pragma unroll
            for (int i = 0; i < B; ++i) v[i] *= C.vol;
        } else {
            constexpr int NE = npack<D>() + 1;             // the last entry of a point is cM w
            all_passes<double, Q, D, false>(v, C.Ig);
            const double* K = cell_data<double, B, GEO>(L, cell0 + (int)threadIdx.x, 0);
#pragma unroll
            for (int q = 0; q < B; ++q) {
                const int e = q * NE + NE - 1;
                v[q] *= K[(size_t)(e / 2) * 128 + e % 2] * inv_cM;
            }
            all_passes<double, Q, D, true>(v, C.Ig);
        }
#pragma unroll
        for (int i = 0; i < B; ++i) fc[i] = v[i];
    }
    __syncthreads();
#pragma unroll
    for (int k = 0; k < R; ++k) {
        const int e = (int)threadIdx.x + k * 256;
        if (e >= rows) continue;
        b[t0 + e] = sh[at(e)];
        if (xout) xout[t0 + e] = u[k];
    }
}

}  // namespace dgmg
