// Device helpers shared by the kernel files.
#pragma once

#include <algorithm>

#include "nlth_impl.hpp"

namespace nlth {

// ---------------------------------------------------------------------------
// constants
// ---------------------------------------------------------------------------

// 4-point degree-2 rule: barycentric (a, b, b, b) and permutations, weight V/4.
#define QA_ 0.5854101966249685
#define QB_ 0.1381966011250105

// Consistent mass of the 10-node tet divided by its volume: the classical
// pattern /420 (corner diagonal 6, corner-corner 1, corner and an edge through
// it -4, corner and the opposite-side edge -6, edge diagonal 32, edges sharing
// a vertex 16, opposite edges 8).
__host__ __device__ constexpr double mass_ref(int a, int b)
{
    // edges as vertex pairs
    constexpr int E[6][2] = {{0, 1}, {1, 2}, {2, 0}, {0, 3}, {1, 3}, {2, 3}};
    if (a < 4 && b < 4) return (a == b ? 6.0 : 1.0) / 420.0;
    if (a < 4 || b < 4) {
        int c = a < 4 ? a : b;
        int e = (a < 4 ? b : a) - 4;
        return (E[e][0] == c || E[e][1] == c ? -4.0 : -6.0) / 420.0;
    }
    if (a == b) return 32.0 / 420.0;
    int ea = a - 4, eb = b - 4;
    bool share = E[ea][0] == E[eb][0] || E[ea][0] == E[eb][1] || E[ea][1] == E[eb][0] ||
                 E[ea][1] == E[eb][1];
    return (share ? 16.0 : 8.0) / 420.0;
}

// index of (r, c) in the row-by-row upper triangle of a symmetric 6x6
__host__ __device__ constexpr int sym6(int r, int c)
{
    return r <= c ? r * 6 - r * (r - 1) / 2 + (c - r) : c * 6 - c * (c - 1) / 2 + (r - c);
}

template <typename T> __device__ __forceinline__ const T* geo_of(const DevMesh& M);
template <> __device__ __forceinline__ const double* geo_of<double>(const DevMesh& M) { return M.geo64; }
template <> __device__ __forceinline__ const float* geo_of<float>(const DevMesh& M) { return M.geo32; }

__device__ __forceinline__ double matv(const double* mat, int l, int f, int MB, int m)
{
    return mat[((long)l * MAT_N + f) * MB + m];
}

__device__ __forceinline__ uint32_t f2bf(double x)
{
    // round to nearest even on the FP32 bit pattern
    const uint32_t u = __float_as_uint((float)x);
    return (u + 0x7FFFu + ((u >> 16) & 1u)) >> 16;
}
__device__ __forceinline__ float bf2f(uint32_t b) { return __uint_as_float(b << 16); }


// element i of an array at a wavefront-uniform base: the byte offset is
// formed in 32 bits, so the load takes the scalar-base + 32-bit vector-offset
// form (no per-lane 64-bit address arithmetic).  i * sizeof(T) < 2^32.
template <typename T>
__device__ __forceinline__ T ld_u(const T* base, uint32_t i)
{
    return *reinterpret_cast<const T*>(reinterpret_cast<const char*>(base) + i * (uint32_t)sizeof(T));
}

template <typename T>
__device__ __forceinline__ T ld_u_nt(const T* base, uint32_t i)
{
    return __builtin_nontemporal_load(
        reinterpret_cast<const T*>(reinterpret_cast<const char*>(base) + i * (uint32_t)sizeof(T)));
}

// dashpot force at boundary node i (index into the boundary-node lists) for
// member m: coef * sum over its faces of rho (Vp n n^T + Vs (I - n n^T)) int N_a N_b dA x_b,
// plus, with vI, the incident-wave force 2 C_base v_I on base faces.  Only
// every parts-th face of the node, from the part-th on (lanes share a node).
// x(i): the nodal value at index i.
template <typename XF>
__device__ __forceinline__ void dashpot_at(const DevMesh& M, int MB, int m, int i, const double* __restrict__ mat,
                                           double coef, XF x, const double* __restrict__ vI,
                                           double acc[3], int part = 0, int parts = 1)
{
    for (int q = M.bn_ptr[i] + part; q < M.bn_ptr[i + 1]; q += parts) {
        const int f = M.bn_face[q], a = M.bn_loc[q];
        const int l = M.f_layer[f];
        // all loads of a face issued together: a loop that waits for each node
        // in turn is a chain of twelve round trips
        long nb[6];
        double Mab[6], xb[6][3];
#pragma unroll
        for (int b = 0; b < 6; ++b) {
            nb[b] = M.f_node[6 * (long)f + b];
            Mab[b] = M.f_M[36 * (long)f + 6 * a + b];
        }
        const double* np = M.f_n + 3 * (long)f;
        const double nv[3] = {np[0], np[1], np[2]};
        const double rho = matv(mat, l, MAT_RHO, MB, m);
        const double vs = matv(mat, l, MAT_VS, MB, m);
        const double vp = matv(mat, l, MAT_VP, MB, m);
#pragma unroll
        for (int b = 0; b < 6; ++b)
#pragma unroll
            for (int c = 0; c < 3; ++c) xb[b][c] = (double)x((size_t)((nb[b] * 3 + c) * MB + m));
        double X[3] = {0, 0, 0}, rs = 0;
#pragma unroll
        for (int b = 0; b < 6; ++b) {
            rs += Mab[b];
#pragma unroll
            for (int c = 0; c < 3; ++c) X[c] += Mab[b] * xb[b][c];
        }
        double nx = nv[0] * X[0] + nv[1] * X[1] + nv[2] * X[2];
        for (int c = 0; c < 3; ++c) acc[c] += coef * rho * (vs * X[c] + (vp - vs) * nx * nv[c]);
        if (vI && M.f_kind[f] == 0) {  // incident wave: 2 C_base v_I
            double V[3] = {vI[0 * MB + m], vI[1 * MB + m], vI[2 * MB + m]};
            double nV = nv[0] * V[0] + nv[1] * V[1] + nv[2] * V[2];
            for (int c = 0; c < 3; ++c) acc[c] += 2.0 * rs * rho * (vs * V[c] + (vp - vs) * nV * nv[c]);
        }
    }
}

// ---------------------------------------------------------------------------
// element-by-element operator (Eq. 1 left-hand side, Eq. 2 stiffness)
// ---------------------------------------------------------------------------
//
// Per (element, member): gather the 10 nodal displacements, add the mass
// term (consistent P2 mass applied through corner and edge sums), then the
// stiffness term of Eq. 2 with the 4-point rule.  Straight-sided tets make the
// shape-function gradients linear in the barycentrics, so the strain at the
// four points is a combination of four per-element 6-vectors E_k and the
// point forces fold back onto the nodes the same way; D_j is streamed once.

// Voigt symmetric part of u (x) g  (F_cd = u_c g_d, engineering shear)
template <typename T>
__device__ __forceinline__ void vsym_acc(const T u[3], const T g[3], T o[6])
{
    // each component a chain of fused multiply-adds into the accumulator
    o[0] = fma(u[0], g[0], o[0]);
    o[1] = fma(u[1], g[1], o[1]);
    o[2] = fma(u[2], g[2], o[2]);
    o[3] = fma(u[0], g[1], fma(u[1], g[0], o[3]));
    o[4] = fma(u[1], g[2], fma(u[2], g[1], o[4]));
    o[5] = fma(u[2], g[0], fma(u[0], g[2], o[5]));
}

// f += s * sigma . g  (sigma in Voigt order xx, yy, zz, xy, yz, zx)
template <typename T>
__device__ __forceinline__ void tdot_acc(const T sg[6], const T g[3], T s, T f[3])
{
    f[0] += s * (sg[0] * g[0] + sg[3] * g[1] + sg[5] * g[2]);
    f[1] += s * (sg[3] * g[0] + sg[1] * g[1] + sg[4] * g[2]);
    f[2] += s * (sg[5] * g[0] + sg[4] * g[1] + sg[2] * g[2]);
}

// f += sigma . g as chains of fused multiply-adds into f
template <typename T>
__device__ __forceinline__ void tdot_add(const T sg[6], const T g[3], T f[3])
{
    f[0] = fma(sg[0], g[0], fma(sg[3], g[1], fma(sg[5], g[2], f[0])));
    f[1] = fma(sg[3], g[0], fma(sg[1], g[1], fma(sg[4], g[2], f[1])));
    f[2] = fma(sg[5], g[0], fma(sg[4], g[1], fma(sg[2], g[2], f[2])));
}

// index of D(e, j, k) for member m: elements in blocks of EB so that a
// wavefront's lanes (EB elements x MB members) read contiguous memory
__device__ __forceinline__ long d_index(long e, int j, int k, int MB, int EB, int m)
{
    return (((e / EB) * 84 + j * 21 + k) * EB + e % EB) * (long)MB + m;
}

// bfloat16 storage of D for the inner operator: pairs of consecutive upper-
// triangle entries (k = 2q, 2q+1; k = 21 is padding) packed in one 32-bit word
__device__ __forceinline__ long d16_index(long e, int j, int q, int MB, int EB, int m)
{
    return (((e / EB) * 44 + j * 11 + q) * EB + e % EB) * (long)MB + m;
}
// element-mean D of the inner operator in bfloat16 pairs: 11 words per element
__device__ __forceinline__ long d16m_index(long e, int q, int MB, int EB, int m)
{
    return (((e / EB) * 11 + q) * EB + e % EB) * (long)MB + m;
}
constexpr int kEdgeOpp[6] = {5, 3, 4, 1, 2, 0};  // edge opposite each edge

// scales of the element's mass and stiffness terms (and, for the right-hand
// side, of v in the mass term) from its density, volume and damping; the
// quotients by dt are formed on the host
template <typename T, int MODE>
__device__ __forceinline__ void op_scales(const StepConst& sc, double rho, double vol, double he, T& sm, T& sk, T& cv)
{
    if (MODE == OP_A) {
        sm = (T)(rho * vol * (sc.m4 + sc.a2 * he));
        sk = (T)(1.0 + sc.b2 * he);
    } else if (MODE == OP_K) {
        sm = 0; sk = 1;
    } else if (MODE == OP_M) {
        sm = (T)(rho * vol); sk = 0;
    } else {  // RHS: M (a + (4/dt + alpha) v) + beta K v
        sm = (T)(rho * vol);
        sk = (T)(sc.bhat * he);
        cv = (T)(sc.c4 + sc.ahat * he);
    }
}

// Forces of one element-member: the 30 nodal values of the operator of MODE
// applied to x(n, c, 0) (and x(n, c, 1) for the right-hand side), to f.  Dp: the
// element's D in the storage DK: 0, T itself, entry (j, k) at Dp[(j * 21 + k) * rs + m];
// 1, bfloat16 pairs, word (j, q) at Dp[(j * 11 + q) * rs + m]; 2, T in a row of 84;
// 4, one D for the element in bfloat16 pairs, word q at Dp[q * rs + m].
template <typename T, int DK, int MODE, class XF>
__device__ __forceinline__ void element_forces(const T gL[4][3], T vol, T sm, T sk, T cv, const void* __restrict__ Dp,
                                               uint32_t rs, uint32_t m, XF x, T f[10][3])
{
    T xk[10][3];
    // ---- mass: consistent P2 mass applied through corner/edge sums; with
    // the scale folded into the coefficients each node's force is a short
    // chain of fused multiply-adds on the corner and edge sums
    const T s420 = sm * (T)(1.0 / 420.0);
    const T c2 = s420 * (T)2, c5 = s420 * (T)5, c6 = s420 * (T)6, c8 = s420 * (T)8, c16 = s420 * (T)16;
#pragma unroll
    for (int c = 0; c < 3; ++c) {
        T xm[10];
#pragma unroll
        for (int n = 0; n < 10; ++n) {
            const T v1 = x(n, c, 0);
            xk[n][c] = v1;
            xm[n] = (MODE == OP_RHS) ? x(n, c, 1) + cv * v1 : v1;
        }
        if (MODE == OP_K) {
#pragma unroll
            for (int n = 0; n < 10; ++n) f[n][c] = 0;
        } else {
            constexpr int E[6][2] = {{0, 1}, {1, 2}, {2, 0}, {0, 3}, {1, 3}, {2, 3}};
            const T Sc = xm[0] + xm[1] + xm[2] + xm[3];
            const T Se = xm[4] + xm[5] + xm[6] + xm[7] + xm[8] + xm[9];
            // corner i: (5 x_i + Sc + 2 A_i - 6 Se) / 420, A_i = the edges at i;
            // edge q (a, b): (2 (x_a + x_b) - 6 Sc + 16 x_q + 16 Se - 8 x_opp) / 420
            const T bc = fma(-c6, Se, s420 * Sc);
            const T be = fma(c16, Se, -c6 * Sc);
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                T A = 0;
#pragma unroll
                for (int q = 0; q < 6; ++q)
                    if (E[q][0] == i || E[q][1] == i) A += xm[4 + q];
                f[i][c] = fma(c5, xm[i], fma(c2, A, bc));
            }
#pragma unroll
            for (int q = 0; q < 6; ++q)
                f[4 + q][c] = fma(c2, xm[E[q][0]] + xm[E[q][1]],
                                  fma(c16, xm[4 + q], fma(-c8, xm[4 + kEdgeOpp[q]], be)));
        }
    }
    // ---- stiffness (Eq. 2)
    if (MODE != OP_M && sk != (T)0) {
        constexpr int E[6][2] = {{0, 1}, {1, 2}, {2, 0}, {0, 3}, {1, 3}, {2, 3}};
        // E_k = voigt(G_k), G_k = 4 x_k gL_k^T - H + 4 sum_{edges (k,o)} x_ko gL_o^T,
        // H = sum_k x_k gL_k^T: the corner products P_k are formed once
        T Ek[4][6], H[6];
#pragma unroll
        for (int k = 0; k < 4; ++k) {
#pragma unroll
            for (int q = 0; q < 6; ++q) Ek[k][q] = 0;
            vsym_acc<T>(xk[k], gL[k], Ek[k]);
        }
#pragma unroll
        for (int q = 0; q < 6; ++q) {
            H[q] = Ek[0][q] + Ek[1][q] + Ek[2][q] + Ek[3][q];
#pragma unroll
            for (int k = 0; k < 4; ++k) Ek[k][q] = (T)4 * Ek[k][q] - H[q];
        }
#pragma unroll
        for (int q = 0; q < 6; ++q) {
            const T u4[3] = {(T)4 * xk[4 + q][0], (T)4 * xk[4 + q][1], (T)4 * xk[4 + q][2]};
            vsym_acc<T>(u4, gL[E[q][1]], Ek[E[q][0]]);
            vsym_acc<T>(u4, gL[E[q][0]], Ek[E[q][1]]);
        }
        T S[6];
#pragma unroll
        for (int q = 0; q < 6; ++q) S[q] = Ek[0][q] + Ek[1][q] + Ek[2][q] + Ek[3][q];
        const T w = sk * vol * (T)0.25;
        const T c1 = (T)(QA_ - QB_);
        T dm[22];  // DK 4: one D for the element, read once
        if constexpr (DK == 4) {
            const uint32_t* D = (const uint32_t*)Dp;
#pragma unroll
            for (int q = 0; q < 11; ++q) {
                const uint32_t wv = ld_u_nt(D, (uint32_t)q * rs + m);
                dm[2 * q] = (T)bf2f(wv & 0xFFFFu);
                dm[2 * q + 1] = (T)bf2f(wv >> 16);
            }
        }
        if constexpr (DK == 4) {
            // One D for the element: the stress sigma(L) = sum_k L_k D E_k is
            // linear in the barycentrics and the forces integrate in closed form
            // with int L_a L_b dV = V (1 + delta_ab) / 20:
            //   corner i:     (V/20) (4 s_i - T) . gL_i,
            //   edge (a, b):  (4V/20) ((T + s_a) . gL_b + (T + s_b) . gL_a),
            // with s_k = D E_k and T = s_1 + ... + s_4 (the 4-point rule gives the
            // same values for constant D).
            const T v20 = sk * vol * (T)0.05;
            T sgk[4][6], T6[6] = {0, 0, 0, 0, 0, 0};
#pragma unroll
            for (int k = 0; k < 4; ++k)
#pragma unroll
                for (int r = 0; r < 6; ++r) {
                    T a = 0;
#pragma unroll
                    for (int c = 0; c < 6; ++c) a += dm[sym6(r, c)] * Ek[k][c];
                    sgk[k][r] = a * v20;
                    T6[r] += sgk[k][r];
                }
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                T v[6];
#pragma unroll
                for (int r = 0; r < 6; ++r) v[r] = (T)4 * sgk[i][r] - T6[r];
                tdot_add<T>(v, gL[i], f[i]);
            }
            T T4[6];  // the edges' factor 4 folded into their stress sums
#pragma unroll
            for (int r = 0; r < 6; ++r) T4[r] = (T)4 * T6[r];
#pragma unroll
            for (int q = 0; q < 6; ++q) {
                const int a = E[q][0], b = E[q][1];
                T va[6], vb[6];
#pragma unroll
                for (int r = 0; r < 6; ++r) {
                    va[r] = fma((T)4, sgk[a][r], T4[r]);
                    vb[r] = fma((T)4, sgk[b][r], T4[r]);
                }
                tdot_add<T>(va, gL[b], f[4 + q]);
                tdot_add<T>(vb, gL[a], f[4 + q]);
            }
            return;
        }
        T ST[6] = {0, 0, 0, 0, 0, 0};
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            T eps[6], sg[6];
#pragma unroll
            for (int q = 0; q < 6; ++q) eps[q] = (T)QB_ * S[q] + c1 * Ek[j][q];
            T d[22];
            if constexpr (DK == 0) {
                const T* D = (const T*)Dp;
#pragma unroll
                for (int k = 0; k < 21; ++k)
                    d[k] = ld_u_nt(D, (uint32_t)(j * 21 + k) * rs + m);
            } else if constexpr (DK == 2) {  // a row of 84 in LDS
                const T* D = (const T*)Dp;
#pragma unroll
                for (int k = 0; k < 21; ++k) d[k] = D[j * 21 + k];
            } else {
                const uint32_t* D = (const uint32_t*)Dp;
#pragma unroll
                for (int q = 0; q < 11; ++q) {
                    const uint32_t wv = ld_u_nt(D, (uint32_t)(j * 11 + q) * rs + m);
                    d[2 * q] = (T)bf2f(wv & 0xFFFFu);
                    d[2 * q + 1] = (T)bf2f(wv >> 16);
                }
            }
#pragma unroll
            for (int r = 0; r < 6; ++r) {
                T a = 0;
#pragma unroll
                for (int c = 0; c < 6; ++c) a += d[sym6(r, c)] * eps[c];
                sg[r] = a * w;
                ST[r] += sg[r];
            }
            // point-j part of the nodal forces
#pragma unroll
            for (int i = 0; i < 4; ++i) tdot_acc<T>(sg, gL[i], i == j ? (T)3 * c1 : -c1, f[i]);
#pragma unroll
            for (int q = 0; q < 6; ++q) {
                if (E[q][0] == j) tdot_acc<T>(sg, gL[E[q][1]], (T)4 * c1, f[4 + q]);
                if (E[q][1] == j) tdot_acc<T>(sg, gL[E[q][0]], (T)4 * c1, f[4 + q]);
            }
        }
#pragma unroll
        for (int q = 0; q < 6; ++q) {
            T g[3] = {gL[E[q][0]][0] + gL[E[q][1]][0], gL[E[q][0]][1] + gL[E[q][1]][1],
                      gL[E[q][0]][2] + gL[E[q][1]][2]};
            tdot_acc<T>(ST, g, (T)(4.0 * QB_), f[4 + q]);
        }
    }
}

// the same of element e and member m on member-innermost vectors x1 (and x2);
// nbase[n] is the offset of node n's row in them
template <typename T, int DK, int MODE>
__device__ __forceinline__ void ebe_element(const DevMesh& M, int MB, int m, long e, const void* __restrict__ Dv,
                                            const double* __restrict__ h, const double* __restrict__ mat,
                                            const StepConst& sc, const T* __restrict__ x1,
                                            const T* __restrict__ x2, T f[10][3], size_t nbase[10])
{
    const int EB = MB >= 64 ? 1 : 64 / MB;
    const long ne = M.ne;
    const T* geo = geo_of<T>(M);
    T gL[4][3];
#pragma unroll
    for (int k = 0; k < 12; ++k) gL[k / 3][k % 3] = geo[k * ne + e];
    const T vol = geo[12 * ne + e];
    int nodes[10];
#pragma unroll
    for (int k = 0; k < 10; ++k) nodes[k] = M.conn[k * ne + e];
    const int l = M.layer[e];
    const double rho = matv(mat, l, MAT_RHO, MB, m);
    double he = 0.0;
    if (sc.damping_mode == 0 && h) he = h[e * MB + m];
    else if (sc.damping_mode == 1) he = sc.h0;
    T sm, sk, cv = 0;
    op_scales<T, MODE>(sc, rho, (double)vol, he, sm, sk, cv);
    // addresses: a base per node (wave-uniform when a wavefront is one element)
    // plus a 32-bit lane offset, so loads use a scalar base and no 64-bit math;
    // the component's offset joins the uniform base
#pragma unroll
    for (int n = 0; n < 10; ++n) nbase[n] = (size_t)nodes[n] * 3 * MB;
    // element base (uniform per wavefront) + 32-bit row offsets
    constexpr int W = DK == 4 ? 11 : (DK == 1 ? 44 : 84);
    constexpr size_t B = DK == 0 ? sizeof(T) : 4;
    const size_t eb = (size_t)(e / EB) * EB, ei = (size_t)(e % EB);
    element_forces<T, DK, MODE>(
        gL, vol, sm, sk, cv, (const char*)Dv + (eb * W + ei) * MB * B, (uint32_t)(EB * MB), (uint32_t)m,
        [&](int n, int c, int v) { return ld_u((v ? x2 : x1) + (size_t)c * MB + nbase[n], (uint32_t)m); }, f);
}

// Dashpot rows of the boundary nodes: rows[(i * 3 + c) * MB + m] = (dashpot x)
// at boundary node i, summed in FP64, by block blk of nblk blocks of nthreads
// threads; returns the thread's share of x . (dashpot x) (its member: t % MB).
// MB <= 256.  Below 64 slots up to 8 lanes share a node's faces (a vertex of a
// face mesh has about six): the chain of dependent loads of a single lane
// walking them was the longest of a small problem's operator (9.5 us of 45 us
// per CG iteration with 360 elements).
template <typename T, typename XF>
__device__ __forceinline__ double boundary_rows(const DevMesh& M, int MB, int nm, const double* __restrict__ mat,
                                                double coef, XF x, const double* __restrict__ vI, bool on,
                                                T* __restrict__ rows, int blk, int nblk, int nthreads)
{
    const int parts = MB >= 64 ? 1 : (64 / MB < 8 ? 64 / MB : 8);
    const int t = threadIdx.x, m = t % MB, q = t / MB, part = q % parts;
    const int npb = nthreads / (MB * parts);  // nodes per block pass
    const bool act = m < nm && on;
    double dot = 0.0;
    for (long i = (long)blk * npb + q / parts; i < M.nbn; i += (long)nblk * npb) {
        double acc[3] = {0.0, 0.0, 0.0};
        if (act) dashpot_at(M, MB, m, (int)i, mat, coef, x, vI, acc, part, parts);
        for (int o = MB; o < MB * parts; o <<= 1)  // the lanes of a node: a fixed tree
#pragma unroll
            for (int c = 0; c < 3; ++c) acc[c] += __shfl_xor(acc[c], o);
        if (part == 0 && act) {
            const size_t node = M.bn_node[i];
#pragma unroll
            for (int c = 0; c < 3; ++c) {
                const T v = (T)acc[c];
                rows[((size_t)i * 3 + c) * MB + m] = v;
                dot += (double)x((node * 3 + c) * MB + m) * (double)v;
            }
        }
    }
    return dot;
}

// Diagonal 3x3 block of node n of one element:
//   c_M rho V Mref(n, n) I + c_K (V/4) sum_j B_n(j)^T D_j B_n(j)
// with B_n^T D B_n [c][d] = sum_{p,q} g_p g_q D[v(c, p)][v(d, q)], g = grad N_n
// at point j and v(c, p) the Voigt index of du_c/dx_p.  Per point the
// coefficients of the quadratic forms in (gx^2, gy^2, gz^2, gx gy, gy gz, gz gx)
// are formed once and shared by the nodes.
__device__ __forceinline__ constexpr int voigt_of(int c, int p)
{
    return c == p ? c : ((c + p == 1) ? 3 : ((c + p == 3) ? 4 : 5));
}

// those of the block's entries C0 .. C0 + NC - 1 in the order 00 01 02 11 12 22
template <int C0, int NC>
__device__ __forceinline__ void diag_coef(const double* __restrict__ d, double C[NC][6])
{
    constexpr int PQ[6][2] = {{0, 0}, {1, 1}, {2, 2}, {0, 1}, {1, 2}, {2, 0}};
    constexpr int CD[6][2] = {{0, 0}, {0, 1}, {0, 2}, {1, 1}, {1, 2}, {2, 2}};
#pragma unroll
    for (int i = 0; i < NC; ++i)
#pragma unroll
        for (int pq = 0; pq < 6; ++pq) {
            const int c = CD[C0 + i][0], dd = CD[C0 + i][1], p = PQ[pq][0], q = PQ[pq][1];
            double v = d[sym6(voigt_of(c, p), voigt_of(dd, q))];
            if (p != q) v += d[sym6(voigt_of(c, q), voigt_of(dd, p))];
            C[i][pq] = v;
        }
}

// adds w g^T C g (NC entries of the symmetric 3x3 block) for node n (a
// compile-time index after unrolling) with g = grad N_n at barycentrics L
template <int NC>
__device__ __forceinline__ void diag_node_add(int n, const double L[4], const double gL[4][3], const double C[NC][6],
                                              double w, double acc[NC])
{
    constexpr int E[6][2] = {{0, 1}, {1, 2}, {2, 0}, {0, 3}, {1, 3}, {2, 3}};
    double g[3];
    if (n < 4) {
#pragma unroll
        for (int a = 0; a < 3; ++a) g[a] = (4.0 * L[n] - 1.0) * gL[n][a];
    } else {
        const int ea = E[n - 4][0], eb = E[n - 4][1];
#pragma unroll
        for (int a = 0; a < 3; ++a) g[a] = 4.0 * (L[ea] * gL[eb][a] + L[eb] * gL[ea][a]);
    }
    const double gg[6] = {g[0] * g[0], g[1] * g[1], g[2] * g[2], g[0] * g[1], g[1] * g[2], g[2] * g[0]};
#pragma unroll
    for (int cd = 0; cd < NC; ++cd) {
        double a = 0.0;
#pragma unroll
        for (int pq = 0; pq < 6; ++pq) a += gg[pq] * C[cd][pq];
        acc[cd] += w * a;
    }
}

// With D constant over the element (the inner operator's bfloat16 element
// mean) the stiffness block of node n is C : int grad N_n grad N_n^T dV, and
// that integral has a closed form in the barycentric gradients g (int L_a^2 =
// V/10, int L_a L_b = V/20, int L_a = V/4): corner a 0.6 V g_a g_a^T; edge
// (a, b) 1.6 V (g_a g_a^T + g_b g_b^T) + 0.8 V (g_a g_b^T + g_b g_a^T).
// G = int d_p N_n d_q N_n dV / V in the order 00 11 22 01 12 20.
__device__ __forceinline__ void mean_grad_products(int n, const double gL[4][3], double G[6])
{
    constexpr int PQ[6][2] = {{0, 0}, {1, 1}, {2, 2}, {0, 1}, {1, 2}, {2, 0}};
    constexpr int E[6][2] = {{0, 1}, {1, 2}, {2, 0}, {0, 3}, {1, 3}, {2, 3}};
#pragma unroll
    for (int pq = 0; pq < 6; ++pq) {
        const int p = PQ[pq][0], q = PQ[pq][1];
        if (n < 4) {
            G[pq] = 0.6 * gL[n][p] * gL[n][q];
        } else {
            const int a = E[n - 4][0], b = E[n - 4][1];
            G[pq] = 1.6 * (gL[a][p] * gL[a][q] + gL[b][p] * gL[b][q]) +
                    0.8 * (gL[a][p] * gL[b][q] + gL[b][p] * gL[a][q]);
        }
    }
}

// Per-member sums of ND x nblk partial rows of MB <= 32 slots by the first NT
// threads of a block of TB (valid in threads t < MB).  The order depends on NT and MB
// alone, so every kernel that forms the same stage with the same NT gets the same
// bits.  Eight loads of a thread in flight at a time.
template <int ND, int NT = 256, int TB = NT>
__device__ __forceinline__ void member_sums(const double* __restrict__ partial, int nblk, int MB, double* __restrict__ sh,
                                            double S[ND])
{
    constexpr int nw = NT / 64;
    const int t = threadIdx.x, m = t % MB, rpb = NT / MB;
    const bool sums = TB == NT || t < NT;
    double a[ND];
#pragma unroll
    for (int k = 0; k < ND; ++k) a[k] = 0.0;
    for (int b = sums ? t / MB : nblk; b < nblk; b += 8 * rpb) {
        double v[ND][8];
#pragma unroll
        for (int k = 0; k < ND; ++k)
#pragma unroll
            for (int q = 0; q < 8; ++q)
                v[k][q] = b + q * rpb < nblk ? partial[((size_t)k * nblk + b + q * rpb) * MB + m] : 0.0;
#pragma unroll
        for (int k = 0; k < ND; ++k)
#pragma unroll
            for (int q = 0; q < 8; ++q) a[k] += v[k][q];
    }
#pragma unroll
    for (int k = 0; k < ND; ++k) {
        for (int o = 32; o >= MB; o >>= 1) a[k] += __shfl_xor(a[k], o);
        if (sums && (t & 63) < MB) sh[(k * nw + (t >> 6)) * MB + (t & 63)] = a[k];
    }
    __syncthreads();
#pragma unroll
    for (int k = 0; k < ND; ++k) {
        S[k] = 0.0;
        if (t < MB)
            for (int w = 0; w < nw; ++w) S[k] += sh[(k * nw + w) * MB + t];
    }
}

// The beta stage by every block of the kernel that updates p (few partial sums: a launch of
// its own costs more than the sums, 5 us a stage against 2): S = (r.r, r.z) of
// member t, for threads t < MB.  What block 0 writes here (convergence, counts,
// r.z) the other blocks read from what the alpha stage left (inner_upd, rz_prev,
// iters_prev).  `on`: the member iterates on.  Same logic as stage_logic(FIN_BETA / FIN_IN_BETA).
template <bool INNER>
__device__ __forceinline__ double fused_beta(const StageIn& st, int m, const double S[2], bool upd, double rz_prev,
                                             int it, double ref, int MB, bool write, bool& on)
{
    const CgScalars& cs = st.cs;
    on = false;
    if (!upd) return 0.0;
    ++it;
    const bool conv = S[0] <= st.tol2 * ref, stop = conv || it >= st.maxit;
    const double beta = stop ? 0.0 : S[1] / rz_prev;
    on = !stop;
    if (write) {
        if (INNER) {
            cs.inner_iters[m] = it;
            cs.inner_total[m] += 1;
            if (stop) {
                cs.inner_active[m] = 0;
            } else {
                cs.ibeta[m] = beta;
                cs.irz[m] = S[1];
                if (it <= kLanczosMax) cs.lz[(long)(kLanczosMax + it - 1) * MB + m] = beta;
            }
        } else {
            cs.iters[m] = it;
            cs.rr[m] = S[0];
            if (stop) {
                cs.active[m] = 0;
                if (!conv) cs.status[m] = -5;
            } else {
                cs.beta[m] = beta;
                cs.rz[m] = S[1];
            }
        }
    }
    return beta;
}

// the stage's inputs of member t, loaded ahead of its sums
template <bool INNER>
struct BetaState {
    bool upd = false;
    double rz_prev = 0.0, ref = 0.0;
    int it = 0;
    __device__ __forceinline__ BetaState(const CgScalars& cs, int MB, int nm)
    {
        const int t = threadIdx.x;
        if (t >= MB || t >= nm) return;
        upd = cs.inner_upd[t];
        rz_prev = cs.rz_prev[t];
        ref = INNER ? cs.ir0[t] : cs.bb[t];
        it = cs.iters_prev[t];
    }
};

}  // namespace nlth
