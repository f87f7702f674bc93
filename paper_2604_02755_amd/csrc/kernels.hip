// HIP kernels (gfx950) for the nonlinear time-history ensemble solver.
//
// Method: Ichimura et al., arXiv 2604.02755.  Section 2.1, Eq. 1 (Newmark
// incremental step), Eq. 2 (K_e from D at the integration points), the
// multi-spring Ramberg-Osgood/Masing law; Section 2.2, Algorithm 4 (EBE
// operator inside CG, law update per step).
//
// All per-member data is member-innermost (index * MB + m): one lane handles
// one (element, member) or (node, member) pair; when MB >= 64 a wavefront
// covers 64 members of one element, so element data is wave-uniform and
// member data is read in contiguous 256/512-byte rows.
//
// Element forces reach the nodes without atomics and in a fixed order: a block
// sums those of a cluster of consecutive elements in LDS and writes the cluster's
// node rows, which a node pass sums (here for 64 to 256 member slots, in
// slots.hip below that); above 256 slots a launch covers one colour of the
// element colouring (no two elements of a colour share a node) and adds into the
// nodal vector, the colours in sequence on one stream.
#include <math.h>

#include "device.hpp"

namespace nlth {

// Shape-function gradients of the quadratic tet at integration point j.
template <typename T>
__device__ __forceinline__ void shape_grads(int j, const T gL[4][3], T G[10][3])
{
    T L[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) L[i] = (i == j) ? (T)QA_ : (T)QB_;
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int a = 0; a < 3; ++a) G[i][a] = ((T)4 * L[i] - (T)1) * gL[i][a];
    constexpr int E[6][2] = {{0, 1}, {1, 2}, {2, 0}, {0, 3}, {1, 3}, {2, 3}};
#pragma unroll
    for (int e = 0; e < 6; ++e)
#pragma unroll
        for (int a = 0; a < 3; ++a)
            G[4 + e][a] = (T)4 * (L[E[e][0]] * gL[E[e][1]][a] + L[E[e][1]] * gL[E[e][0]][a]);
}

// engineering strain (Voigt xx, yy, zz, xy, yz, zx) of nodal field u at one point
template <typename T>
__device__ __forceinline__ void strain(const T G[10][3], const T u[10][3], T eps[6])
{
#pragma unroll
    for (int k = 0; k < 6; ++k) eps[k] = 0;
#pragma unroll
    for (int n = 0; n < 10; ++n) {
        eps[0] += G[n][0] * u[n][0];
        eps[1] += G[n][1] * u[n][1];
        eps[2] += G[n][2] * u[n][2];
        eps[3] += G[n][1] * u[n][0] + G[n][0] * u[n][1];
        eps[4] += G[n][2] * u[n][1] + G[n][1] * u[n][2];
        eps[5] += G[n][0] * u[n][2] + G[n][2] * u[n][0];
    }
}

// ---------------------------------------------------------------------------
// simple vector kernels
// ---------------------------------------------------------------------------

__global__ void k_fill(double* p, double v, long n)
{
    long i = blockIdx.x * (long)blockDim.x + threadIdx.x;
    if (i < n) p[i] = v;
}
__global__ void k_fill32(float* p, float v, long n)
{
    long i = blockIdx.x * (long)blockDim.x + threadIdx.x;
    if (i < n) p[i] = v;
}
__global__ void k_neg_copy(const double* a, double* b, long n)
{
    long i = blockIdx.x * (long)blockDim.x + threadIdx.x;
    if (i < n) b[i] = -a[i];
}
__global__ void k_copy_i32(const int* a, int* b, int n)
{
    int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) b[i] = a[i];
}

static inline unsigned nblocks(long n, int bs = 256) { return (unsigned)((n + bs - 1) / bs); }

void launch_copy_i32(hipStream_t s, const int* src, int* dst, int n)
{
    if (n > 0) hipLaunchKernelGGL(k_copy_i32, dim3(nblocks(n)), dim3(256), 0, s, src, dst, n);
}
void launch_fill(hipStream_t s, double* p, double v, long n)
{
    if (n > 0) hipLaunchKernelGGL(k_fill, dim3(nblocks(n)), dim3(256), 0, s, p, v, n);
}
void launch_fill32(hipStream_t s, float* p, float v, long n)
{
    if (n > 0) hipLaunchKernelGGL(k_fill32, dim3(nblocks(n)), dim3(256), 0, s, p, v, n);
}
void launch_neg_copy(hipStream_t s, const double* a, double* b, long n)
{
    if (n > 0) hipLaunchKernelGGL(k_neg_copy, dim3(nblocks(n)), dim3(256), 0, s, a, b, n);
}

// ---------------------------------------------------------------------------
// element-by-element operator, colour and cluster forms (the element's
// arithmetic is in device.hpp; the form for few member slots in slots.hip)
// ---------------------------------------------------------------------------

// Colour form (more than 256 member slots, or scatter = 1): positions [e0, e1)
// of the colour lists (tets of one colour share no node), forces added into y.
template <typename T, int DK, int MODE, bool WAVE_ELEM>
__global__ __launch_bounds__(256) void k_ebe(DevMesh M, int MB, int nm, int e0, int e1,
                                            const void* __restrict__ Dv, const double* __restrict__ h,
                                            const double* __restrict__ mat, StepConst sc,
                                            const T* __restrict__ x1, const T* __restrict__ x2,
                                            T* __restrict__ y, const int* __restrict__ active)
{
    const long t = blockIdx.x * (long)blockDim.x + threadIdx.x;
    const int m = (int)(t % MB);
    long e = e0 + t / MB;
    if (WAVE_ELEM) e = __builtin_amdgcn_readfirstlane((int)e);  // one element per wavefront
    if (e >= e1 || m >= nm) return;
    if (active && !active[m]) return;
    e = WAVE_ELEM ? __builtin_amdgcn_readfirstlane(M.celem[e]) : M.celem[e];
    size_t nbase[10];
    T f[10][3];
    ebe_element<T, DK, MODE>(M, MB, m, e, Dv, h, mat, sc, x1, x2, f, nbase);
#pragma unroll
    for (int n = 0; n < 10; ++n) {
        T* yb = y + nbase[n];
#pragma unroll
        for (int c = 0; c < 3; ++c) yb[(uint32_t)(c * MB + m)] += f[n][c];
    }
}

// Cluster form of the operator (members padded to a multiple of 64): a block
// takes one cluster of consecutive storage elements (at most kClusterNodes
// distinct nodes) and 64 members; its four wavefronts compute four elements
// at a time (one element, 64 members per wavefront) and add their forces into
// the cluster's node rows in LDS, wavefront after wavefront, so the order of
// the sums is fixed.  The cluster's node rows are then written to
// co[(row * 3 + c) * MB + m] (row = the cluster's first row + local node) and
// a gather over the node -> rows lists finishes the sum.  nbb blocks spread
// over the grid write the dashpot rows of the boundary nodes (first in the grid
// they held every CU for 30 us); FP32 launches of more cluster blocks than
// kBoundaryApart leave them to a launch of their own (element-mean D, with and
// apart, us: 24,576 blocks (221,184 elements, 64 members) 649 and 665; 32,768 (147,456,
// 128 members) 862 and 850; 36,864 (442,368, 64) 1,107 and 1,085; 65,536 (786,432, 64)
// 1,987 and 1,920, with D per point 2,868 and 2,805).  With partial, the per-member sums of x1 .
// (operator x1) over a block's rows go to partial[block * MB + m] (nbb + clusters
// rows), so the node sums need not read x for a dot product.
// LDS of a cluster block: the node rows, padded so that NB blocks share a CU
// (160 KB of LDS per CU, allocated in 8 KB steps).  With one bfloat16 D per
// element four FP32 blocks per CU run fastest; with D per point four thrash
// the L2 that holds the nodal rows shared by neighbouring clusters and three
// are faster; two leave too few wavefronts to cover latency.
template <typename T, int NB>
constexpr int cluster_lds_elems()
{
    constexpr int rows = kClusterNodes * 3 * 64;
    constexpr int want = (NB == 3 ? 46 * 1024 : (NB == 2 ? 64 * 1024 : 0)) / (int)sizeof(T);
    return want > rows ? want : rows;
}

template <typename T, int DK, int MODE, int NB>
__global__ __launch_bounds__(256) void k_ebe_cluster(DevMesh M, int MB, int nm, int ngroups, int nbb,
                                                    const void* __restrict__ Dv, const double* __restrict__ h,
                                                    const double* __restrict__ mat, StepConst sc,
                                                    const T* __restrict__ x1, const T* __restrict__ x2,
                                                    T* __restrict__ co, const int* __restrict__ active, double dcoef,
                                                    const double* __restrict__ vI, double* __restrict__ partial)
{
    __shared__ T ys[cluster_lds_elems<T, NB>()];
    // groups of eight blocks, one per XCD; every gs-th group is a boundary group, or
    // the last ones of a launch of few rounds, where they took the places of clusters
    // (833 clusters of 64 members: FP32 71 us, at the end 52; FP64 173 and 132)
    const int gi = blockIdx.x >> 3, nb8 = nbb >> 3, ng = gridDim.x >> 3, gs = nb8 ? ng / nb8 : 1;
    const bool at_end = (int)gridDim.x - nbb <= kBoundaryAtEnd;
    const bool bnd = nb8 && (at_end ? gi >= ng - nb8 : gi % gs == gs - 1 && gi / gs < nb8);
    int gb = 0;  // boundary groups before this one
    if (at_end) gb = bnd ? gi - (ng - nb8) : 0;
    else if (nb8) gb = gi / gs < nb8 ? gi / gs : nb8;
    if (bnd) {
        const int bb = gb * 8 + (blockIdx.x & 7);
        const int mm = threadIdx.x % MB;
        const double d = boundary_rows<T>(M, MB, nm, mat, dcoef, [&](size_t n) { return x1[n]; }, vI,
                                          !active || (mm < nm && active[mm]), co + (size_t)M.cl_rows * 3 * MB, bb, nbb,
                                          256);
        if (!partial) return;
        double* sh = (double*)ys;
        sh[threadIdx.x] = d;  // all of member t % MB
        __syncthreads();
        if ((int)threadIdx.x < MB) {
            double a = d;
            for (int o = MB; o < 256; o += MB) a += sh[threadIdx.x + o];
            partial[(size_t)bb * MB + threadIdx.x] = a;
        }
        return;
    }
    // XCD-contiguous clusters
    const long blk = (long)(blockIdx.x & 7) * ((gridDim.x - nbb) >> 3) + (gi - gb);
    const int c = (int)(blk / ngroups), g = (int)(blk % ngroups);
    if (c >= M.ncl) return;  // whole block: padding of the grid to a multiple of 8
    // the wavefront index is uniform: saying so keeps the element's
    // connectivity and row bases in scalar registers (scalar loads and
    // address arithmetic instead of per-lane 64-bit adds)
    const int t = threadIdx.x, lane = t & 63, w = __builtin_amdgcn_readfirstlane(t >> 6);
    const int m = g * 64 + lane;
    const int e0 = M.cl_off[c], nec = M.cl_off[c + 1] - e0;
    const int r0 = M.cl_noff[c], ncn = M.cl_noff[c + 1] - r0;
    for (int i = t; i < ncn * 3 * 64; i += 256) ys[i] = (T)0;
    const bool act = m < nm && (!active || active[m]);
    __syncthreads();
    for (int r = 0; r < nec; r += 4) {
        const int le = r + w;
        T f[10][3];
        if (le < nec && act) {
            size_t nbase[10];
            ebe_element<T, DK, MODE>(M, MB, m, e0 + le, Dv, h, mat, sc, x1, x2, f, nbase);
        } else {
#pragma unroll
            for (int n = 0; n < 10; ++n) f[n][0] = f[n][1] = f[n][2] = (T)0;
        }
        // local node indices, four per 32-bit word (uniform: scalar loads)
        uint32_t lw[3] = {0u, 0u, 0u};
        if (le < nec) {
            const uint32_t* lp = M.cl_lconn + (size_t)(e0 + le) * 4;
            lw[0] = lp[0];
            lw[1] = lp[1];
            lw[2] = lp[2];
        }
        for (int ww = 0; ww < 4; ++ww) {
            __syncthreads();
            if (w == ww && le < nec) {
                // LDS read-add-write (the no-return LDS atomic add measured 3.5x
                // slower for the whole kernel).  An element's ten nodes are
                // distinct rows: all thirty values are read before any is
                // written back, one LDS round trip instead of ten.
                T* yr[10];
                T v[10][3];
#pragma unroll
                for (int n = 0; n < 10; ++n) {
                    yr[n] = ys + (int)((lw[n / 4] >> (8 * (n % 4))) & 0xFFu) * 3 * 64 + lane;
                    v[n][0] = yr[n][0];
                    v[n][1] = yr[n][64];
                    v[n][2] = yr[n][128];
                }
#pragma unroll
                for (int n = 0; n < 10; ++n) {
                    yr[n][0] = v[n][0] + f[n][0];
                    yr[n][64] = v[n][1] + f[n][1];
                    yr[n][128] = v[n][2] + f[n][2];
                }
            }
        }
    }
    __syncthreads();
    if (!partial) {
        for (int i = t; i < ncn * 3 * 64; i += 256) {
            const int q = i >> 6;  // row * 3 + component within the cluster
            co[((size_t)r0 * 3 + q) * MB + g * 64 + (i & 63)] = ys[i];
        }
        return;
    }
    // with the dot: a wavefront writes a row's three components, every fourth row,
    // the loads of x four rows at a time (one at a time their latency showed:
    // FP64 1141 us a launch against 1110, FP32 794 against 727)
    double dot = 0.0;
    const int* nodes = M.cl_nodes + (size_t)c * M.cl_node_stride;
    for (int q0 = w; q0 < ncn; q0 += 16) {
        T xv[4][3];
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const int q = q0 + 4 * u < ncn ? q0 + 4 * u : q0;
            const T* xp = x1 + (size_t)nodes[q] * 3 * MB + m;
#pragma unroll
            for (int cc = 0; cc < 3; ++cc) xv[u][cc] = xp[cc * MB];
        }
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const int q = q0 + 4 * u;
            if (q < ncn) {
                T* p = co + ((size_t)r0 + q) * 3 * MB + m;
#pragma unroll
                for (int cc = 0; cc < 3; ++cc) {
                    const T y = ys[(q * 3 + cc) * 64 + lane];
                    p[cc * MB] = y;
                    dot += (double)xv[u][cc] * (double)y;
                }
            }
        }
    }
    __syncthreads();
    double* sh = (double*)ys;  // the four wavefronts one after another
    sh[t] = act ? dot : 0.0;
    __syncthreads();
    if (t < 64) partial[((size_t)nbb + c) * MB + m] = sh[t] + sh[t + 64] + sh[t + 128] + sh[t + 192];
}

// boundary blocks of a cluster launch (a multiple of 8, so that the clusters
// keep their XCDs) and its rows of partial sums
static int cluster_bnd_blocks(const DevMesh& M, int MB, double dcoef)
{
    if (dcoef == 0.0 || M.nbn <= 0) return 0;
    const long npb = 256 / MB, n = (M.nbn + npb - 1) / npb;
    return (int)((n < kDashpotBlocks ? n : kDashpotBlocks) + 7) / 8 * 8;
}

// The dashpot rows as a launch of their own, a pass a block.
template <typename T>
__global__ __launch_bounds__(256) void k_boundary_rows(DevMesh M, int MB, int nm, const double* __restrict__ mat,
                                                      double dcoef, const T* __restrict__ x,
                                                      const int* __restrict__ active, T* __restrict__ rows)
{
    const int m = threadIdx.x % MB;
    boundary_rows<T>(M, MB, nm, mat, dcoef, [&](size_t n) { return x[n]; }, nullptr, !active || (m < nm && active[m]),
                     rows, blockIdx.x, gridDim.x, 256);
}

// blocks of the FP32 cluster launches per CU (a tuning knob, per host thread)
static thread_local int t_cluster_blocks = 3;
void set_cluster_blocks(int b) { t_cluster_blocks = (b == 2 || b == 3 || b == 4) ? b : 3; }

template <typename T, int DK, int MODE, int NB>
static void cluster_launch(hipStream_t s, const DevMesh& M, int MB, int nm, const void* D, const double* h,
                           const double* mat, StepConst sc, const T* x1, const T* x2, T* co, const int* active,
                           double dcoef, const double* vI, double* partial, int* nblk)
{
    const int ngroups = MB / 64;
    const long g = ((long)M.ncl * ngroups + 7) / 8 * 8;
    int nbb = cluster_bnd_blocks(M, MB, dcoef);
    if (sizeof(T) == 4 && nbb && !partial && g > kBoundaryApart) {
        const int npb = 256 / MB;
        hipLaunchKernelGGL((k_boundary_rows<T>), dim3((M.nbn + npb - 1) / npb), dim3(256), 0, s, M, MB, nm, mat, dcoef, x1,
                           active, co + (size_t)M.cl_rows * 3 * MB);
        nbb = 0;
    }
    if (nblk) *nblk = nbb + M.ncl;
    hipLaunchKernelGGL((k_ebe_cluster<T, DK, MODE, NB>), dim3((unsigned)(nbb + g)), dim3(256), 0, s, M, MB, nm, ngroups,
                       nbb, D, h, mat, sc, x1, x2, co, active, dcoef, vI, partial);
}

// FP32 operator (A) with D storage DK, NB blocks per CU
template <int DK>
static void cluster32(hipStream_t s, const DevMesh& M, int MB, int nm, const void* D, const double* h,
                      const double* mat, StepConst sc, const float* x, float* co, const int* active, double dcoef,
                      double* partial, int* nblk)
{
    const float* none = nullptr;
    switch (t_cluster_blocks) {
    case 2: cluster_launch<float, DK, OP_A, 2>(s, M, MB, nm, D, h, mat, sc, x, none, co, active, dcoef, nullptr, partial, nblk); break;
    case 4: cluster_launch<float, DK, OP_A, 4>(s, M, MB, nm, D, h, mat, sc, x, none, co, active, dcoef, nullptr, partial, nblk); break;
    default: cluster_launch<float, DK, OP_A, 3>(s, M, MB, nm, D, h, mat, sc, x, none, co, active, dcoef, nullptr, partial, nblk); break;
    }
}

void launch_ebe_cluster64(hipStream_t s, OpMode mode, const DevMesh& M, int MB, int nm, const double* D,
                          const double* h, const double* mat, StepConst sc, const double* x1, const double* x2,
                          double* co, const int* active, double dcoef, const double* vI, double* partial, int* nblk)
{
    // FP64 rows take 72 KB: two blocks per CU
    switch (mode) {
    case OP_A: cluster_launch<double, 0, OP_A, 2>(s, M, MB, nm, D, h, mat, sc, x1, x2, co, active, dcoef, vI, partial, nblk); break;
    case OP_K: cluster_launch<double, 0, OP_K, 2>(s, M, MB, nm, D, h, mat, sc, x1, x2, co, active, dcoef, vI, partial, nblk); break;
    case OP_M: cluster_launch<double, 0, OP_M, 2>(s, M, MB, nm, D, h, mat, sc, x1, x2, co, active, dcoef, vI, partial, nblk); break;
    case OP_RHS: cluster_launch<double, 0, OP_RHS, 2>(s, M, MB, nm, D, h, mat, sc, x1, x2, co, active, dcoef, vI, partial, nblk); break;
    }
}

void launch_ebe_cluster32(hipStream_t s, const DevMesh& M, int MB, int nm, const float* D32, const uint32_t* D16,
                          bool d16_mean, const double* h, const double* mat, StepConst sc, const float* x, float* co,
                          const int* active, double dcoef, double* partial, int* nblk)
{
    if (D16 && d16_mean) cluster32<4>(s, M, MB, nm, D16, h, mat, sc, x, co, active, dcoef, partial, nblk);
    else if (D16) cluster32<1>(s, M, MB, nm, D16, h, mat, sc, x, co, active, dcoef, partial, nblk);
    else cluster32<0>(s, M, MB, nm, D32, h, mat, sc, x, co, active, dcoef, partial, nblk);
}

// sum of a node's rows: cluster rows ascending, then (bnd) its dashpot row, so
// the sum is reproducible; W lanes per row
template <typename T>
__device__ __forceinline__ void node_rows(const DevMesh& M, long node, const T* __restrict__ f, int W, int m, bool bnd,
                                          T a[3])
{
    a[0] = a[1] = a[2] = 0;
    const int q1 = M.cn_ptr[node + 1] - (!bnd && M.bn_of_node[node] >= 0);
#pragma unroll 4
    for (int q = M.cn_ptr[node]; q < q1; ++q) {
        const T* fb = f + (size_t)M.cn_row[q] * 3 * W + m;
        a[0] += fb[0];
        a[1] += fb[W];
        a[2] += fb[2 * W];
    }
}

// y = the node's rows + bscale * base (base may be NULL and may alias y);
// members with active[m] == 0 keep y and add nothing.  With DOT the per-member
// partial sums of x . y over the block's nodes (a fixed tree in LDS).  A block takes a contiguous range of
// nodes, 256 / MB per pass (MB <= 256): with nodes in Morton order,
// interleaving the blocks' passes over the whole range was 40 % slower
// (concurrent blocks then read cluster rows of one small region).
template <typename T, bool DOT>
__global__ __launch_bounds__(256) void k_gather(DevMesh M, int MB, int nm, const T* __restrict__ f, int bnd,
                                               const T* base, T bscale, T* y, const int* __restrict__ active,
                                               const int* __restrict__ ymap, const T* __restrict__ x,
                                               double* __restrict__ partial)
{
    const int t = threadIdx.x, m = t % MB;
    const int rpb = 256 / MB;
    const int slot = t / MB;
    const bool act = m < nm && (!active || active[m]);
    double dot = 0.0;
    const long per = ((M.nn + gridDim.x - 1) / gridDim.x + rpb - 1) / rpb * rpb;
    const long n0 = (long)blockIdx.x * per, n1 = n0 + per < M.nn ? n0 + per : M.nn;
    for (long nd = n0 + slot; act && nd < n1; nd += rpb) {
        const int node = MB >= 64 ? __builtin_amdgcn_readfirstlane((int)nd) : (int)nd;
        T a[3];
        node_rows<T>(M, node, f, MB, m, bnd, a);
        const size_t yi = (size_t)(ymap ? ymap[node] : node) * 3 * MB + m;
#pragma unroll
        for (int c = 0; c < 3; ++c) {
            if (base) a[c] += bscale * base[yi + (size_t)c * MB];
            y[yi + (size_t)c * MB] = a[c];
            if (DOT) dot += (double)x[yi + (size_t)c * MB] * (double)a[c];
        }
    }
    if (DOT) {
        __shared__ double sh[256];
        sh[t] = dot;
        __syncthreads();
        for (int s = 128; s >= MB; s >>= 1) {
            if (t < s) sh[t] += sh[t + s];
            __syncthreads();
        }
        if (t < MB) partial[(size_t)blockIdx.x * MB + t] = sh[t];
    }
}

// blocks of a gather launch: node passes of 256 / MB nodes, at most maxblk
static int gather_blocks(int nn, int MB, int maxblk)
{
    const long rpb = 256 / MB;
    const long g = (nn + rpb - 1) / rpb;
    return (int)(g < 1 ? 1 : (g > maxblk ? maxblk : g));
}

template <typename T>
void launch_gather(hipStream_t s, const DevMesh& M, int MB, int nm, const T* rows, bool bnd, const T* base, T bscale,
                   T* y, const int* active, const int* ymap)
{
    hipLaunchKernelGGL((k_gather<T, false>), dim3(gather_blocks(M.nn, MB, 1 << 24)), dim3(256), 0, s, M, MB, nm, rows,
                       (int)bnd, base, bscale, y, active, ymap, nullptr, nullptr);
}
void launch_gather_dot(hipStream_t s, const DevMesh& M, int MB, int nm, const float* rows, float* y, const int* active,
                       const float* x, double* partial, int* nblk)
{
    const int g = gather_blocks(M.nn, MB, kGatherBlocks);
    const float* none = nullptr;
    *nblk = g;
    hipLaunchKernelGGL((k_gather<float, true>), dim3(g), dim3(256), 0, s, M, MB, nm, rows, 1, none, 0.0f, y, active,
                       nullptr, x, partial);
}
template void launch_gather<double>(hipStream_t, const DevMesh&, int, int, const double*, bool, const double*, double,
                                    double*, const int*, const int*);
template void launch_gather<float>(hipStream_t, const DevMesh&, int, int, const float*, bool, const float*, float,
                                   float*, const int*, const int*);

// The node sums of a CG iteration's operator application with the update that
// needs them, so q = A p is not written and read back: with alpha from p . q
// (taken on the rows by the operator; the FP32 operator of 64 and more slots is
// not bound by memory and pays more for the dot than this saves: 727 + 509 us
// against 610 + 300 + 262 for the gather and k_inner_update, 221,184 elements and
// 64 members; the FP64 one 1100 + 357 + 203 against 1040 + 270 + 362 + 128 with
// the x update in the p update),
//   UPD_PZ: r -= alpha q, z = P r; partials (r.r, r.z)       (the PCGs)
//   UPD_XR: r -= alpha q, x += alpha p, Ap = q; partial r.r  (the outer flexible
//           CG, whose beta reads Ap)
// for the active members.  G = 0: full rows of MB lanes; 16 or 32: the compact
// rows of the listed members, partials in the full layout.  Bound by HBM: per
// DOF-member of the FP32 inner CG on 64 members the rows (2.7 per node) 11 B, r
// read and written and z written 12 B, the inverse 8 B.
// FUSED (few slots, few partial sums): every block forms the alpha stage from the
// operator's partial sums itself, with its first node's loads under way, and
// block 0 writes what stage_logic(FIN_ALPHA / FIN_IN_ALPHA) would; no thread reads
// those (sg.partial is not this launch's own `partial`).
template <typename T, int KIND, int G, bool FUSED>
__global__ __launch_bounds__(256) void k_rows_update(DevMesh M, int MB, int nm, const int* __restrict__ tl,
                                                    const T* __restrict__ f, T* __restrict__ r, T* __restrict__ z,
                                                    const T* __restrict__ pinv, T* __restrict__ x,
                                                    const T* __restrict__ p, const double* __restrict__ alpha,
                                                    const int* __restrict__ active, double* __restrict__ partial,
                                                    StageIn sg)
{
    const int W = G ? G : MB, t = threadIdx.x, k = t % W, slot = t / W;
    const int npb = 256 / W;
    const int m = !G ? k : (k < min(tl[0], W) ? tl[1 + k] : -1);
    const bool act = m >= 0 && m < nm && active[m];
    double d0 = 0.0, d1 = 0.0;
    const long per = ((M.nn + gridDim.x - 1) / gridDim.x + npb - 1) / npb * npb;
    const long n0 = (long)blockIdx.x * per, n1 = n0 + per < M.nn ? n0 + per : M.nn;
    T q[3], R[3], P[6];
    auto load = [&](long node) {
        const size_t i = (size_t)node * 3 * W + k;
#pragma unroll
        for (int c = 0; c < 3; ++c) R[c] = r[i + (size_t)c * W];
        if (KIND == UPD_PZ) {
            const T* pv = pinv + (size_t)node * 6 * W + k;
#pragma unroll
            for (int c = 0; c < 6; ++c) P[c] = pv[(size_t)c * W];
        }
        node_rows<T>(M, node, f, W, k, true, q);
    };
    T al = 0;
    if constexpr (FUSED) {
        constexpr bool INNER = sizeof(T) == 4;
        const CgScalars& cs = sg.cs;
        if (act && n0 + slot < n1) load(n0 + slot);
        __shared__ double sum[4 * 32];
        __shared__ double sa[32];
        bool on = false;
        double rz = 0.0, S[1];
        if (t < MB && t < nm) {
            on = active[t];
            rz = INNER ? cs.irz[t] : cs.rz[t];
        }
        member_sums<1>(sg.partial, sg.nblk, MB, sum, S);
        if (t < MB) {
            const double a = on ? rz / S[0] : 0.0;
            sa[t] = a;
            if (blockIdx.x == 0 && t < nm) {
                const int it = INNER ? cs.inner_iters[t] : cs.iters[t];
                (INNER ? cs.ialpha : cs.alpha)[t] = a;
                cs.inner_upd[t] = on;
                cs.rz_prev[t] = rz;
                cs.iters_prev[t] = it;
                if (INNER) {
                    if (on && it < kLanczosMax) cs.lz[(long)it * MB + t] = a;
                } else {
                    cs.pAp[t] = S[0];
                }
            }
        }
        __syncthreads();
        al = (T)sa[k];
    } else if (act) {
        al = (T)alpha[m];
    }
    if (act) {
        for (long nd = n0 + slot; nd < n1; nd += npb) {
            const long node = !G && MB >= 64 ? (long)__builtin_amdgcn_readfirstlane((int)nd) : nd;
            if (!FUSED || nd != n0 + slot) load(node);
            const size_t i = (size_t)node * 3 * W + k;
#pragma unroll
            for (int c = 0; c < 3; ++c) {
                R[c] -= al * q[c];
                r[i + (size_t)c * W] = R[c];
                d0 += (double)R[c] * (double)R[c];
            }
            if (KIND == UPD_PZ) {
                const T Z[3] = {P[0] * R[0] + P[1] * R[1] + P[2] * R[2], P[1] * R[0] + P[3] * R[1] + P[4] * R[2],
                                P[2] * R[0] + P[4] * R[1] + P[5] * R[2]};
#pragma unroll
                for (int c = 0; c < 3; ++c) {
                    z[i + (size_t)c * W] = Z[c];
                    d1 += (double)R[c] * (double)Z[c];
                }
            } else {
#pragma unroll
                for (int c = 0; c < 3; ++c) {
                    z[i + (size_t)c * W] = q[c];
                    x[i + (size_t)c * W] += al * p[i + (size_t)c * W];
                }
            }
        }
    }
    constexpr int ND = KIND == UPD_PZ ? 2 : 1;
    if constexpr (G != 0) {
        double acc[ND];
        acc[0] = d0;
        if constexpr (ND > 1) acc[1] = d1;
        tail_partials<ND, G>(acc, MB, m, partial, 0, gridDim.x);
    } else {
        __shared__ double sh[ND][256];
        sh[0][t] = d0;
        if constexpr (ND > 1) sh[ND - 1][t] = d1;
        __syncthreads();
        for (int s = 128; s >= MB; s >>= 1) {
            if (t < s)
#pragma unroll
                for (int j = 0; j < ND; ++j) sh[j][t] += sh[j][t + s];
            __syncthreads();
        }
        if (t < MB)
#pragma unroll
            for (int j = 0; j < ND; ++j) partial[((size_t)j * gridDim.x + blockIdx.x) * MB + t] = sh[j][t];
    }
}

template <typename T>
void launch_rows_update(hipStream_t s, int kind, const DevMesh& M, int MB, int nm, int G, const int* tl, const T* rows,
                        T* r, T* z, const T* pinv, T* x, const T* p, const double* alpha, const int* active,
                        double* partial, int* nblk, const StageIn* fused)
{
    const int g = gather_blocks(M.nn, G ? G : MB, kMaxPartialBlocks);
    *nblk = g;
    const StageIn sg = fused ? *fused : StageIn{};
#define NLTH_UPD(KIND, GG, F)                                                                                        \
    hipLaunchKernelGGL((k_rows_update<T, KIND, GG, F>), dim3(g), dim3(256), 0, s, M, MB, nm, tl, rows, r, z, pinv, x, \
                       p, alpha, active, partial, sg)
    if (fused) {
        NLTH_UPD(UPD_PZ, 0, true);
        return;
    }
    if constexpr (sizeof(T) == 8) {
        if (kind == UPD_XR) {
            if (G == 0) NLTH_UPD(UPD_XR, 0, false);
            else if (G == 16) NLTH_UPD(UPD_XR, 16, false);
            else NLTH_UPD(UPD_XR, 32, false);
            return;
        }
    }
    if (G == 0) NLTH_UPD(UPD_PZ, 0, false);
    else if (G == 16) NLTH_UPD(UPD_PZ, 16, false);
    else NLTH_UPD(UPD_PZ, 32, false);
#undef NLTH_UPD
}
template void launch_rows_update<double>(hipStream_t, int, const DevMesh&, int, int, int, const int*, const double*,
                                         double*, double*, const double*, double*, const double*, const double*,
                                         const int*, double*, int*, const StageIn*);
template void launch_rows_update<float>(hipStream_t, int, const DevMesh&, int, int, int, const int*, const float*,
                                        float*, float*, const float*, float*, const float*, const double*, const int*,
                                        double*, int*, const StageIn*);

// threads per block of the element-by-element launches (a tuning knob; per
// host thread so concurrent contexts do not interfere)
static thread_local int t_ebe_block = 256;
void set_ebe_block(int bs) { t_ebe_block = (bs == 64 || bs == 128 || bs == 256) ? bs : 256; }

template <typename T, int DK, int MODE>
static void ebe_dispatch(hipStream_t s, const DevMesh& M, int MB, int nm, int e0, int e1, const void* D,
                         const double* h, const double* mat, StepConst sc, const T* x1, const T* x2, T* y,
                         const int* active)
{
    const dim3 g(nblocks((long)(e1 - e0) * MB, t_ebe_block)), b(t_ebe_block);
    if (MB >= 64) hipLaunchKernelGGL((k_ebe<T, DK, MODE, true>), g, b, 0, s, M, MB, nm, e0, e1, D, h, mat, sc, x1, x2, y, active);
    else hipLaunchKernelGGL((k_ebe<T, DK, MODE, false>), g, b, 0, s, M, MB, nm, e0, e1, D, h, mat, sc, x1, x2, y, active);
}

// inner FP32 operator (Eq. 1 left-hand side) with D stored in FP32 or bfloat16
void launch_ebe32(hipStream_t s, const DevMesh& M, int MB, int nm, int e0, int e1, const float* D32,
                  const uint32_t* D16, const double* h, const double* mat, StepConst sc, const float* x, float* y,
                  const int* active, bool d16_mean)
{
    if (e1 <= e0) return;
    if (D16 && d16_mean) ebe_dispatch<float, 4, OP_A>(s, M, MB, nm, e0, e1, D16, h, mat, sc, x, nullptr, y, active);
    else if (D16) ebe_dispatch<float, 1, OP_A>(s, M, MB, nm, e0, e1, D16, h, mat, sc, x, nullptr, y, active);
    else ebe_dispatch<float, 0, OP_A>(s, M, MB, nm, e0, e1, D32, h, mat, sc, x, nullptr, y, active);
}

// ---------------------------------------------------------------------------
// convergence tail: once at most G (16 or 32) members are still iterating,
// their CG runs on compact copies, lane k of a row being member tl[1 + k]
// (tl[0] = the count): the member-innermost rows of the full arrays would
// otherwise be fetched whole for a few members each.  The mixed path packs the
// element-mean D, h, the material rows and the FP32 block-Jacobi inverse once
// per outer iteration for its inner CG; the FP64 PCG packs the FP64 D per
// point, h, the material rows, its inverse and the CG vectors once per step.
// The operator (slots.hip) sums its element forces per element cluster into compact
// rows and takes p . A p on them, a partial sum of G lanes a block; the update
// (k_rows_update) sums the rows per node and keeps the full [block][MB] layout of
// its partial sums (zero for members not listed), so the stage logic is the same.
// ---------------------------------------------------------------------------

// rows of a member-innermost array, listed members only: compact row rc of G
// lanes <-> full row r of MB lanes.  With EBc > 1 the rows are W per element
// and the compact copy is blocked by EBc elements (the D layout of G slots).
template <typename T, bool UNPACK>
__global__ __launch_bounds__(256) void k_tail_rows(long nrows, int MB, int G, int W, int EBc,
                                                  const int* __restrict__ tl, const T* __restrict__ src,
                                                  T* __restrict__ dst)
{
    const long t = blockIdx.x * (long)blockDim.x + threadIdx.x;
    const int k = (int)(t % G);
    const long r = t / G;
    if (r >= nrows || k >= min(tl[0], G)) return;
    const int m = tl[1 + k];
    long rc = r;
    if (EBc > 1) {
        const long e = r / W;
        rc = ((e / EBc) * W + (r - e * W)) * EBc + e % EBc;
    }
    if (UNPACK) dst[r * MB + m] = src[rc * G + k];
    else dst[rc * G + k] = src[r * MB + m];
}

template <typename T>
static void tail_rows(hipStream_t s, long nrows, int MB, int G, int W, int EBc, const int* tl, const T* src, T* dst,
                      bool unpack)
{
    const long n = nrows * G;
    if (n <= 0) return;
    if (unpack)
        hipLaunchKernelGGL((k_tail_rows<T, true>), dim3(nblocks(n)), dim3(256), 0, s, nrows, MB, G, W, EBc, tl, src, dst);
    else
        hipLaunchKernelGGL((k_tail_rows<T, false>), dim3(nblocks(n)), dim3(256), 0, s, nrows, MB, G, W, EBc, tl, src, dst);
}

void launch_tail_pack(hipStream_t s, const DevMesh& M, int MB, int G, int n_layers, const int* tl,
                      const uint32_t* D16, const double* h, const double* mat, const float* pinv32, uint32_t* cD,
                      double* ch, double* cmat, float* cpinv)
{
    tail_rows<uint32_t>(s, (long)M.ne * 11, MB, G, 11, 64 / G, tl, D16, cD, false);
    if (h) tail_rows<double>(s, M.ne, MB, G, 1, 1, tl, h, ch, false);
    tail_rows<double>(s, (long)n_layers * MAT_N, MB, G, 1, 1, tl, mat, cmat, false);
    tail_rows<float>(s, (long)M.nn * 6, MB, G, 1, 1, tl, pinv32, cpinv, false);
}

void launch_tail_unpack(hipStream_t s, long nrows, int MB, int G, const int* tl, const float* c, float* full)
{
    tail_rows<float>(s, nrows, MB, G, 1, 1, tl, c, full, true);
}

void launch_tail_pack64(hipStream_t s, const DevMesh& M, int MB, int G, int n_layers, const int* tl,
                        const double* D64, const double* h, const double* mat, const double* pinv, double* cD,
                        double* ch, double* cmat, double* cpinv)
{
    tail_rows<double>(s, (long)M.ne * 84, MB, G, 84, 64 / G, tl, D64, cD, false);
    if (h) tail_rows<double>(s, M.ne, MB, G, 1, 1, tl, h, ch, false);
    tail_rows<double>(s, (long)n_layers * MAT_N, MB, G, 1, 1, tl, mat, cmat, false);
    tail_rows<double>(s, (long)M.nn * 6, MB, G, 1, 1, tl, pinv, cpinv, false);
}

void launch_tail_rows64(hipStream_t s, long nrows, int MB, int G, const int* tl, const double* src, double* dst,
                        bool unpack)
{
    tail_rows<double>(s, nrows, MB, G, 1, 1, tl, src, dst, unpack);
}

template <typename T>
void launch_ebe(hipStream_t s, OpMode mode, const DevMesh& M, int MB, int nm, int e0, int e1, const T* D,
                const double* h, const double* mat, int, StepConst sc, const T* x1, const T* x2, T* y,
                const int* active)
{
    if (e1 <= e0) return;
    switch (mode) {
    case OP_A: ebe_dispatch<T, 0, OP_A>(s, M, MB, nm, e0, e1, D, h, mat, sc, x1, x2, y, active); break;
    case OP_K: ebe_dispatch<T, 0, OP_K>(s, M, MB, nm, e0, e1, D, h, mat, sc, x1, x2, y, active); break;
    case OP_M: ebe_dispatch<T, 0, OP_M>(s, M, MB, nm, e0, e1, D, h, mat, sc, x1, x2, y, active); break;
    case OP_RHS: ebe_dispatch<T, 0, OP_RHS>(s, M, MB, nm, e0, e1, D, h, mat, sc, x1, x2, y, active); break;
    }
}
template void launch_ebe<double>(hipStream_t, OpMode, const DevMesh&, int, int, int, int, const double*,
                                 const double*, const double*, int, StepConst, const double*,
                                 const double*, double*, const int*);

// ---------------------------------------------------------------------------
// absorbing boundary: node-centric gather over boundary faces (deterministic)
// dashpot on a face: rho (Vp n n^T + Vs (I - n n^T)) times int N_a N_b dA
// ---------------------------------------------------------------------------

// y += dashpot at the boundary nodes (the colour form of the operator; the
// others write dashpot rows), one (node, member) pair per thread
template <typename T>
__global__ __launch_bounds__(256) void k_dashpot(DevMesh M, int MB, int nm, const double* __restrict__ mat, double coef,
                                                const T* __restrict__ x, T* __restrict__ y,
                                                const double* __restrict__ vI, const int* __restrict__ active)
{
    const long g = (long)blockIdx.x * 256 + threadIdx.x;
    const int m = (int)(g % MB);
    const long i = g / MB;
    if (i >= M.nbn || m >= nm || (active && !active[m])) return;
    double acc[3] = {0, 0, 0};
    dashpot_at(M, MB, m, (int)i, mat, coef, [&](size_t n) { return x[n]; }, vI, acc);
    const size_t yi = (size_t)M.bn_node[i] * 3 * MB + m;
#pragma unroll
    for (int c = 0; c < 3; ++c) y[yi + (size_t)c * MB] += (T)acc[c];
}

template <typename T>
void launch_dashpot(hipStream_t s, const DevMesh& M, int MB, int nm, const double* mat, T coef, const T* x, T* y,
                    const double* vI, const int* active)
{
    const long n = (long)M.nbn * MB;
    if (n > 0)
        hipLaunchKernelGGL((k_dashpot<T>), dim3(nblocks(n)), dim3(256), 0, s, M, MB, nm, mat, (double)coef, x, y, vI,
                           active);
}
template void launch_dashpot<double>(hipStream_t, const DevMesh&, int, int, const double*, double, const double*,
                                     double*, const double*, const int*);
template void launch_dashpot<float>(hipStream_t, const DevMesh&, int, int, const double*, float, const float*, float*,
                                    const double*, const int*);

// One fused Chebyshev iteration on the gather paths (MB <= 256): per node the
// rows are summed as the gather does, and with q = that sum
//   iz += id,  ir -= q,  id_next = c1_k id + c2_k P ir   (no id_next on the last)
// so the operator result never goes to memory.  Node ranges per block as in
// the gather.
__global__ __launch_bounds__(256) void k_gather_cheb(DevMesh M, int MB, int nm, int k, int last,
                                                    const float* __restrict__ rows,
                                                    float* __restrict__ iz, float* __restrict__ ir,
                                                    const float* __restrict__ id, float* __restrict__ id_next,
                                                    const float* __restrict__ pinv32, const float* __restrict__ cheb,
                                                    const int* __restrict__ active)
{
    const int t = threadIdx.x, m = t % MB;
    const int rpb = 256 / MB;
    const int slot = t / MB;
    const bool act = m < nm && (!active || active[m]);
    if (!act) return;
    float c1 = 0.0f, c2 = 0.0f;
    if (!last) {
        c1 = cheb[(long)(2 * k) * MB + m];
        c2 = cheb[(long)(2 * k + 1) * MB + m];
    }
    const long per = ((M.nn + gridDim.x - 1) / gridDim.x + rpb - 1) / rpb * rpb;
    const long n0 = (long)blockIdx.x * per, n1 = n0 + per < M.nn ? n0 + per : M.nn;
    for (long nd = n0 + slot; nd < n1; nd += rpb) {
        const int node = MB >= 64 ? __builtin_amdgcn_readfirstlane((int)nd) : (int)nd;
        float a[3];
        node_rows<float>(M, node, rows, MB, m, true, a);
        const size_t yi = (size_t)node * 3 * MB + m;
        const float d0 = id[yi], d1 = id[yi + MB], d2 = id[yi + 2 * MB];
        iz[yi] += d0;
        iz[yi + MB] += d1;
        iz[yi + 2 * MB] += d2;
        const float r0 = ir[yi] - a[0], r1 = ir[yi + MB] - a[1], r2 = ir[yi + 2 * MB] - a[2];
        ir[yi] = r0;
        ir[yi + MB] = r1;
        ir[yi + 2 * MB] = r2;
        if (last) continue;
        const float* pv = pinv32 + (size_t)node * 6 * MB + m;
        const float p0 = pv[0], p1 = pv[MB], p2 = pv[2 * MB], p3 = pv[3 * MB], p4 = pv[4 * MB], p5 = pv[5 * MB];
        const float w0 = p0 * r0 + p1 * r1 + p2 * r2;
        const float w1 = p1 * r0 + p3 * r1 + p4 * r2;
        const float w2 = p2 * r0 + p4 * r1 + p5 * r2;
        id_next[yi] = c1 * d0 + c2 * w0;
        id_next[yi + MB] = c1 * d1 + c2 * w1;
        id_next[yi + 2 * MB] = c1 * d2 + c2 * w2;
    }
}

void launch_gather_cheb(hipStream_t s, const DevMesh& M, int MB, int nm, int k, bool last, const float* rows,
                        float* iz, float* ir, const float* id, float* id_next, const float* pinv32,
                        const float* cheb, const int* active)
{
    const int g = gather_blocks(M.nn, MB, 1 << 24);
    hipLaunchKernelGGL(k_gather_cheb, dim3(g), dim3(256), 0, s, M, MB, nm, k, (int)last, rows, iz, ir, id, id_next,
                       pinv32, cheb, active);
}

// ---------------------------------------------------------------------------
// 3x3 block-Jacobi preconditioner (Section 2.2): diagonal blocks of A
// ---------------------------------------------------------------------------

// The blocks by colours (more than 256 slots): the elements of one colour share
// no node.  A thread takes one element-member
// and one part of the nodes (the 4 corners, edges 01 12 20, or edges 03 13
// 23), so it holds at most 4 blocks: FP64 register pressure sets the
// occupancy here, and each part re-reads D (from L2).
__global__ __launch_bounds__(256) void k_diag(DevMesh M, int MB, int nm, int e0, int e1,
                                             const double* __restrict__ D, const double* __restrict__ h,
                                             const double* __restrict__ mat, StepConst sc,
                                             double* __restrict__ diag)
{
    const long t = blockIdx.x * (long)blockDim.x + threadIdx.x;
    const int m = (int)(t % MB);
    long r = t / MB;
    if (MB >= 64) r = __builtin_amdgcn_readfirstlane((int)r);  // wavefront-uniform element and part
    const int part = (int)(r % 3);
    const long pos = e0 + r / 3;  // position in the colour lists
    if (pos >= e1 || m >= nm) return;
    const long e = MB >= 64 ? (long)__builtin_amdgcn_readfirstlane(M.celem[pos]) : (long)M.celem[pos];
    const long ne = M.ne;
    double gL[4][3];
#pragma unroll
    for (int k = 0; k < 12; ++k) gL[k / 3][k % 3] = M.geo64[k * ne + e];
    const double vol = M.geo64[12 * ne + e];
    const int l = M.layer[e];
    const double rho = matv(mat, l, MAT_RHO, MB, m);
    double he = 0.0;
    if (sc.damping_mode == 0 && h) he = h[e * MB + m];
    else if (sc.damping_mode == 1) he = sc.h0;
    const double dt = sc.dt;
    const double sm = rho * vol * (4.0 / (dt * dt) + 2.0 * sc.ahat * he / dt);
    const double w = (1.0 + 2.0 * sc.bhat * he / dt) * vol * 0.25;
    double blk[4][6];
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int k = 0; k < 6; ++k) blk[i][k] = 0.0;
    const int EB = MB >= 64 ? 1 : 64 / MB;
#pragma unroll 1
    for (int j = 0; j < 4; ++j) {
        double C[6][6];  // C[cd][pq]
        {
            double d[21];
            const double* Dj = D + d_index(e, j, 0, MB, EB, 0);  // uniform when MB >= 64
            const uint32_t rs = (uint32_t)(EB * MB);
#pragma unroll
            for (int k = 0; k < 21; ++k) d[k] = ld_u(Dj, (uint32_t)k * rs + (uint32_t)m);
            diag_coef<0, 6>(d, C);
        }
        double L[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) L[i] = (i == j) ? QA_ : QB_;
        if (part == 0) {
#pragma unroll
            for (int i = 0; i < 4; ++i) diag_node_add<6>(i, L, gL, C, w, blk[i]);
        } else if (part == 1) {
#pragma unroll
            for (int i = 0; i < 3; ++i) diag_node_add<6>(4 + i, L, gL, C, w, blk[i]);
        } else {
#pragma unroll
            for (int i = 0; i < 3; ++i) diag_node_add<6>(7 + i, L, gL, C, w, blk[i]);
        }
    }
    const int nn = part == 0 ? 4 : 3, n0 = part == 0 ? 0 : 1 + 3 * part;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        if (i >= nn) break;
        const int n = n0 + i;
        const long node = M.conn[n * ne + e];
        const double md = sm * mass_ref(n, n);
        double* dg = diag + node * 6 * MB;
#pragma unroll
        for (int k = 0; k < 6; ++k) {
            double& o = *reinterpret_cast<double*>(reinterpret_cast<char*>(dg) + (uint32_t)(k * MB + m) * 8u);
            o += blk[i][k] + ((k == 0 || k == 3 || k == 5) ? md : 0.0);
        }
    }
}

// The inner operator's blocks (one D per element) by colours, one lane per
// element-member.
__global__ __launch_bounds__(256) void k_diag_mean(DevMesh M, int MB, int nm, int e0, int e1,
                                                  const uint32_t* __restrict__ D16, const double* __restrict__ h,
                                                  const double* __restrict__ mat, StepConst sc,
                                                  double* __restrict__ diag)
{
    const long t = blockIdx.x * (long)blockDim.x + threadIdx.x;
    const int m = (int)(t % MB);
    long r = t / MB;
    if (MB >= 64) r = __builtin_amdgcn_readfirstlane((int)r);
    const long pos = e0 + r;
    if (pos >= e1 || m >= nm) return;
    const long e = MB >= 64 ? (long)__builtin_amdgcn_readfirstlane(M.celem[pos]) : (long)M.celem[pos];
    const long ne = M.ne;
    double gL[4][3];
#pragma unroll
    for (int k = 0; k < 12; ++k) gL[k / 3][k % 3] = M.geo64[k * ne + e];
    const double vol = M.geo64[12 * ne + e];
    const int l = M.layer[e];
    const double rho = matv(mat, l, MAT_RHO, MB, m);
    double he = 0.0;
    if (sc.damping_mode == 0 && h) he = h[e * MB + m];
    else if (sc.damping_mode == 1) he = sc.h0;
    const double dt = sc.dt;
    const double sm = rho * vol * (4.0 / (dt * dt) + 2.0 * sc.ahat * he / dt);
    const double sk = (1.0 + 2.0 * sc.bhat * he / dt) * vol;
    const int EB = MB >= 64 ? 1 : 64 / MB;
    double C[6][6];
    {
        double d[22];
#pragma unroll
        for (int q = 0; q < 11; ++q) {
            const uint32_t wv = D16[d16m_index(e, q, MB, EB, m)];
            d[2 * q] = (double)bf2f(wv & 0xFFFFu);
            d[2 * q + 1] = (double)bf2f(wv >> 16);
        }
        diag_coef<0, 6>(d, C);
    }
#pragma unroll
    for (int n = 0; n < 10; ++n) {
        double G[6];
        mean_grad_products(n, gL, G);
        const long node = M.conn[n * ne + e];
        const double md = sm * mass_ref(n, n);
        double* dg = diag + node * 6 * MB;
#pragma unroll
        for (int cd = 0; cd < 6; ++cd) {
            double a = 0.0;
#pragma unroll
            for (int pq = 0; pq < 6; ++pq) a += G[pq] * C[cd][pq];
            double& o = *reinterpret_cast<double*>(reinterpret_cast<char*>(dg) + (uint32_t)(cd * MB + m) * 8u);
            o += sk * a + ((cd == 0 || cd == 3 || cd == 5) ? md : 0.0);
        }
    }
}

void launch_diag_mean(hipStream_t s, const DevMesh& M, int MB, int nm, int e0, int e1, const uint32_t* D16,
                      const double* h, const double* mat, StepConst sc, double* diag)
{
    const long n = (long)(e1 - e0) * MB;
    if (n > 0) hipLaunchKernelGGL(k_diag_mean, dim3(nblocks(n)), dim3(256), 0, s, M, MB, nm, e0, e1, D16, h, mat, sc, diag);
}

void launch_diag(hipStream_t s, const DevMesh& M, int MB, int nm, int e0, int e1, const double* D, const double* h,
                 const double* mat, int, StepConst sc, double* diag)
{
    long n = (long)(e1 - e0) * 3 * MB;
    if (n > 0) hipLaunchKernelGGL(k_diag, dim3(nblocks(n)), dim3(256), 0, s, M, MB, nm, e0, e1, D, h, mat, sc, diag);
}

// the dashpot's part of the diagonal block of boundary node i
__device__ __forceinline__ void dashpot_diag(const DevMesh& M, int MB, int m, long i, const double* __restrict__ mat,
                                             double coef, double acc[6])
{
    for (int k = 0; k < 6; ++k) acc[k] = 0.0;
    for (int q = M.bn_ptr[i]; q < M.bn_ptr[i + 1]; ++q) {
        const int f = M.bn_face[q], a = M.bn_loc[q];
        const int l = M.f_layer[f];
        const double rho = matv(mat, l, MAT_RHO, MB, m);
        const double vs = matv(mat, l, MAT_VS, MB, m);
        const double vp = matv(mat, l, MAT_VP, MB, m);
        const double* n = M.f_n + 3 * (long)f;
        const double Maa = M.f_M[36 * (long)f + 7 * a] * coef * rho;
        acc[0] += Maa * (vs + (vp - vs) * n[0] * n[0]);
        acc[1] += Maa * ((vp - vs) * n[0] * n[1]);
        acc[2] += Maa * ((vp - vs) * n[0] * n[2]);
        acc[3] += Maa * (vs + (vp - vs) * n[1] * n[1]);
        acc[4] += Maa * ((vp - vs) * n[1] * n[2]);
        acc[5] += Maa * (vs + (vp - vs) * n[2] * n[2]);
    }
}

__global__ void k_diag_dashpot(DevMesh M, int MB, int nm, const double* __restrict__ mat, double coef,
                               double* __restrict__ diag)
{
    const long t = blockIdx.x * (long)blockDim.x + threadIdx.x;
    const int m = (int)(t % MB);
    const long i = t / MB;
    if (i >= M.nbn || m >= nm) return;
    const long node = M.bn_node[i];
    double acc[6];
    dashpot_diag(M, MB, m, i, mat, coef, acc);
    for (int k = 0; k < 6; ++k) diag[(node * 6 + k) * MB + m] += acc[k];
}

void launch_diag_dashpot(hipStream_t s, const DevMesh& M, int MB, int nm, const double* mat, int, double coef,
                         double* diag)
{
    long n = (long)M.nbn * MB;
    if (n > 0) hipLaunchKernelGGL(k_diag_dashpot, dim3(nblocks(n)), dim3(256), 0, s, M, MB, nm, mat, coef, diag);
}

// pinv of node i: the inverse of its block a = [a0 a1 a2; a1 a3 a4; a2 a4 a5]
__device__ __forceinline__ void invert_block(const double a[6], long i, int MB, int m, double* __restrict__ pinv,
                                             float* __restrict__ pinv32)
{
    const double c00 = a[3] * a[5] - a[4] * a[4];
    const double c01 = a[2] * a[4] - a[1] * a[5];
    const double c02 = a[1] * a[4] - a[2] * a[3];
    const double c11 = a[0] * a[5] - a[2] * a[2];
    const double c12 = a[1] * a[2] - a[0] * a[4];
    const double c22 = a[0] * a[3] - a[1] * a[1];
    const double det = a[0] * c00 + a[1] * c01 + a[2] * c02;
    double inv[6] = {0, 0, 0, 0, 0, 0};
    if (det != 0.0) {
        const double r = 1.0 / det;
        inv[0] = c00 * r; inv[1] = c01 * r; inv[2] = c02 * r;
        inv[3] = c11 * r; inv[4] = c12 * r; inv[5] = c22 * r;
    }
#pragma unroll
    for (int k = 0; k < 6; ++k) {
        pinv[(i * 6 + k) * MB + m] = inv[k];
        if (pinv32) pinv32[(i * 6 + k) * MB + m] = (float)inv[k];
    }
}

__global__ void k_invert_diag(int nn, int MB, int nm, const double* __restrict__ diag,
                              double* __restrict__ pinv, float* __restrict__ pinv32)
{
    const long t = blockIdx.x * (long)blockDim.x + threadIdx.x;
    const int m = (int)(t % MB);
    const long i = t / MB;
    if (i >= nn || m >= nm) return;
    double a[6];
#pragma unroll
    for (int k = 0; k < 6; ++k) a[k] = diag[(i * 6 + k) * MB + m];
    invert_block(a, i, MB, m, pinv, pinv32);
}

void launch_invert_diag(hipStream_t s, int nn, int MB, int nm, const double* diag, double* pinv, float* pinv32)
{
    long n = (long)nn * MB;
    if (n > 0) hipLaunchKernelGGL(k_invert_diag, dim3(nblocks(n)), dim3(256), 0, s, nn, MB, nm, diag, pinv, pinv32);
}

// Node sums of the rows of k_diag_slots: half 0 writes its three entries of the
// diagonal blocks; half 1 has the other three in registers, adds the dashpot's
// part at boundary nodes, writes them and the inverse.
template <int HALF>
__global__ __launch_bounds__(256) void k_diag_rows(DevMesh M, int MB, int nm, const double* __restrict__ rows,
                                                  const double* __restrict__ mat, double coef,
                                                  double* __restrict__ diag, double* __restrict__ pinv,
                                                  float* __restrict__ pinv32)
{
    const long t = blockIdx.x * 256l + threadIdx.x;
    const int m = (int)(t % MB);
    const long nd = t / MB;
    if (nd >= M.nn || m >= nm) return;
    const long node = MB >= 64 ? (long)__builtin_amdgcn_readfirstlane((int)nd) : nd;
    double* dg = diag + node * 6 * MB + m;
    double s[3];
    if constexpr (HALF == 0) {
        node_rows<double>(M, node, rows, MB, m, false, s);
#pragma unroll
        for (int c = 0; c < 3; ++c) dg[(size_t)c * MB] = s[c];
    } else {
        double a[6];
#pragma unroll
        for (int c = 0; c < 3; ++c) a[c] = dg[(size_t)c * MB];
        node_rows<double>(M, node, rows, MB, m, false, s);
#pragma unroll
        for (int c = 0; c < 3; ++c) a[3 + c] = s[c];
        const int i = M.bn_of_node[node];
        if (i >= 0) {
            double b[6];
            dashpot_diag(M, MB, m, i, mat, coef, b);
#pragma unroll
            for (int k = 0; k < 6; ++k) a[k] += b[k];
#pragma unroll
            for (int c = 0; c < 3; ++c) dg[(size_t)c * MB] = a[c];
        }
#pragma unroll
        for (int c = 3; c < 6; ++c) dg[(size_t)c * MB] = a[c];
        invert_block(a, node, MB, m, pinv, pinv32);
    }
}

void launch_diag_rows(hipStream_t s, const DevMesh& M, int MB, int nm, int half, const double* rows, const double* mat,
                      double coef, double* diag, double* pinv, float* pinv32)
{
    const dim3 g(nblocks((long)M.nn * MB)), b(256);
    if (half == 0) hipLaunchKernelGGL((k_diag_rows<0>), g, b, 0, s, M, MB, nm, rows, mat, coef, diag, pinv, pinv32);
    else hipLaunchKernelGGL((k_diag_rows<1>), g, b, 0, s, M, MB, nm, rows, mat, coef, diag, pinv, pinv32);
}

// ---------------------------------------------------------------------------
// multi-spring law (Section 2.1): modified Ramberg-Osgood skeleton + Masing
// ---------------------------------------------------------------------------

// normalised skeleton inverse: s with s (1 + |2s|^beta) = e.  Newton in FP32
// (hardware log2/exp2 and reciprocal) from the upper bound
// min(|e|, (|e| / 2^beta)^(1/(1+beta))), on which the iteration decreases
// monotonically, then in FP64 until the step is below 2^-44 |s|.  The FP64
// power is evaluated once, p0 = (2 s0)^beta at the FP32 root s0, and at the
// later iterates s = s0 (1 + d) as p0 (1 + d)^beta from its series, which is
// exact to rounding for |d| < 1e-4 (the FP32 root is good to ~1e-7).  The FP64
// steps divide by the derivative at s0 (a chord step: it differs from the
// derivative at s by ~1e-7 relative, so each step still squares the error to
// rounding; two steps in the usual case).  *pw receives |2s|^beta at the last
// FP64 iterate.
__device__ __forceinline__ float pow2s_f32(float s, float beta)
{
    return __builtin_amdgcn_exp2f(beta * __builtin_amdgcn_logf(2.0f * s));
}

__device__ __forceinline__ double pow2s_f64(double s, double beta) { return exp2(beta * log2(2.0 * s)); }

// 1/x in FP64 from the FP32 hardware reciprocal (1 ulp) and one Newton step:
// relative error ~1e-14 for x within the FP32 normal range
__device__ __forceinline__ double rcp_refined(double x)
{
    const double r = (double)__builtin_amdgcn_rcpf((float)x);
    return r * fma(-x, r, 2.0);
}

// (2 s)^beta for 2 s > 0 in the FP64 normal range, without the library's
// special-case handling and extra-precise argument: log2 of the mantissa
// reduced to [sqrt(1/2), sqrt(2)) from the series
// ln m = 2 (f + f^3/3 + f^5/5 + ...), f = (m - 1)/(m + 1), |f| < 0.172,
// to f^21; 2^y as 2^n e^t, n = rint(y), |t| <= ln2/2, from the Taylor series
// of e^t to t^12.  Relative error below 1e-14 while |beta log2(2 s)| < 60.
// a constant materialised in scalar registers where it is used: keeps the
// compiler from hoisting the series coefficients below out of the spring loop
// into vector registers (38 of them, which then spill)
__device__ __forceinline__ double sconst(double c)
{
    asm volatile("" : "+s"(c));
    return c;
}

__device__ __forceinline__ double pow2s_fast(double s, double beta)
{
    const double x = 2.0 * s;
    double m = __builtin_amdgcn_frexp_mant(x);  // [0.5, 1)
    int ex = __builtin_amdgcn_frexp_exp(x);
    if (m < sconst(0.70710678118654752)) {
        m *= 2.0;
        --ex;
    }
    const double f = (m - 1.0) * rcp_refined(m + 1.0), f2 = f * f;
    double q = sconst(1.0 / 21);
    q = fma(q, f2, sconst(1.0 / 19));
    q = fma(q, f2, sconst(1.0 / 17));
    q = fma(q, f2, sconst(1.0 / 15));
    q = fma(q, f2, sconst(1.0 / 13));
    q = fma(q, f2, sconst(1.0 / 11));
    q = fma(q, f2, sconst(1.0 / 9));
    q = fma(q, f2, sconst(1.0 / 7));
    q = fma(q, f2, sconst(1.0 / 5));
    q = fma(q, f2, sconst(1.0 / 3));
    const double lnm = 2.0 * f * fma(q, f2, 1.0);
    const double y = beta * fma(lnm, sconst(1.4426950408889634), (double)ex);
    const double n = __builtin_rint(y), t = (y - n) * sconst(0.69314718055994531);
    double r = sconst(1.0 / 479001600.0);  // 1/12!
    r = fma(r, t, sconst(1.0 / 39916800.0));
    r = fma(r, t, sconst(1.0 / 3628800.0));
    r = fma(r, t, sconst(1.0 / 362880.0));
    r = fma(r, t, sconst(1.0 / 40320.0));
    r = fma(r, t, sconst(1.0 / 5040.0));
    r = fma(r, t, sconst(1.0 / 720.0));
    r = fma(r, t, sconst(1.0 / 120.0));
    r = fma(r, t, sconst(1.0 / 24.0));
    r = fma(r, t, sconst(1.0 / 6.0));
    r = fma(r, t, sconst(0.5));
    r = fma(r, t, 1.0);
    r = fma(r, t, 1.0);
    return __builtin_amdgcn_ldexp(r, (int)n);
}

__device__ __forceinline__ double ro_inverse_pw(double e, double beta, double* pw)
{
    const double a = fabs(e);
    if (!(a >= 1e-30)) {  // (2a)^beta < 1e-27: s = a to FP64 precision
        *pw = a == 0.0 ? 0.0 : pow2s_f64(a, beta);
        return e;
    }
    const float af = (float)a, bf = (float)beta, bp1f = 1.0f + bf;
    float sf = fminf(af, __builtin_amdgcn_exp2f((__builtin_amdgcn_logf(af) - bf) * __builtin_amdgcn_rcpf(bp1f)));
#pragma unroll 1
    for (int it = 0; it < 12; ++it) {
        const float p = pow2s_f32(sf, bf);
        const float f = sf * (1.0f + p) - af;
        if (f <= 0.0f) break;
        const float ds = f * __builtin_amdgcn_rcpf(fmaf(bp1f, p, 1.0f));
        sf -= ds;
        if (ds <= 1e-7f * sf) break;
    }
    const double c1 = beta, c2 = 0.5 * beta * (beta - 1.0), c3 = c2 * (beta - 2.0) * (1.0 / 3.0);
    double s = (double)sf, s0 = 0.0, p0 = 0.0, r0 = 0.0, rd = 0.0, p = 0.0;
    bool fresh = true;  // take the power afresh at the current iterate
#pragma unroll 1
    for (int it = 0; it < 60; ++it) {
        if (fresh) {
            s0 = s;
            p0 = p = pow2s_fast(s0, beta);
            r0 = rcp_refined(s0);
            rd = rcp_refined(fma(1.0 + beta, p0, 1.0));
        }
        const double ds = fma(s, 1.0 + p, -a) * rd;
        s -= ds;
        const double d = (s - s0) * r0;
        fresh = !(fabs(d) < 1e-4);  // far from the FP32 root (its iteration cap)
        if (!fresh) {
            p = p0 * fma(d, fma(d, fma(d, c3, c2), c1), 1.0);
            if (fabs(ds) <= 0x1p-44 * s) break;
        }
    }
    *pw = p;
    return e < 0 ? -s : s;
}

struct SpringPar { double G0, gref, hmax, beta; };

// Law state of a chunk of ecp elements (ecp a multiple of EB): four FP64
// fields (gp, gr, tr, sm: the strain, the reversal strain and stress, and the
// normalised skeleton stress at the largest strain reached on the skeleton)
// then one int32 field packing the loading direction,
// the skeleton flag and the count of older reversal points kept,
// (dir + 1) | skel << 2 | count << 3 (36 B per spring and point); with a
// reversal memory of depth K > 1 the int32 field is followed by 2 (K - 1)
// FP64 fields, the older points' (gr, tr) pairs, oldest first (36 + 16 (K - 1)
// B).  Within a field: element blocks of EB, then spring, point,
// element-in-block, member.
__device__ __forceinline__ int theta_flags(int dir, int skel) { return (dir + 1) | (skel << 2); }

struct ThetaView {
    double* d;
    int* i;
    double* od;    // older reversal points: gr of point k at od[2k * field_n], tr at od[(2k + 1) * field_n]
    long field_n;  // entries per field = ecp * 4 * ns * MB
    int ns, MB, EB;
    __device__ __forceinline__ long at(long el, int s, int j, int m) const
    {
        return (((el / EB) * ns + s) * 4 + j) * (long)EB * MB * 1 + (el % EB) * MB + m;
    }
};

__device__ __forceinline__ ThetaView theta_view(void* base, long ecp, int ns, int MB)
{
    ThetaView v;
    v.field_n = ecp * 4 * (long)ns * MB;
    v.d = (double*)base;
    v.i = (int*)(v.d + 4 * v.field_n);
    v.od = (double*)(v.i + v.field_n);  // field_n is a multiple of 4: 8-byte aligned
    v.ns = ns;
    v.MB = MB;
    v.EB = MB >= 64 ? 1 : 64 / MB;
    return v;
}

__global__ void k_theta_init(void* base, long ecp, int ns, int MB)
{
    ThetaView v = theta_view(base, ecp, ns, MB);
    const long i = blockIdx.x * (long)blockDim.x + threadIdx.x;
    if (i >= v.field_n) return;
    for (int f = 0; f < 4; ++f) v.d[f * v.field_n + i] = 0.0;
    v.i[i] = theta_flags(0, 1);  // no loading yet, on the skeleton
}

void launch_theta_init(hipStream_t s, void* base, long ecp, int ns, int MB)
{
    long n = ecp * 4 * (long)ns * MB;
    if (n > 0) hipLaunchKernelGGL(k_theta_init, dim3(nblocks(n)), dim3(256), 0, s, base, ecp, ns, MB);
}

// write D of point j in FP64 and in the inner operator's storage (FP32 or
// bfloat16 pairs, whichever is allocated)
__device__ __forceinline__ void store_D(const double d[21], long e, int j, int MB, int EB, int m,
                                        double* __restrict__ D, float* __restrict__ D32, uint32_t* __restrict__ D16)
{
#pragma unroll
    for (int k = 0; k < 21; ++k) {
        const long idx = d_index(e, j, k, MB, EB, m);
        D[idx] = d[k];
        if (D32) D32[idx] = (float)d[k];
    }
    if (D16) {
#pragma unroll
        for (int q = 0; q < 11; ++q) {
            const uint32_t lo = f2bf(d[2 * q]);
            const uint32_t hi = (2 * q + 1 < 21) ? f2bf(d[2 * q + 1]) : 0u;
            D16[d16_index(e, j, q, MB, EB, m)] = lo | (hi << 16);
        }
    }
}

// D of a point from the spring tangents: Kb m m^T + sum c_k G_k n_k n_k^T
__global__ void k_law_init(DevMesh M, int MB, int nm, const double* __restrict__ mat, int ns,
                           const double* __restrict__ dirs, const double* __restrict__ w,
                           double* __restrict__ D, float* __restrict__ D32, uint32_t* __restrict__ D16,
                           double* __restrict__ h, int only_m, bool d16_mean)
{
    const long t = blockIdx.x * (long)blockDim.x + threadIdx.x;
    const int m = only_m >= 0 ? only_m : (int)(t % MB);
    const long e = only_m >= 0 ? t : t / MB;
    if (e >= M.ne || m >= nm) return;
    const int EB = MB >= 64 ? 1 : 64 / MB;
    const int l = M.layer[e];
    const double G0 = matv(mat, l, MAT_G0, MB, m), Kb = matv(mat, l, MAT_KB, MB, m);
    double d[21];
    for (int k = 0; k < 21; ++k) d[k] = 0;
    for (int s = 0; s < ns; ++s) {
        const double* n = dirs + 6 * s;
        const double c = w[s] * G0;
        for (int r = 0; r < 6; ++r)
            for (int q = r; q < 6; ++q) d[sym6(r, q)] += c * n[r] * n[q];
    }
    for (int r = 0; r < 3; ++r)
        for (int q = r; q < 3; ++q) d[sym6(r, q)] += Kb;
    for (int j = 0; j < 4; ++j) store_D(d, e, j, MB, EB, m, D, D32, d16_mean ? nullptr : D16);
    if (d16_mean && D16)
        for (int q = 0; q < 11; ++q)
            D16[d16m_index(e, q, MB, EB, m)] = f2bf(d[2 * q]) | ((2 * q + 1 < 21 ? f2bf(d[2 * q + 1]) : 0u) << 16);
    h[e * MB + m] = 0.0;
}

void launch_law_init(hipStream_t s, const DevMesh& M, int MB, int nm, const double* mat, int, int ns,
                     const double* dirs, const double* w, double* D, float* D32, uint32_t* D16, double* h,
                     int only_m, bool d16_mean)
{
    long n = only_m >= 0 ? (long)M.ne : (long)M.ne * MB;
    if (n > 0)
        hipLaunchKernelGGL(k_law_init, dim3(nblocks(n)), dim3(256), 0, s, M, MB, nm, mat, ns, dirs, w, D, D32, D16, h,
                           only_m, d16_mean);
}

// reset the law state of one member (serving: a new request takes the slot)
__global__ void k_theta_reset_member(void* base, long ecp, int ns, int MB, int m)
{
    ThetaView v = theta_view(base, ecp, ns, MB);
    const long n = ecp * 4 * (long)ns;  // (element, spring, point) triples
    const long t = blockIdx.x * (long)blockDim.x + threadIdx.x;
    if (t >= n) return;
    const long el = t / (4L * ns);
    const int s = (int)((t / 4) % ns), j = (int)(t % 4);
    const long idx = v.at(el, s, j, m);
    for (int f = 0; f < 4; ++f) v.d[f * v.field_n + idx] = 0.0;
    v.i[idx] = theta_flags(0, 1);
}

void launch_theta_reset_member(hipStream_t s, void* base, long ecp, int ns, int MB, int m)
{
    long n = ecp * 4 * (long)ns;
    if (n > 0) hipLaunchKernelGGL(k_theta_reset_member, dim3(nblocks(n)), dim3(256), 0, s, base, ecp, ns, MB, m);
}

// zero column m of a member-innermost array with `rows` rows
__global__ void k_zero_member(double* p, long rows, int MB, int m)
{
    const long r = blockIdx.x * (long)blockDim.x + threadIdx.x;
    if (r < rows) p[r * MB + m] = 0.0;
}

void launch_zero_member(hipStream_t s, double* p, long rows, int MB, int m)
{
    if (rows > 0) hipLaunchKernelGGL(k_zero_member, dim3(nblocks(rows)), dim3(256), 0, s, p, rows, MB, m);
}

// One lane per (element, point, member) of the chunk [e0, e0 + ec), the four
// points of an element-member in adjacent lanes: strain increment at the point
// from du, then every spring's Masing/RO update and tangent,
// D = Kb m m^T + sum c_k G_t n n^T at the point, and the element damping h
// (the mean over the four points, summed across the four lanes).
// WAVE_ELEM: a wavefront covers one element (MB >= 16): its geometry and
// connectivity are then wave-uniform and live in scalar registers.
// LDS_NS > 0 (at most that many springs): each lane parks its springs' c_k G_k
// in LDS during the spring loop and forms D after it, so the 21 FP64
// accumulators of D are not live across the skeleton inversions: 139
// registers instead of 178 (3 wavefronts per SIMD instead of 2), and with the
// launch bound of 4 wavefronts per SIMD 128 registers and 36 B of spills
// (4 % faster again); 0: D accumulated in registers.
// MEM: a reversal memory of `depth` > 1 points (inner loops close, as the
// oracle's law with that depth); false: the three-rule law.
// PARTS > 1 (many springs, few lanes): a block's PARTS wavefronts take the same 64
// lanes and a share of the springs each; the first sums their D and damping.
// The law is bound by issue (about 1,500 cycles of a SIMD a spring and wavefront:
// two springs ahead or a third wavefront a SIMD change nothing), so this pays only
// while SIMDs idle: 150 springs on 12,288 elements (768 wavefronts) 300 -> 249 us,
// on 360 (23) 272 -> 70 with 8 parts, on 331,776 elements 3.8 -> 5.0 ms.
constexpr int kLawLdsSprings = 16;
constexpr long kLawPartLanes = 1l << 16;  // a wavefront a SIMD without parts
constexpr long kLawManyParts = 1l << 14;
template <bool WAVE_ELEM, int LDS_NS, bool MEM, int PARTS>
__global__ __launch_bounds__(PARTS == 8 ? 512 : 256, LDS_NS > 0 ? 4 : 1) void k_law(DevMesh M, int MB, int nm, int e0, int ec, long ecp,
                                            const double* __restrict__ mat, const int* __restrict__ nonlinear,
                                            int ns, int depth, const double* __restrict__ dirs,
                                            const double* __restrict__ w, const double* __restrict__ du,
                                            void* theta, double* __restrict__ D, float* __restrict__ D32,
                                            uint32_t* __restrict__ D16, double* __restrict__ h,
                                            const int* __restrict__ stepping, bool d16_mean)
{
    const int part = PARTS > 1 ? (int)threadIdx.x >> 6 : 0;
    const long t = PARTS > 1 ? blockIdx.x * 64l + (threadIdx.x & 63) : blockIdx.x * (long)blockDim.x + threadIdx.x;
    const int j = (int)(t & 3);
    const long q = t >> 2;
    const int m = (int)(q % MB);
    long el = q / MB;
    // (lanes that leave here leave in every wavefront of the block)
    if (WAVE_ELEM) el = __builtin_amdgcn_readfirstlane((int)el);
    if (el >= ec || m >= nm) return;
    if (stepping && !stepping[m]) return;
    const long e = e0 + el;
    const long ne = M.ne;
    const int l = M.layer[e];
    if (!nonlinear[l]) return;
    const int EB = MB >= 64 ? 1 : 64 / MB;
    SpringPar P;
    P.G0 = matv(mat, l, MAT_G0, MB, m);
    P.gref = matv(mat, l, MAT_GREF, MB, m);
    P.hmax = matv(mat, l, MAT_HMAX, MB, m);
    P.beta = matv(mat, l, MAT_BETA, MB, m);
    const double Kb = matv(mat, l, MAT_KB, MB, m);
    const double rgref = 1.0 / P.gref;
    // strain increment at point j, node by node (gradient of N_n at the point
    // times the node's increment)
    double ej[6] = {0.0, 0.0, 0.0, 0.0, 0.0, 0.0};
    {
        double gL[4][3];
#pragma unroll
        for (int k = 0; k < 12; ++k) gL[k / 3][k % 3] = M.geo64[k * ne + e];
        double L[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) L[i] = (i == j) ? QA_ : QB_;
        constexpr int E[6][2] = {{0, 1}, {1, 2}, {2, 0}, {0, 3}, {1, 3}, {2, 3}};
#pragma unroll
        for (int n = 0; n < 10; ++n) {
            const long node = M.conn[n * ne + e];
            const double* un = du + node * 3 * MB + m;
            const double u0 = un[0], u1 = un[MB], u2 = un[2 * MB];
            double g[3];
#pragma unroll
            for (int a = 0; a < 3; ++a)
                g[a] = n < 4 ? (4.0 * L[n] - 1.0) * gL[n][a]
                             : 4.0 * (L[E[n - 4][0]] * gL[E[n - 4][1]][a] + L[E[n - 4][1]] * gL[E[n - 4][0]][a]);
            ej[0] += g[0] * u0;
            ej[1] += g[1] * u1;
            ej[2] += g[2] * u2;
            ej[3] += g[1] * u0 + g[0] * u1;
            ej[4] += g[2] * u1 + g[1] * u2;
            ej[5] += g[0] * u2 + g[2] * u0;
        }
    }
    ThetaView th = theta_view(theta, ecp, ns, MB);
    const long fn = th.field_n;
    __shared__ double cgs[LDS_NS > 0 ? LDS_NS * 256 : 1];
    if (LDS_NS > 0) {
        // each spring's strain increment waits in its LDS slot (the slot takes
        // c_k G_k after the update), so the strain is not live across the loop
#pragma unroll 1
        for (int sp = 0; sp < ns; ++sp) {
            const double* n = dirs + 6 * sp;
            cgs[sp * 256 + threadIdx.x] =
                n[0] * ej[0] + n[1] * ej[1] + n[2] * ej[2] + n[3] * ej[3] + n[4] * ej[4] + n[5] * ej[5];
        }
    }
    double d[21];
#pragma unroll
    for (int k = 0; k < 21; ++k) d[k] = 0;
    double hs = 0.0;
    // the next spring's state is loaded while this one is updated
    const int sp0 = part * ns / PARTS, sp1 = (part + 1) * ns / PARTS;
    long nidx = th.at(el, sp0, j, m);
    double ngp = th.d[nidx], ngr = th.d[fn + nidx], ntr = th.d[2 * fn + nidx], nsm = th.d[3 * fn + nidx];
    int nfl = th.i[nidx];
#pragma unroll 1
    for (int sp = sp0; sp < sp1; ++sp) {
        const double* n = dirs + 6 * sp;
        const double dg = LDS_NS > 0 ? cgs[sp * 256 + threadIdx.x]
                                     : n[0] * ej[0] + n[1] * ej[1] + n[2] * ej[2] + n[3] * ej[3] + n[4] * ej[4] +
                                           n[5] * ej[5];
        const long idx = nidx;
        double gp = ngp, gr = ngr, tr = ntr, sm = nsm;
        int dir = (nfl & 3) - 1, skel = (nfl >> 2) & 1;
        int cnt = MEM ? nfl >> 3 : 0;  // older reversal points kept
        if (sp + 1 < sp1) {
            nidx = th.at(el, sp + 1, j, m);
            ngp = th.d[nidx]; ngr = th.d[fn + nidx]; ntr = th.d[2 * fn + nidx]; nsm = th.d[3 * fn + nidx];
            nfl = th.i[nidx];
        }
        const int dsg = dg > 0.0 ? 1 : (dg < 0.0 ? -1 : 0);
        const bool reverse = dsg != 0 && dir != 0 && dsg != dir;
        // largest strain reached on the skeleton: |gp| while on it; off it, from
        // the stored normalised skeleton stress sm through the explicit forward
        // relation gm = gref sm (1 + pm), pm = (2 sm)^beta, whose power also
        // gives the damping of an off-skeleton spring
        double pm = 0.0, gm = fabs(gp);
        if ((!skel || reverse) && sm > 0.0) {
            pm = pow2s_fast(sm, P.beta);
            if (!skel) gm = P.gref * sm * (1.0 + pm);
        }
        bool rev2 = false;     // reversal on a branch: the skeleton inverted at rev_arg
        double rev_arg = 0.0;
        if (dsg != 0) {
            if (reverse) {  // a Masing branch starts here
                double trev = 0.0;
                if (skel) {
                    // the skeleton stress at gp = +-gm is +-sm (stored by the last update on the skeleton)
                    trev = P.G0 * P.gref * copysign(sm, gp);
                } else {
                    rev_arg = 0.5 * (gp - gr);
                    if (MEM) {
                        double pk;
                        trev = tr + 2.0 * P.G0 * P.gref * ro_inverse_pw(rev_arg * rgref, P.beta, &pk);
                    } else {
                        rev2 = true;
                    }
                }
                if (MEM) {
                    // the origin of the branch being left is kept (the oldest dropped when
                    // full); a closed loop below may replace the new branch
                    if (!skel) {
                        if (cnt == depth - 1) {
                            for (int k = 0; k + 1 < cnt; ++k) {
                                th.od[(2 * k) * fn + idx] = th.od[(2 * k + 2) * fn + idx];
                                th.od[(2 * k + 1) * fn + idx] = th.od[(2 * k + 3) * fn + idx];
                            }
                            --cnt;
                        }
                        th.od[(2 * cnt) * fn + idx] = gr;
                        th.od[(2 * cnt + 1) * fn + idx] = tr;
                        ++cnt;
                    }
                }
                if (!rev2) tr = trev;
                gr = gp;
                skel = 0;
            }
            dir = dsg;
            const double g = gp + dg;
            if (!skel && (double)dsg * g >= gm) {  // rejoin the skeleton
                skel = 1;
                cnt = 0;
            }
            if (MEM) {  // closed inner loops: on along the branch before the previous one
                while (!skel && cnt >= 2 && (double)dsg * g >= (double)dsg * th.od[(2 * cnt - 2) * fn + idx]) {
                    gr = th.od[(2 * cnt - 4) * fn + idx];
                    tr = th.od[(2 * cnt - 3) * fn + idx];
                    cnt -= 2;
                }
            }
            gp = g;
        }
        const double xi = skel ? gp : 0.5 * (gp - gr);
        // the inversions through one copy of the solver: a branch reversal's, then xi's
        double s_rev = 0.0, s_xi = 0.0, pw = 0.0;
#pragma unroll 1
        for (int k = 0; k < 2; ++k) {
            if (k == 0 && !rev2) continue;
            double pk;
            const double sv = ro_inverse_pw((k == 0 ? rev_arg : xi) * rgref, P.beta, &pk);
            if (k == 0) s_rev = sv;
            else { s_xi = sv; pw = pk; }
        }
        if (rev2) tr += 2.0 * P.G0 * P.gref * s_rev;
        if (skel) sm = fabs(s_xi);  // on the skeleton gm = |gp|
        if (dsg != 0) {
            th.d[idx] = gp; th.d[fn + idx] = gr; th.d[2 * fn + idx] = tr; th.d[3 * fn + idx] = sm;
            th.i[idx] = theta_flags(dir, skel) | (cnt << 3);
        }
        const double Gt = P.G0 / (1.0 + (1.0 + P.beta) * pw);
        // damping 1 - S(em)/em at em = gm/gref: with em = s (1 + (2s)^beta) at s = S(em)
        // it is p/(1 + p), p the power at the skeleton stress of the largest strain
        const double ph = skel ? pw : pm;
        const double hk = P.hmax * ph / (1.0 + ph);
        hs += hk;
        const double c = w[sp] * Gt;
        if (LDS_NS > 0) {
            cgs[sp * 256 + threadIdx.x] = c;
        } else {
#pragma unroll
            for (int r = 0; r < 6; ++r)
#pragma unroll
                for (int qq = r; qq < 6; ++qq) d[sym6(r, qq)] += c * n[r] * n[qq];
        }
    }
    if (LDS_NS > 0) {
#pragma unroll 1
        for (int sp = 0; sp < ns; ++sp) {
            const double* n = dirs + 6 * sp;
            const double c = cgs[sp * 256 + threadIdx.x];
#pragma unroll
            for (int r = 0; r < 6; ++r)
#pragma unroll
                for (int qq = r; qq < 6; ++qq) d[sym6(r, qq)] += c * n[r] * n[qq];
        }
    }
    if constexpr (PARTS > 1) {
        __shared__ double ps[PARTS - 1][22][64];
        const int lane = threadIdx.x & 63;
        if (part > 0) {
#pragma unroll
            for (int k = 0; k < 21; ++k) ps[part - 1][k][lane] = d[k];
            ps[part - 1][21][lane] = hs;
        }
        __syncthreads();
        if (part > 0) return;
#pragma unroll
        for (int p = 0; p < PARTS - 1; ++p) {
#pragma unroll
            for (int k = 0; k < 21; ++k) d[k] += ps[p][k][lane];
            hs += ps[p][21][lane];
        }
    }
#pragma unroll
    for (int r = 0; r < 3; ++r)
#pragma unroll
        for (int qq = r; qq < 3; ++qq) d[sym6(r, qq)] += Kb;
    store_D(d, e, j, MB, EB, m, D, D32, d16_mean ? nullptr : D16);
    if (d16_mean && D16) {  // element-mean D of the inner operator (the four point lanes)
#pragma unroll
        for (int k = 0; k < 21; ++k) {
            d[k] += __shfl_xor(d[k], 1);
            d[k] += __shfl_xor(d[k], 2);
        }
        if (j == 0)
#pragma unroll
            for (int q = 0; q < 11; ++q)
                D16[d16m_index(e, q, MB, EB, m)] =
                    f2bf(0.25 * d[2 * q]) | ((2 * q + 1 < 21 ? f2bf(0.25 * d[2 * q + 1]) : 0u) << 16);
    }
    // element damping: mean over the 4 points (adjacent lanes) and the springs
    double hsum = hs / ns;
    hsum += __shfl_xor(hsum, 1);
    hsum += __shfl_xor(hsum, 2);
    if (j == 0) h[e * MB + m] = 0.25 * hsum;
}

template <int LDS_NS, bool MEM, int PARTS>
static void law_dispatch(hipStream_t s, long n, const DevMesh& M, int MB, int nm, int e0, int ec, long ecp,
                         const double* mat, const int* nonlinear, int ns, int depth, const double* dirs,
                         const double* w, const double* du, void* theta, double* D, float* D32, uint32_t* D16,
                         double* h, const int* stepping, bool d16_mean)
{
    const dim3 g(PARTS > 1 ? (unsigned)((n + 63) / 64) : nblocks(n));
    if (MB >= 16)
        hipLaunchKernelGGL((k_law<true, LDS_NS, MEM, PARTS>), g, dim3(PARTS > 1 ? 64 * PARTS : 256), 0, s, M, MB, nm, e0, ec, ecp, mat, nonlinear, ns,
                           depth, dirs, w, du, theta, D, D32, D16, h, stepping, d16_mean);
    else
        hipLaunchKernelGGL((k_law<false, LDS_NS, MEM, PARTS>), g, dim3(PARTS > 1 ? 64 * PARTS : 256), 0, s, M, MB, nm, e0, ec, ecp, mat, nonlinear, ns,
                           depth, dirs, w, du, theta, D, D32, D16, h, stepping, d16_mean);
}

void launch_law(hipStream_t s, const DevMesh& M, int MB, int nm, int e0, int ec, long ecp, const double* mat, int,
                const int* nonlinear, int ns, int depth, const double* dirs, const double* w, const double* du,
                void* theta, double* D, float* D32, uint32_t* D16, double* h, const int* stepping, bool d16_mean)
{
    long n = (long)ec * MB * 4;
    if (n <= 0) return;
    const bool small = ns <= kLawLdsSprings, mem = depth > 1;
    // by the whole mesh, not the chunk: a paged run sums the springs as the resident one
    const long all = (long)M.ne * MB * 4;
    const int parts = all <= kLawManyParts ? 8 : (all <= kLawPartLanes ? 4 : 1);
#define NLTH_LAW(LDS_NS, MEM, PARTS)                                                                                 \
    law_dispatch<LDS_NS, MEM, PARTS>(s, n, M, MB, nm, e0, ec, ecp, mat, nonlinear, ns, depth, dirs, w, du, theta, D, \
                                     D32, D16, h, stepping, d16_mean)
    if (small && !mem) NLTH_LAW(kLawLdsSprings, false, 1);
    else if (small) NLTH_LAW(kLawLdsSprings, true, 1);
    else if (!mem && parts == 8) NLTH_LAW(0, false, 8);
    else if (!mem && parts == 4) NLTH_LAW(0, false, 4);
    else if (!mem) NLTH_LAW(0, false, 1);
    else if (parts == 8) NLTH_LAW(0, true, 8);
    else if (parts == 4) NLTH_LAW(0, true, 4);
    else NLTH_LAW(0, true, 1);
#undef NLTH_LAW
}

// ---------------------------------------------------------------------------
// Newmark state updates (Section 2.1), receivers, incident wave
// ---------------------------------------------------------------------------

__global__ void k_newmark(long n, int MB, int nm, const double* __restrict__ du, double* __restrict__ u,
                          double* __restrict__ v, double* __restrict__ a, double dt, const int* __restrict__ stepping)
{
    const long i = blockIdx.x * (long)blockDim.x + threadIdx.x;
    const int m = (int)(i % MB);
    if (i >= n || m >= nm || !stepping[m]) return;
    const double d = du[i], vo = v[i];
    u[i] += d;
    a[i] = -a[i] - 4.0 / dt * vo + 4.0 / (dt * dt) * d;
    v[i] = -vo + 2.0 / dt * d;
}

void launch_newmark(hipStream_t s, long n, int MB, int nm, const double* du, double* u, double* v, double* a,
                    double dt, const int* stepping)
{
    long N = n * MB;
    hipLaunchKernelGGL(k_newmark, dim3(nblocks(N)), dim3(256), 0, s, N, MB, nm, du, u, v, a, dt, stepping);
}

// Initial guess of the step's CG from the increments of the previous steps
// (du holds du^{n-1}, d2 du^{n-2}, d3 du^{n-3}; zero before a member's first
// steps, which is its true history from rest), extrapolated by a polynomial
// of degree `order` in time: 0 keeps du^{n-1}, 1 gives 2 du^{n-1} - du^{n-2},
// 2 gives 3 du^{n-1} - 3 du^{n-2} + du^{n-3}.  The history shifts every step
// whatever the order.
__global__ void k_predict(long n, int MB, int nm, int order, double* __restrict__ du, double* __restrict__ d2,
                          double* __restrict__ d3, const int* __restrict__ stepping)
{
    const long i = blockIdx.x * (long)blockDim.x + threadIdx.x;
    const int m = (int)(i % MB);
    if (i >= n || m >= nm || !stepping[m]) return;
    const double a = du[i], b = d2[i], c = d3[i];
    d3[i] = b;
    d2[i] = a;
    if (order == 1) du[i] = 2.0 * a - b;
    else if (order == 2) du[i] = 3.0 * (a - b) + c;
}

void launch_predict(hipStream_t s, long n, int MB, int nm, int order, double* du, double* d2, double* d3,
                    const int* stepping)
{
    const long N = n * MB;
    hipLaunchKernelGGL(k_predict, dim3(nblocks(N)), dim3(256), 0, s, N, MB, nm, order, du, d2, d3, stepping);
}

__global__ void k_receivers(int nrecv, const int* __restrict__ recv, int MB, int nm, const double* __restrict__ v,
                            double* __restrict__ hist, const int* __restrict__ member_step, int ns,
                            double* __restrict__ vmax, const int* __restrict__ stepping)
{
    const long t = blockIdx.x * (long)blockDim.x + threadIdx.x;
    const int m = (int)(t % MB);
    const long r = t / MB;
    if (r >= nrecv || m >= nm || !stepping[m]) return;
    const long node = recv[r];
    const int step = member_step[m];
    double nrm = 0.0;
    for (int c = 0; c < 3; ++c) {
        const double val = v[(node * 3 + c) * MB + m];
        hist[(((long)m * ns + step) * nrecv + r) * 3 + c] = val;
        nrm += val * val;
    }
    nrm = sqrt(nrm);
    const long vi = (long)m * nrecv + r;
    if (nrm > vmax[vi]) vmax[vi] = nrm;
}

void launch_receivers(hipStream_t s, int nrecv, const int* recv, int MB, int nm, const double* v, double* hist,
                      const int* member_step, int ns, double* vmax, const int* stepping)
{
    long n = (long)nrecv * MB;
    if (n > 0)
        hipLaunchKernelGGL(k_receivers, dim3(nblocks(n)), dim3(256), 0, s, nrecv, recv, MB, nm, v, hist, member_step,
                           ns, vmax, stepping);
}

// Incident velocity by the trapezoid rule from the incident acceleration (zero at
// t = 0): one block per member, a wavefront a component, samples added one after
// another (sums of runs of the record made a velocity depend on the record's
// length).  Bound by that chain of FP64 additions: the lanes load the next 64 samples
// while the terms of 64 are added in registers, from LDS and back (2,048 samples:
// a load a step took 379 us, terms by lane reads 50; this 44).
__global__ __launch_bounds__(192) void k_incident_velocity(int ns, const double* __restrict__ acc,
                                                          double* __restrict__ vI, double dt)
{
    const int c = threadIdx.x >> 6, lane = threadIdx.x & 63;
    const size_t base = (size_t)blockIdx.x * ns * 3 + c;
    __shared__ __align__(16) double tiles[3][64];
    double* tile = tiles[c];  // of the wavefront
    auto fence = [] { __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront"); };
    double v = 0.0, ap, an;
    auto load = [&](int n) {  // past the end any sample: its sum is not stored
        n = min(n, ns - 1);
        ap = acc[base + (size_t)max(n - 1, 0) * 3];
        an = acc[base + (size_t)n * 3];
    };
    load(lane);
    for (int n = lane; n - lane < ns; n += 64) {
        tile[lane] = (n > 0 ? ap : 0.0) + an;
        load(n + 64);
        fence();
        double x[64];
#pragma unroll
        for (int k = 0; k < 64; ++k) x[k] = tile[k];
#pragma unroll
        for (int k = 0; k < 64; ++k) {
            v += 0.5 * dt * x[k];
            x[k] = v;
        }
        fence();
        if (lane == 0)
#pragma unroll
            for (int k = 0; k < 64; ++k) tile[k] = x[k];
        fence();
        if (n < ns) vI[base + (size_t)n * 3] = tile[lane];
        fence();
    }
}

void launch_incident_velocity(hipStream_t s, int, int nm, int ns, const double* acc, double* vI, double dt)
{
    hipLaunchKernelGGL(k_incident_velocity, dim3(nm), dim3(192), 0, s, ns, acc, vI, dt);
}

// incident velocity of each member at its current step, member-innermost [3][MB]
__global__ void k_pick_vI(int MB, int nm, int ns, const double* __restrict__ vI_all, const int* __restrict__ member_step,
                          double* __restrict__ vI_cur)
{
    const int t = blockIdx.x * blockDim.x + threadIdx.x;
    if (t >= MB * 3) return;
    const int m = t % MB, c = t / MB;
    double v = 0.0;
    if (m < nm) {
        const int st = member_step[m];
        if (st >= 0 && st < ns) v = vI_all[((long)m * ns + st) * 3 + c];
    }
    vI_cur[c * MB + m] = v;
}

void launch_pick_vI(hipStream_t s, int MB, int nm, int ns, const double* vI_all, const int* member_step,
                    double* vI_cur)
{
    hipLaunchKernelGGL(k_pick_vI, dim3(nblocks(MB * 3)), dim3(256), 0, s, MB, nm, ns, vI_all, member_step, vI_cur);
}

__global__ void k_record_iters(int MB, int nm, int ns, const int* __restrict__ member_step,
                               const int* __restrict__ stepping, const int* __restrict__ iters,
                               const int* __restrict__ inner_total, int* __restrict__ out)
{
    const int m = blockIdx.x * blockDim.x + threadIdx.x;
    if (m >= nm || !stepping[m]) return;
    const int st = member_step[m];
    if (st < 0 || st >= ns) return;
    out[((long)m * ns + st) * 2] = iters[m];
    out[((long)m * ns + st) * 2 + 1] = inner_total[m];
}

void launch_record_iters(hipStream_t s, int MB, int nm, int ns, const int* member_step, const int* stepping,
                         const int* iters, const int* inner_total, int* out)
{
    hipLaunchKernelGGL(k_record_iters, dim3(nblocks(MB)), dim3(256), 0, s, MB, nm, ns, member_step, stepping, iters,
                       inner_total, out);
}

}  // namespace nlth
