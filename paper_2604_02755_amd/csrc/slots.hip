// Element-by-element operator of ensembles with few member slots (fewer than
// 64), of the compact rows of the convergence tail, and of the single-member
// application: Section 2.2, Eq. 1 and 2.
//
// A wavefront of the wide kernels (kernels.hip) covers one element and 64
// members.  With fewer slots its lanes hold different elements, so nothing is
// wave-uniform, the nodal loads scatter, and a small mesh leaves the chip
// nearly empty: what counts then is the number of round trips to memory in a
// block's chain and the number of launches, and on a large mesh the bytes of
// the intermediate sums.
#include "device.hpp"

namespace nlth {

// Sums of a cluster row's incidences: its list groups p0..p1 in LDS,
// out[(3 * node + component) * OS + pair].  Lists are padded to groups of four
// with the entry of rows of zeros, so all loads of a group are issued together:
// an entry at a time, with a test, was a chain of 48 LDS round trips at a vertex.
template <typename T>
__device__ __forceinline__ void row_sums(const uint2* __restrict__ lists, int p0, int p1, const T* __restrict__ out,
                                         int OS, int lg, int mm, T s[3])
{
    s[0] = s[1] = s[2] = 0;
    uint2 w = lists[p0];
    for (int p = p0; p < p1; ++p) {
        const uint2 wn = lists[p + 1];  // (one group past the row: the next row's, or the rows' pointers)
        const uint32_t en[4] = {w.x & 0xFFFFu, w.x >> 16, w.y & 0xFFFFu, w.y >> 16};
        T v[4][3];
#pragma unroll
        for (int q = 0; q < 4; ++q)
#pragma unroll
            for (int c = 0; c < 3; ++c) v[q][c] = out[((en[q] >> 6) * 3 + c) * OS + ((en[q] & 63u) << lg) + mm];
#pragma unroll
        for (int q = 0; q < 4; ++q)
#pragma unroll
            for (int c = 0; c < 3; ++c) s[c] += v[q][c];
        w = wn;
    }
}

// per-member sums of the threads' values (a thread's are all of member t % MB)
// to partial[m], in a fixed order: the lanes of a wavefront by
// exchanges, then the wavefronts one after another (a tree over the block with
// a barrier a level took 0.9 us of a block's 8)
__device__ __forceinline__ void slot_partials(double dot, int MB, double* __restrict__ sh, double* __restrict__ partial)
{
    const int t = threadIdx.x, nw = blockDim.x >> 6;
    for (int o = 32; o >= MB; o >>= 1) dot += __shfl_xor(dot, o);
    __syncthreads();
    if ((t & 63) < MB) sh[(t >> 6) * MB + (t & 63)] = dot;
    __syncthreads();
    if (t < MB) {
        double a = 0.0;
        for (int w = 0; w < nw; ++w) a += sh[w * MB + t];
        partial[t] = a;
    }
}

// Shape of the kernel for 1 << LG member lanes: up to 8 slots the wide clusters
// (64 elements: a block then has 64 to 512 lanes of work and 2.6 rows go out per
// element), the regular ones (12 elements, 3.75 rows) with 16 and 32, whose
// nodal values would not fit the LDS otherwise.
template <typename T, int LG>
struct SlotShape {
    static constexpr bool WIDE = (1 << LG) <= kWideSlots;
    static constexpr int ELEMS = WIDE ? kWideElems : kClusterElems, NODES = WIDE ? kWideNodes : kClusterNodes;
    static constexpr int PAIRS = ELEMS << LG, OS = PAIRS + 4;  // element-members; stride of the LDS rows
    static constexpr int XS = NODES << LG;                      // staged values of a component
    // nodal values staged in LDS, where a wavefront's lanes read 32 or 64
    // scattered addresses otherwise (1 slot 19.7 -> 16.1 us below; from 4 slots on
    // the staging cost more than it saved)
    static constexpr bool STAGE = LG <= 1;
    // least threads: a wavefront or two more than the pairs fill, for the row sums
    // (331,776 elements, FP32, 1 slot: 64 threads 39 us, 128 33, 256 46;
    // 98,304 elements, 16 slots: 192 threads 92 us, 256 86, 320 146)
    static constexpr int THREADS = LG == 0 ? 128 : (LG < 4 ? 64 << LG : 16 << LG);
    static_assert(LG > 1 || (THREADS == kLagThreads && (ELEMS << LG) <= THREADS), "k_op_p and k_pz sum in one order");
};

// DK 2, doubles of a staged D row in LDS: 16 bytes more than the row, so the lanes'
// reads spread over all banks
constexpr int kInputRow = 86;

// One block per element cluster, one lane per element-member: forces of all its
// element-members to LDS, summed there per node row over the cluster's
// incidence lists (a fixed order), the rows out for the gather.  Blocks after
// the clusters write the dashpot rows of the boundary nodes.  MB / L groups
// of L = 1 << LG members.  tl (may be NULL): compact
// rows, lane k is member tl[1 + k].  partial (may be NULL): the per-member sums
// of x1 . (operator x1) over the block's rows.  The tables of a cluster (nodes,
// lists) lie at fixed strides, so a block's chain of dependent loads is
// tables -> values and element data -> LDS -> rows; one trip is about 0.9 us
// (2200 cycles: what another kernel has just written comes from beyond the L2).
// Bound: instruction issue (about 1200 a wavefront) on large meshes, that chain
// on small ones.  Operator with its node sums and the dashpot on 98,304
// elements, against element outputs to memory, a gather of ten per element and
// a dashpot kernel: FP32 with bfloat16 element-mean D 1 slot 45 -> 23 us, 8 slots
// 89 -> 60, 32 slots 250 -> 197; FP64 1 slot 59 -> 38, 8 slots 226 -> 183, 32 slots
// 808 -> 675.  Four lanes per element-member, one per integration point, had a
// shorter chain but 1.5 times the instructions: no faster on small meshes, 124
// against 45 us (FP32, without the sums) at 8 slots.
// PF (1 and 2 slots): the p update of the CG iteration before joins the staging of
// p: every block forms the beta stage and p_new of its own nodes, and the first
// cluster of a node writes it with the x update (owner rows: kOwnerRow).
template <typename T, int DK, int MODE, int LG, bool PF = false>
__device__ __forceinline__ void op_slots_block(const DevMesh& M, int MB, int nm, int ncb, int nbb,
                                               const int* __restrict__ tl, const void* __restrict__ Dv,
                                               const int* __restrict__ order, const double* __restrict__ h,
                                               const double* __restrict__ mat, const StepConst& sc,
                                               const T* __restrict__ x1, const T* __restrict__ x2, T* __restrict__ rows,
                                               const int* __restrict__ active, double dcoef,
                                               const double* __restrict__ vI, double* __restrict__ partial,
                                               const PUpdate<T>* pu = nullptr)
{
    using S = SlotShape<T, LG>;
    constexpr int L = 1 << LG, OS = S::OS, XS = S::XS;
    constexpr bool STAGE = S::STAGE && MODE != OP_RHS;
    constexpr bool DIN = DK == 2 && MODE != OP_M;  // D rows staged where `out` comes later
    extern __shared__ __align__(16) char smem[];
    const int t = threadIdx.x, NT = blockDim.x;
    if (tl) nm = min(tl[0], MB);
    double dot = 0.0;
    const int blk = (int)blockIdx.x, g = blk / ncb * L, cb = blk % ncb;  // first member of the group; cluster block
    const int c = (cb % 8) * (ncb / 8) + cb / 8;                        // XCD-contiguous clusters
    const int ncl_blocks = ncb * (MB / L);
    bool on_m = false;  // PF: this lane's member iterates
    T be = 0, al = 0;
    bool upd = false;
    // PF: z, p and x of the rows that this thread stages, under way while the sums are formed
    constexpr int RP = (S::NODES + (S::THREADS >> LG) - 1) / (S::THREADS >> LG);
    T zr[PF ? RP : 1][3], pr[PF ? RP : 1][3], xr[PF ? RP : 1][3];
    size_t ir[PF ? RP : 1];
    bool own[PF ? RP : 1];
    if constexpr (PF) {
        constexpr bool INNER = sizeof(T) == 4;
        __shared__ double ps[2 * S::THREADS / 64 * L];  // (the block has S::THREADS: at most 64 elements of L lanes)
        __shared__ double pb[L];
        __shared__ int pon[L];
        const int mt = t & (L - 1);
        if (blk < ncl_blocks && c < M.ncl) {
            const int ncn = M.cl_head[c].w;
#pragma unroll
            for (int q = 0; q < RP; ++q) {
                const int lr = (t >> LG) + q * (NT >> LG);
                own[q] = false;
                if (lr >= ncn) continue;
                ir[q] = (size_t)M.cl_nodes[(size_t)c * M.cl_node_stride + lr] * 3 * MB + mt;
                own[q] = M.cl_lptr[(size_t)c * M.cl_node_stride + lr] & kOwnerRow;
#pragma unroll
                for (int cc = 0; cc < 3; ++cc) {
                    zr[q][cc] = pu->z[ir[q] + (size_t)cc * MB];
                    pr[q][cc] = x1[ir[q] + (size_t)cc * MB];
                    if (own[q]) xr[q][cc] = pu->x[ir[q] + (size_t)cc * MB];
                }
            }
        }
        const BetaState<INNER> bs(pu->sg.cs, MB, nm);
        double S2[2];
        member_sums<2, kLagThreads>(pu->sg.partial, pu->sg.nblk, MB, ps, S2);
        if (t < MB) {
            bool on;
            pb[t] = fused_beta<INNER>(pu->sg, t, S2, bs.upd, bs.rz_prev, bs.it, bs.ref, MB, blk == 0, on);
            pon[t] = (int)on | ((int)bs.upd << 1);
        }
        __syncthreads();
        on_m = pon[mt] & 1;
        upd = pon[mt] & 2;
        be = (T)pb[mt];
        al = upd ? (T)pu->alpha[mt] : (T)0;
    }
    auto lane_on = [&](int mm) { return PF ? on_m : mm < nm && (!active || active[mm]); };
    if (blk >= ncl_blocks) {
        dot = boundary_rows<T>(M, MB, nm, mat, dcoef,
                               [&](size_t n) { return PF ? pu->z[n] + be * x1[n] : x1[n]; }, vI, lane_on(t % MB),
                               rows + (size_t)M.cl_rows * 3 * MB, blk - ncl_blocks, nbb, NT);
        if (partial) slot_partials(dot, MB, (double*)smem, partial + (size_t)(ncb + blk - ncl_blocks) * MB);
        return;
    }
    if (c < M.ncl) {
        T* out = (T*)smem;  // [33][OS], the last three rows zeros
        T* xs = out + (DIN ? S::ELEMS * kInputRow : 33 * OS);  // [3][XS]
        uint2* lists = (uint2*)(xs + (STAGE ? 3 * XS : 0));
        uint16_t* lptr = (uint16_t*)(lists + M.cl_list_stride);
        int* nds = (int*)(lptr + 256);
        const int4 ch = M.cl_head[c];
        const int e0 = ch.x, r0 = ch.y, nec = ch.z, ncn = ch.w;
        const int slot = t >> LG, lane = t & (L - 1), m = g + lane;
        if constexpr (PF) {
#pragma unroll
            for (int q = 0; q < RP; ++q) {
                const int lr = slot + q * (NT >> LG);
                if (lr >= ncn) continue;
#pragma unroll
                for (int cc = 0; cc < 3; ++cc) {
                    const T pn = zr[q][cc] + be * pr[q][cc];
                    xs[cc * XS + (lr << LG) + lane] = pn;
                    if (own[q] && upd) {
                        pu->p_new[ir[q] + (size_t)cc * MB] = pn;
                        pu->x[ir[q] + (size_t)cc * MB] = xr[q][cc] + al * pr[q][cc];
                    }
                }
            }
        } else if constexpr (STAGE) {
            // the member lanes of a row read its node's three values
            for (int lr = slot; lr < ncn; lr += NT >> LG) {
                const size_t x0 = (size_t)M.cl_nodes[(size_t)c * M.cl_node_stride + lr] * 3 * MB + m;
#pragma unroll
                for (int cc = 0; cc < 3; ++cc) xs[cc * XS + (lr << LG) + lane] = x1[x0 + (size_t)cc * MB];
            }
        } else {
            for (int i = t; i < ncn; i += NT) nds[i] = M.cl_nodes[(size_t)c * M.cl_node_stride + i];
        }
        const uint4* lsrc = (const uint4*)(M.cl_lists + (size_t)c * M.cl_list_stride);
        for (int i = t; 2 * i < M.cl_list_stride; i += NT) ((uint4*)lists)[i] = lsrc[i];
        for (int i = t; i < M.cl_node_stride; i += NT) lptr[i] = M.cl_lptr[(size_t)c * M.cl_node_stride + i] & ~kOwnerRow;
        if constexpr (DIN) {
            const double* Di = (const double*)Dv;
            const bool wide = ((uintptr_t)Di & 15) == 0;  // (rows of 672 bytes)
            constexpr int Q = 11;
            for (int u0 = t; u0 < nec * 42; u0 += Q * NT) {
                double v[Q][2];
#pragma unroll
                for (int q = 0; q < Q; ++q) {
                    const int u = min(u0 + q * NT, nec * 42 - 1), r = u / 42;
                    const double* p = Di + (size_t)order[e0 + r] * 84 + (u - 42 * r) * 2;
                    if (wide) {
                        const double2 w = *(const double2*)p;
                        v[q][0] = w.x, v[q][1] = w.y;
                    } else {
                        v[q][0] = p[0], v[q][1] = p[1];
                    }
                }
#pragma unroll
                for (int q = 0; q < Q; ++q) {
                    const int u = u0 + q * NT, r = u / 42;
                    if (u < nec * 42) *(double2*)((double*)smem + r * kInputRow + (u - 42 * r) * 2) = make_double2(v[q][0], v[q][1]);
                }
            }
        } else {
            for (int i = t; i < 3 * OS; i += NT) out[30 * OS + i] = (T)0;
        }
        const bool act = m < nm && lane_on(m), on = slot < nec && act;
        const int e = e0 + (slot < nec ? slot : 0);
        const T* geo = geo_of<T>(M);
        T gL[4][3];
#pragma unroll
        for (int k = 0; k < 12; ++k) gL[k / 3][k % 3] = geo[(size_t)k * M.ne + e];
        const T vol = geo[(size_t)12 * M.ne + e];
        const double rho = MODE == OP_K ? 0.0 : matv(mat, M.layer[e], MAT_RHO, MB, m);
        double he = 0.0;
        if (sc.damping_mode == 0 && h) he = h[DK == 2 ? (size_t)order[e] : (size_t)e * MB + m];
        else if (sc.damping_mode == 1) he = sc.h0;
        T sm, sk, cv = 0;
        op_scales<T, MODE>(sc, rho, (double)vol, he, sm, sk, cv);
        // D in blocks of 64 (element, member) pairs; DK 2: rows staged in LDS
        constexpr int W = DK == 4 ? 11 : (DK == 1 ? 44 : 84);
        constexpr size_t B = DK == 0 ? sizeof(T) : 4;
        const size_t pe = (size_t)e * MB;
        const char* Dp = DK == 2 ? smem + (size_t)slot * kInputRow * 8
                                 : (const char*)Dv + ((pe >> 6) * W * 64 + (pe & 63) + m) * B;
        constexpr uint32_t rs = 64;
        T f[10][3];
        if constexpr (STAGE) {
            const uint4 lw = ((const uint4*)M.cl_lconn)[e];
            const uint32_t w[3] = {lw.x, lw.y, lw.z};
            __syncthreads();
            if (on)
                element_forces<T, DK, MODE>(
                    gL, vol, sm, sk, cv, Dp, rs, 0u,
                    [&](int n, int cc, int) { return xs[cc * XS + (int)(((w[n / 4] >> (8 * (n % 4))) & 0xFFu) << LG) + lane]; },
                    f);
        } else if (on) {
            size_t nb[10];
#pragma unroll
            for (int n = 0; n < 10; ++n) nb[n] = (size_t)M.conn[(size_t)n * M.ne + e] * 3 * MB + m;
            element_forces<T, DK, MODE>(
                gL, vol, sm, sk, cv, Dp, rs, 0u,
                [&](int n, int cc, int v) { return (v ? x2 : x1)[nb[n] + (size_t)cc * MB]; }, f);
        }
        // the forces go where other lanes' D rows are
        if constexpr (DIN) __syncthreads();
        if (on) {
#pragma unroll
            for (int n = 0; n < 10; ++n)
#pragma unroll
                for (int cc = 0; cc < 3; ++cc) out[(3 * n + cc) * OS + t] = f[n][cc];
            if (DIN)
#pragma unroll
                for (int cc = 0; cc < 3; ++cc) out[(30 + cc) * OS + t] = (T)0;
        }
        __syncthreads();
        for (int lr = slot; act && lr < ncn; lr += NT >> LG) {
            T s[3], xv[3] = {0, 0, 0};
            if (partial) {  // (under way while the rows are summed)
#pragma unroll
                for (int cc = 0; cc < 3; ++cc)
                    xv[cc] = STAGE ? xs[cc * XS + (lr << LG) + lane] : x1[((size_t)nds[lr] * 3 + cc) * MB + m];
            }
            row_sums<T>(lists, lptr[lr], lptr[lr + 1], out, OS, LG, lane, s);
            T* rp = rows + ((size_t)r0 + lr) * 3 * MB + m;
#pragma unroll
            for (int cc = 0; cc < 3; ++cc) {
                rp[(size_t)cc * MB] = s[cc];
                dot += (double)xv[cc] * (double)s[cc];
            }
        }
    }
    if (partial) slot_partials(dot, L, (double*)smem, partial + (size_t)cb * MB + g);
}

template <typename T, int DK, int MODE, int LG>
__global__ __launch_bounds__(512) void k_op_slots(DevMesh M, int MB, int nm, int ncb, int nbb, const int* __restrict__ tl,
                                                 const void* __restrict__ Dv, const double* __restrict__ h,
                                                 const double* __restrict__ mat, StepConst sc,
                                                 const T* __restrict__ x1, const T* __restrict__ x2,
                                                 T* __restrict__ rows, const int* __restrict__ active, double dcoef,
                                                 const double* __restrict__ vI, double* __restrict__ partial)
{
    op_slots_block<T, DK, MODE, LG>(M, MB, nm, ncb, nbb, tl, Dv, nullptr, h, mat, sc, x1, x2, rows, active, dcoef, vI,
                                    partial);
}

template <typename T, int DK, int LG>
__global__ __launch_bounds__(512) void k_op_p(DevMesh M, int MB, int nm, int ncb, int nbb, const void* __restrict__ Dv,
                                             const double* __restrict__ h, const double* __restrict__ mat, StepConst sc,
                                             const T* __restrict__ p, T* __restrict__ rows, double dcoef,
                                             double* __restrict__ partial, PUpdate<T> pu)
{
    op_slots_block<T, DK, OP_A, LG, true>(M, MB, nm, ncb, nbb, nullptr, Dv, nullptr, h, mat, sc, p, nullptr, rows,
                                          nullptr, dcoef, nullptr, partial, &pu);
}

// One member, D and h in input order, the material table a kernel argument (a
// launch that put it in memory first took 3 us of a call's 30 on 720 elements).
// The block's D rows are staged in LDS, where `out` comes after them: a lane
// reading its own row of 672 bytes fetched every line sixteen times past an L1 that
// does not hold 64 rows (58,080 elements, D in the last-level cache: 36.5 us, staged
// 25.0).
template <int MODE>
__global__ __launch_bounds__(512) void k_op_input64(DevMesh M, int ncb, int nbb, const double* __restrict__ D,
                                                   const int* __restrict__ order, const double* __restrict__ h,
                                                   LayerMat lm, StepConst sc, const double* __restrict__ x,
                                                   double* __restrict__ rows, double dcoef)
{
    op_slots_block<double, 2, MODE, 0>(M, 1, 1, ncb, nbb, nullptr, D, order, h, lm.v, sc, x, nullptr, rows, nullptr,
                                       dcoef, nullptr, nullptr);
}

// threads, blocks and LDS of a launch for MB slots
struct SlotGrid {
    int NT, ncb, nbb;
    size_t lds;
};
template <typename T, int MODE, int LG, bool DIN = false>
static SlotGrid slot_grid(const DevMesh& M, int MB, double dcoef)
{
    using S = SlotShape<T, LG>;
    SlotGrid g;
    g.NT = std::max(S::THREADS, ((M.cl_max_elems << LG) + 63) / 64 * 64);
    g.ncb = (M.ncl + 7) / 8 * 8;
    // boundary nodes per block: up to 8 lanes of a wavefront share a node
    const int parts = 64 / MB < 8 ? 64 / MB : 8, npb = g.NT / (MB * parts);
    const long nb = dcoef != 0.0 ? ((long)M.nbn + npb - 1) / npb : 0;
    g.nbb = (int)(nb < kDashpotBlocks ? nb : kDashpotBlocks);
    g.lds = ((size_t)(DIN ? S::ELEMS * kInputRow : 33 * S::OS) + (S::STAGE && MODE != OP_RHS ? 3 * S::XS : 0)) * sizeof(T);
    g.lds += (size_t)M.cl_list_stride * 8 + 512 + (size_t)M.cl_node_stride * 4;
    return g;
}

template <typename T, int DK, int MODE, int LG>
static void op_launch(hipStream_t s, const DevMesh& M, int MB, int nm, const int* tl, const void* D, const double* h,
                      const double* mat, StepConst sc, const T* x1, const T* x2, T* rows, const int* active,
                      double dcoef, const double* vI, double* partial, int* nblk)
{
    const SlotGrid g = slot_grid<T, MODE, LG>(M, MB, dcoef);
    if (nblk) *nblk = g.ncb + g.nbb;
    hipLaunchKernelGGL((k_op_slots<T, DK, MODE, LG>), dim3(g.ncb * (MB >> LG) + g.nbb), dim3(g.NT), g.lds, s, M, MB, nm,
                       g.ncb, g.nbb, tl, D, h, mat, sc, x1, x2, rows, active, dcoef, vI, partial);
}

template <typename T, int DK, int MODE>
static void op_slots(hipStream_t s, const DevMesh& M, int MB, int nm, const int* tl, const void* D, const double* h,
                     const double* mat, StepConst sc, const T* x1, const T* x2, T* rows, const int* active,
                     double dcoef, const double* vI, double* partial, int* nblk)
{
#define NLTH_LG(LG) \
    op_launch<T, DK, MODE, LG>(s, M, MB, nm, tl, D, h, mat, sc, x1, x2, rows, active, dcoef, vI, partial, nblk)
    switch (MB) {
    case 1: NLTH_LG(0); break;
    case 2: NLTH_LG(1); break;
    case 4: NLTH_LG(2); break;
    case 8: NLTH_LG(3); break;
    case 16: NLTH_LG(4); break;
    case 32:
        // FP64: two groups of 16 lanes (a block of 12 x 32 lanes fills the registers
        // of a CU alone, with nothing to run across its barriers)
        if constexpr (sizeof(T) == 8) NLTH_LG(4);
        else NLTH_LG(5);
        break;
    }
#undef NLTH_LG
}

void launch_op_slots64(hipStream_t s, OpMode mode, const DevMesh& M, int MB, int nm, const double* D,
                       const double* h, const double* mat, StepConst sc, const double* x1, const double* x2,
                       double* rows, const int* active, double dcoef, const double* vI, double* partial, int* nblk)
{
    switch (mode) {
    case OP_A: op_slots<double, 0, OP_A>(s, M, MB, nm, nullptr, D, h, mat, sc, x1, x2, rows, active, dcoef, vI, partial, nblk); break;
    case OP_K: op_slots<double, 0, OP_K>(s, M, MB, nm, nullptr, D, h, mat, sc, x1, x2, rows, active, dcoef, vI, partial, nblk); break;
    case OP_M: op_slots<double, 0, OP_M>(s, M, MB, nm, nullptr, D, h, mat, sc, x1, x2, rows, active, dcoef, vI, partial, nblk); break;
    case OP_RHS: op_slots<double, 0, OP_RHS>(s, M, MB, nm, nullptr, D, h, mat, sc, x1, x2, rows, active, dcoef, vI, partial, nblk); break;
    }
}

void launch_op_slots32(hipStream_t s, const DevMesh& M, int MB, int nm, const float* D32, const uint32_t* D16,
                       bool d16_mean, const double* h, const double* mat, StepConst sc, const float* x, float* rows,
                       const int* active, double dcoef, double* partial, int* nblk)
{
    const float* none = nullptr;
    if (D16 && d16_mean)
        op_slots<float, 4, OP_A>(s, M, MB, nm, nullptr, D16, h, mat, sc, x, none, rows, active, dcoef, nullptr, partial, nblk);
    else if (D16)
        op_slots<float, 1, OP_A>(s, M, MB, nm, nullptr, D16, h, mat, sc, x, none, rows, active, dcoef, nullptr, partial, nblk);
    else
        op_slots<float, 0, OP_A>(s, M, MB, nm, nullptr, D32, h, mat, sc, x, none, rows, active, dcoef, nullptr, partial, nblk);
}

template <typename T, int DK>
static int op_p(hipStream_t s, const DevMesh& M, int MB, int nm, const void* D, const double* h, const double* mat,
                 StepConst sc, const T* p, T* rows, double dcoef, double* partial, const PUpdate<T>& pu)
{
    if (MB == 1) {
        const SlotGrid g = slot_grid<T, OP_A, 0>(M, 1, dcoef);
        hipLaunchKernelGGL((k_op_p<T, DK, 0>), dim3(g.ncb + g.nbb), dim3(g.NT), g.lds, s, M, 1, nm, g.ncb, g.nbb, D, h,
                           mat, sc, p, rows, dcoef, partial, pu);
        return g.ncb + g.nbb;
    }
    const SlotGrid g = slot_grid<T, OP_A, 1>(M, 2, dcoef);
    hipLaunchKernelGGL((k_op_p<T, DK, 1>), dim3(g.ncb + g.nbb), dim3(g.NT), g.lds, s, M, 2, nm, g.ncb, g.nbb, D, h, mat,
                       sc, p, rows, dcoef, partial, pu);
    return g.ncb + g.nbb;
}

int launch_op_p64(hipStream_t s, const DevMesh& M, int MB, int nm, const double* D, const double* h, const double* mat,
                   StepConst sc, const double* p, double* rows, double dcoef, double* partial, const PUpdate<double>& pu)
{
    return op_p<double, 0>(s, M, MB, nm, D, h, mat, sc, p, rows, dcoef, partial, pu);
}

int launch_op_p32(hipStream_t s, const DevMesh& M, int MB, int nm, const float* D32, const uint32_t* D16,
                   bool d16_mean, const double* h, const double* mat, StepConst sc, const float* p, float* rows,
                   double dcoef, double* partial, const PUpdate<float>& pu)
{
    if (D16 && d16_mean) return op_p<float, 4>(s, M, MB, nm, D16, h, mat, sc, p, rows, dcoef, partial, pu);
    if (D16) return op_p<float, 1>(s, M, MB, nm, D16, h, mat, sc, p, rows, dcoef, partial, pu);
    return op_p<float, 0>(s, M, MB, nm, D32, h, mat, sc, p, rows, dcoef, partial, pu);
}

void launch_op_input64(hipStream_t s, OpMode mode, const DevMesh& M, const int* order, const double* D,
                       const double* h, const LayerMat& lm, StepConst sc, const double* x, double* rows, double dcoef)
{
    SlotGrid g = mode == OP_M ? slot_grid<double, OP_A, 0>(M, 1, dcoef) : slot_grid<double, OP_A, 0, true>(M, 1, dcoef);
    g.NT = 256;  // (threads that stage D: 128 took 28.6 us, 256 25)
    const dim3 nb(g.ncb + g.nbb), nt(g.NT);
    switch (mode) {
    case OP_A: hipLaunchKernelGGL((k_op_input64<OP_A>), nb, nt, g.lds, s, M, g.ncb, g.nbb, D, order, h, lm, sc, x, rows, dcoef); break;
    case OP_K: hipLaunchKernelGGL((k_op_input64<OP_K>), nb, nt, g.lds, s, M, g.ncb, g.nbb, D, order, h, lm, sc, x, rows, dcoef); break;
    default: hipLaunchKernelGGL((k_op_input64<OP_M>), nb, nt, g.lds, s, M, g.ncb, g.nbb, D, order, h, lm, sc, x, rows, dcoef); break;
    }
}

// operator A on the compact rows of the convergence tail (G = 16 or 32 lanes)
void launch_ebe64_ctail(hipStream_t s, const DevMesh& M, int G, const int* tl, const double* cD, const double* ch,
                        const double* cmat, StepConst sc, const double* x, double* co, double dcoef, double* partial,
                        int* nblk)
{
    const double* none = nullptr;
    op_slots<double, 0, OP_A>(s, M, G, G, tl, cD, ch, cmat, sc, x, none, co, nullptr, dcoef, nullptr, partial, nblk);
}

void launch_ebe32_ctail(hipStream_t s, const DevMesh& M, int G, const int* tl, const uint32_t* cD, const double* ch,
                        const double* cmat, StepConst sc, const float* x, float* co, double dcoef, double* partial,
                        int* nblk)
{
    const float* none = nullptr;
    op_slots<float, 4, OP_A>(s, M, G, G, tl, cD, ch, cmat, sc, x, none, co, nullptr, dcoef, nullptr, partial, nblk);
}

// The 3x3 block-Jacobi diagonal blocks, three of their six entries (half 0: 00
// 01 02, half 1: 11 12 22) at a time: the block's three values of a node take
// the place of its three forces in the scheme above (one lane per
// element-member, LDS, rows out, node sums by k_diag_rows), for ensembles of up to 256
// slots.  DK 4: one bfloat16 D per element.  Bound by the FP64 D on many
// members, which both halves read (all six entries at once would take 60 doubles
// of LDS a lane and a rows buffer of twice the size).
// Against one launch per element colour adding to the nodes, with the fill, the
// dashpot and the inversion: 12,288 elements, FP64, 1 slot 31 x 22 -> 36 us; 221,184
// elements, element-mean D, 64 slots 33 x 129 us -> 2 x 1,330 and the node sums.
template <int DK, int LG>
__global__ __launch_bounds__(256) void k_diag_slots(DevMesh M, int MB, int nm, int ncb, int half,
                                                   const void* __restrict__ Dv, const double* __restrict__ h,
                                                   const double* __restrict__ mat, StepConst sc,
                                                   double* __restrict__ rows)
{
    using S = SlotShape<double, LG>;
    constexpr int L = 1 << LG, OS = S::OS;
    extern __shared__ __align__(16) char smem[];
    const int t = threadIdx.x, NT = blockDim.x;
    const int blk = (int)blockIdx.x, g = blk / ncb * L, cb = blk % ncb;
    const int c = (cb % 8) * (ncb / 8) + cb / 8;  // XCD-contiguous clusters
    if (c >= M.ncl) return;
    double* out = (double*)smem;  // [33][OS], the last three rows zeros
    uint2* lists = (uint2*)(out + 33 * OS);
    uint16_t* lptr = (uint16_t*)(lists + M.cl_list_stride);
    const int4 ch = M.cl_head[c];
    const int e0 = ch.x, r0 = ch.y, nec = ch.z, ncn = ch.w;
    const int slot = t >> LG, lane = t & (L - 1), m = g + lane;
    const uint4* lsrc = (const uint4*)(M.cl_lists + (size_t)c * M.cl_list_stride);
    for (int i = t; 2 * i < M.cl_list_stride; i += NT) ((uint4*)lists)[i] = lsrc[i];
    for (int i = t; i < M.cl_node_stride; i += NT) lptr[i] = M.cl_lptr[(size_t)c * M.cl_node_stride + i] & ~kOwnerRow;
    for (int i = t; i < 3 * OS; i += NT) out[30 * OS + i] = 0.0;
    const int e = e0 + slot;
    if (slot < nec && m < nm) {
        double gL[4][3];
#pragma unroll
        for (int k = 0; k < 12; ++k) gL[k / 3][k % 3] = M.geo64[(size_t)k * M.ne + e];
        const double vol = M.geo64[(size_t)12 * M.ne + e];
        const double rho = matv(mat, M.layer[e], MAT_RHO, MB, m);
        double he = 0.0;
        if (sc.damping_mode == 0 && h) he = h[(size_t)e * MB + m];
        else if (sc.damping_mode == 1) he = sc.h0;
        const double dt = sc.dt;
        const double sm = rho * vol * (4.0 / (dt * dt) + 2.0 * sc.ahat * he / dt);
        const double sk = (1.0 + 2.0 * sc.bhat * he / dt) * vol;
        const int EB = MB >= 64 ? 1 : 64 / MB;
        double acc[10][3], C[3][6];
#pragma unroll
        for (int n = 0; n < 10; ++n) acc[n][0] = acc[n][1] = acc[n][2] = 0.0;
        if constexpr (DK == 4) {
            double d[22];
#pragma unroll
            for (int q = 0; q < 11; ++q) {
                const uint32_t wv = ((const uint32_t*)Dv)[d16m_index(e, q, MB, EB, m)];
                d[2 * q] = (double)bf2f(wv & 0xFFFFu);
                d[2 * q + 1] = (double)bf2f(wv >> 16);
            }
            if (half) diag_coef<3, 3>(d, C);
            else diag_coef<0, 3>(d, C);
#pragma unroll
            for (int n = 0; n < 10; ++n) {
                double G[6];
                mean_grad_products(n, gL, G);
#pragma unroll
                for (int k = 0; k < 3; ++k) {
                    double a = 0.0;
#pragma unroll
                    for (int pq = 0; pq < 6; ++pq) a += G[pq] * C[k][pq];
                    acc[n][k] = sk * a;
                }
            }
        } else {
#pragma unroll 1
            for (int j = 0; j < 4; ++j) {
                double d[21], lam[4];
                const double* Dj = (const double*)Dv + d_index(e, j, 0, MB, EB, m);
#pragma unroll
                for (int k = 0; k < 21; ++k) d[k] = Dj[(size_t)k * EB * MB];
                if (half) diag_coef<3, 3>(d, C);
                else diag_coef<0, 3>(d, C);
#pragma unroll
                for (int i = 0; i < 4; ++i) lam[i] = (i == j) ? QA_ : QB_;
#pragma unroll
                for (int n = 0; n < 10; ++n) diag_node_add<3>(n, lam, gL, C, 0.25 * sk, acc[n]);
            }
        }
#pragma unroll
        for (int n = 0; n < 10; ++n) {
            const double md = sm * mass_ref(n, n);  // to 00, or 11 and 22
            out[(3 * n) * OS + t] = acc[n][0] + md;
            out[(3 * n + 1) * OS + t] = acc[n][1];
            out[(3 * n + 2) * OS + t] = acc[n][2] + (half ? md : 0.0);
        }
    }
    __syncthreads();
    for (int lr = slot; m < nm && lr < ncn; lr += NT >> LG) {
        double s[3];
        row_sums<double>(lists, lptr[lr], lptr[lr + 1], out, OS, LG, lane, s);
        double* rp = rows + ((size_t)r0 + lr) * 3 * MB + m;
#pragma unroll
        for (int cc = 0; cc < 3; ++cc) rp[(size_t)cc * MB] = s[cc];
    }
}

void launch_diag_slots(hipStream_t s, const DevMesh& M, int MB, int nm, int half, const double* D64,
                       const uint32_t* D16, const double* h, const double* mat, StepConst sc, double* rows)
{
    const int ncb = (M.ncl + 7) / 8 * 8;
    // lanes of a block: the wide clusters' 64 elements with up to 4 members, the
    // regular ones' 16 with 16 (30 doubles of LDS a lane, two blocks of 256 on a CU)
    const int LG = MB >= 16 ? 4 : (MB >= 4 ? 2 : MB - 1);
    const int NT = std::max(LG == 0 ? 128 : 256, ((M.cl_max_elems << LG) + 63) / 64 * 64);
    const size_t tail = (size_t)M.cl_list_stride * 8 + 512;
#define NLTH_DIAG(LGV)                                                                                               \
    do {                                                                                                             \
        const size_t lds = (size_t)33 * SlotShape<double, LGV>::OS * 8 + tail;                                       \
        if (D16) hipLaunchKernelGGL((k_diag_slots<4, LGV>), dim3(ncb * (MB >> LGV)), dim3(NT), lds, s, M, MB, nm, ncb, half, (const void*)D16, h, mat, sc, rows); \
        else hipLaunchKernelGGL((k_diag_slots<0, LGV>), dim3(ncb * (MB >> LGV)), dim3(NT), lds, s, M, MB, nm, ncb, half, (const void*)D64, h, mat, sc, rows); \
    } while (0)
    switch (LG) {
    case 0: NLTH_DIAG(0); break;
    case 1: NLTH_DIAG(1); break;
    case 2: NLTH_DIAG(2); break;
    default: NLTH_DIAG(4); break;
    }
#undef NLTH_DIAG
}

}  // namespace nlth
