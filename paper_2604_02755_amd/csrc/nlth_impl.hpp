// Internal declarations shared by the host runtime and the HIP kernels of
// libnlth.  Layouts (all on the device):
//   member-innermost: every per-member quantity q of node/element/point i is
//   stored at q[i*MB + m] with MB the padded member count, so a wavefront of
//   lanes that share an element but differ in member reads contiguous memory.
//   node vectors   v[(node*3 + c)*MB + m]
//   elements are grouped in blocks of EB = max(1, 64/MB) so that the EB x MB
//   lanes of a wavefront read contiguous memory:
//   D per point    D[(((e/EB)*84 + ip*21 + k)*EB + e%EB)*MB + m]  (upper
//                  triangle of the symmetric 6x6, row by row)
//   element h      h[e*MB + m]
//   law state      per chunk of ecp elements (a multiple of EB): four FP64
//                  fields {gp, gr, tr, gm} then two int32 fields {dir, skel},
//                  each f[((((el/EB)*ns + s)*4 + ip)*EB + el%EB)*MB + m]
//   mesh arrays    conn[k*ne + e], geo[k*ne + e] (k: 12 barycentric-gradient
//                  entries then the volume), in colour-sorted element order.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace nlth {

enum OpMode { OP_A = 0, OP_K = 1, OP_M = 2, OP_RHS = 3 };

constexpr int kMaxPartialBlocks = 2048;   // blocks of a fused vector kernel's partial sums
constexpr int kGatherBlocks = 16384;      // blocks of a node gather with partial sums
constexpr int kDashpotBlocks = 1024;      // most boundary blocks of an operator launch
constexpr int kBoundaryAtEnd = 4096;      // cluster blocks up to which the boundary blocks come last
constexpr int kBoundaryApart = 28672;     // cluster blocks above which FP32 dashpot rows are a launch of their own
constexpr int kClusterNodes = 48;         // most distinct nodes of an element cluster
constexpr int kClusterElems = 16;         // most elements of an element cluster
constexpr int kWideNodes = 240;           // the same of a wide cluster, which ensembles
constexpr int kWideElems = 64;            // of up to
constexpr int kWideSlots = 8;             // member slots use
constexpr uint16_t kOwnerRow = 0x8000;    // in cl_lptr: the row is its node's first
constexpr int kLagBlocks = 512;           // most operator blocks of an iteration whose p update joins the next operator
constexpr int kLagThreads = 128;          // threads of those blocks: what sums the beta stage with 1 and 2 slots
// most partial sums that each block of the next kernel reads itself, and how many
// they are folded to beyond that with 16 and more slots
constexpr int kFuseSums = 3072;
constexpr int kFoldSums = 1024;
constexpr int kFoldBlocks = 256;          // rows to which long partial sums are folded before the finalize
// length (in MB-rows of doubles) of the partial-sum buffer, without the operator's rows
constexpr int kPartialRows = 3 * kMaxPartialBlocks > kGatherBlocks ? 3 * kMaxPartialBlocks : kGatherBlocks;

struct CgScalars {  // per member [MB] device arrays
    double *bb, *rr, *rz, *alpha, *beta, *pAp;
    int *active, *iters, *status, *stepping;  // stepping: member takes part in this step
    int *inner_active, *inner_iters, *inner_total;
    int* inner_upd;  // members whose alpha was formed this iteration (their x, p still update)
    double* rz_prev;  // r.z and the iteration count before this iteration's beta stage
    int* iters_prev;
    double *irz, *ialpha, *ibeta, *ir0;
    double* lz;  // inner CG coefficients: alpha_k at [k * MB + m], beta_k at [(kLanczosMax + k) * MB + m]
};

// input of a stage that an update kernel forms itself: the partial sums' rows, the
// stage's limits and the scalars
struct StageIn {
    const double* partial;
    int nblk;
    double tol2;
    int maxit;
    CgScalars cs;
};

// The p and x updates of an iteration made by the next one's operator (1 and 2
// slots): with the beta stage from `sg`, p_new = z + beta p and x += alpha p
template <typename T>
struct PUpdate {
    const T* z;
    T *p_new, *x;
    const double* alpha;
    StageIn sg;
};

// Per-member material of one layer, member-innermost: mat[(l*MAT_N + field)*MB + m]
enum MatField { MAT_RHO = 0, MAT_G0, MAT_KB, MAT_VS, MAT_VP, MAT_GREF, MAT_HMAX, MAT_BETA, MAT_N };
// the table of one member, passed to the allocation-free application's kernel by value
constexpr int kNoAllocMaxLayers = 32;
struct LayerMat {
    double v[kNoAllocMaxLayers * MAT_N];
};

struct DevMesh {
    int ne, nn;
    const int* conn;      // [10][ne]
    const double* geo64;  // [13][ne]
    const float* geo32;   // [13][ne]
    const int* layer;     // [ne]
    // boundary nodes (node-centric dashpot gather)
    int nbn;
    const int* bn_node;   // [nbn]
    const int* bn_ptr;    // [nbn+1] into entries
    const int* bn_face;   // [entries]
    const int* bn_loc;    // [entries] local index (0..5) of the node in the face
    const int* f_node;    // [nf*6]
    const double* f_M;    // [nf*36] int N_a N_b dA
    const double* f_n;    // [nf*3] unit normal
    const int* f_layer;   // [nf]
    const uint8_t* f_kind;
    const int* celem;     // [ne] storage positions grouped by colour
    const int* bn_of_node;  // [nn] index into bn_node, or -1
    // element clusters: consecutive storage elements with few distinct nodes
    int ncl;
    const int* cl_off;      // [ncl+1] storage positions
    const int* cl_noff;     // [ncl+1] rows of the clusters' node lists
    const uint32_t* cl_lconn; // [ne*4] local nodes of each element, four 8-bit indices per word
    long cl_rows;           // rows of all clusters
    int cl_max_elems;                    // of a cluster
    int cl_node_stride, cl_list_stride;  // of the tables of a cluster
    const int4* cl_head;      // [ncl] first element, first row, elements, rows
    const int* cl_nodes;      // [ncl][cl_node_stride] node of a row
    const uint16_t* cl_lptr;  // [ncl][cl_node_stride] first list group of a row, one past the last row too
    const uint2* cl_lists;    // [ncl][cl_list_stride] incidences of the rows in groups of four: local node * 64
                              // + element within the cluster, ascending, padded with local node 10
    const int* cn_ptr;      // [nn+1] node -> rows
    const int* cn_row;      // ascending per node: cluster rows, then a boundary node's dashpot row cl_rows + i
};

struct StepConst {
    double dt;
    double ahat, bhat;   // Rayleigh fit
    int damping_mode;    // 0 law, 1 const, 2 none
    double h0;
    double m4, a2, b2, c4;  // 4/dt^2, 2 ahat/dt, 2 bhat/dt, 4/dt
    void quotients()
    {
        m4 = 4.0 / (dt * dt);
        a2 = 2.0 * ahat / dt;
        b2 = 2.0 * bhat / dt;
        c4 = 4.0 / dt;
    }
};

// ---- kernel launchers (kernels.hip) ----
void launch_fill(hipStream_t s, double* p, double v, long n);
// n int32 from src to dst (either may be device-mapped host memory)
void launch_copy_i32(hipStream_t s, const int* src, int* dst, int n);
void launch_fill32(hipStream_t s, float* p, float v, long n);
void launch_neg_copy(hipStream_t s, const double* a, double* b, long n);

// element-by-element operator over elements [e0, e1) of the sorted order
template <typename T>
void launch_ebe(hipStream_t s, OpMode mode, const DevMesh& M, int MB, int nm, int e0, int e1,
                const T* D, const double* h, const double* mat, int n_layers, StepConst sc,
                const T* x1, const T* x2, T* y, const int* active);
// y = sum of the node's cluster rows, with bnd also its dashpot row, + bscale *
// base.  MB <= 256.  ymap: storage node -> row of y (NULL: the same).
template <typename T>
void launch_gather(hipStream_t s, const DevMesh& M, int MB, int nm, const T* rows, bool bnd, const T* base, T bscale,
                   T* y, const int* active, const int* ymap = nullptr);
// the same of FP32 rows with the dashpot rows, and the per-member block partials of x . y
void launch_gather_dot(hipStream_t s, const DevMesh& M, int MB, int nm, const float* rows, float* y, const int* active,
                       const float* x, double* partial, int* nblk);
// the node sums q of an operator application with the CG update that needs
// them (UPD_PZ: r -= alpha q, z = P r, partials (r.r, r.z); UPD_XR: r -= alpha q,
// x += alpha p, z = q, partial r.r); G = 0 full rows, 16 or 32 compact rows
enum { UPD_PZ = 0, UPD_XR = 1 };
template <typename T>
void launch_rows_update(hipStream_t s, int kind, const DevMesh& M, int MB, int nm, int G, const int* tl, const T* rows,
                        T* r, T* z, const T* pinv, T* x, const T* p, const double* alpha, const int* active,
                        double* partial, int* nblk, const StageIn* fused = nullptr);
// operator of `mode` for fewer than 64 member slots: cluster rows and (dcoef
// != 0) the dashpot rows dcoef * C_abs x1 (+ 2 C_base vI) of the boundary
// nodes, to `rows`; with partial the per-member block partials of x1 . y
void launch_op_slots64(hipStream_t s, OpMode mode, const DevMesh& M, int MB, int nm, const double* D,
                       const double* h, const double* mat, StepConst sc, const double* x1, const double* x2,
                       double* rows, const int* active, double dcoef, const double* vI, double* partial, int* nblk);
void launch_op_slots32(hipStream_t s, const DevMesh& M, int MB, int nm, const float* D32, const uint32_t* D16,
                       bool d16_mean, const double* h, const double* mat, StepConst sc, const float* x, float* rows,
                       const int* active, double dcoef, double* partial, int* nblk);
// operator A on p_new of `pu` (x1: the old p), MB 1 or 2, p.Ap to partial
int launch_op_p64(hipStream_t s, const DevMesh& M, int MB, int nm, const double* D, const double* h, const double* mat,
                   StepConst sc, const double* p, double* rows, double dcoef, double* partial, const PUpdate<double>& pu);
int launch_op_p32(hipStream_t s, const DevMesh& M, int MB, int nm, const float* D32, const uint32_t* D16,
                   bool d16_mean, const double* h, const double* mat, StepConst sc, const float* p, float* rows,
                   double dcoef, double* partial, const PUpdate<float>& pu);
// one member, D [ne][4][21] and h [ne] in input tet order (order: storage
// position -> input tet): the operator of launch_op_slots64 on them
void launch_op_input64(hipStream_t s, OpMode mode, const DevMesh& M, const int* order, const double* D,
                       const double* h, const LayerMat& lm, StepConst sc, const double* x, double* rows, double dcoef);
// the same for a multiple of 64 slots (up to 256), co the rows
void launch_ebe_cluster64(hipStream_t s, OpMode mode, const DevMesh& M, int MB, int nm, const double* D,
                          const double* h, const double* mat, StepConst sc, const double* x1, const double* x2,
                          double* co, const int* active, double dcoef, const double* vI, double* partial, int* nblk);
void launch_ebe_cluster32(hipStream_t s, const DevMesh& M, int MB, int nm, const float* D32, const uint32_t* D16,
                          bool d16_mean, const double* h, const double* mat, StepConst sc, const float* x, float* co,
                          const int* active, double dcoef, double* partial, int* nblk);
// absorbing-boundary dashpot of the colour form: y += coef * C_abs x (+ 2 C_base vI)
template <typename T>
void launch_dashpot(hipStream_t s, const DevMesh& M, int MB, int nm, const double* mat, T coef, const T* x, T* y,
                    const double* vI, const int* active);
// diagonal 3x3 blocks of A (sym, 6 entries per node) over elements [e0, e1)
void launch_diag(hipStream_t s, const DevMesh& M, int MB, int nm, int e0, int e1, const double* D,
                 const double* h, const double* mat, int n_layers, StepConst sc, double* diag);
// the same from the bfloat16 element-mean D of the inner operator (closed-form integrals)
void launch_diag_mean(hipStream_t s, const DevMesh& M, int MB, int nm, int e0, int e1, const uint32_t* D16,
                      const double* h, const double* mat, StepConst sc, double* diag);
// the same by clusters, three of the six entries at a time, and their node sums
// (half 1: with the dashpot's part and the inverse); D16 not NULL: element means
void launch_diag_slots(hipStream_t s, const DevMesh& M, int MB, int nm, int half, const double* D64,
                       const uint32_t* D16, const double* h, const double* mat, StepConst sc, double* rows);
void launch_diag_rows(hipStream_t s, const DevMesh& M, int MB, int nm, int half, const double* rows, const double* mat,
                      double coef, double* diag, double* pinv, float* pinv32);
void launch_diag_dashpot(hipStream_t s, const DevMesh& M, int MB, int nm, const double* mat, int n_layers,
                         double coef, double* diag);
void launch_invert_diag(hipStream_t s, int nn, int MB, int nm, const double* diag, double* pinv,
                        float* pinv32);

// law
void launch_law_init(hipStream_t s, const DevMesh& M, int MB, int nm, const double* mat, int n_layers,
                     int ns, const double* dirs, const double* w, double* D, float* D32, uint32_t* D16,
                     double* h, int only_m = -1, bool d16_mean = false);
void launch_theta_reset_member(hipStream_t s, void* base, long ecp, int ns, int MB, int m);
void launch_zero_member(hipStream_t s, double* p, long rows, int MB, int m);
// threads per block of the element-by-element launches on this host thread
void set_ebe_block(int bs);
// blocks per CU of the cluster launches on this host thread
void set_cluster_blocks(int b);
// convergence tail: the CG of at most G (16 or 32) listed members on compact
// rows (lane k = member tl[1 + k], tl[0] = the count).  Mixed path: its inner FP32 solve; FP64 path: PCG.
void launch_tail_pack(hipStream_t s, const DevMesh& M, int MB, int G, int n_layers, const int* tl,
                      const uint32_t* D16, const double* h, const double* mat, const float* pinv32, uint32_t* cD,
                      double* ch, double* cmat, float* cpinv);
void launch_tail_unpack(hipStream_t s, long nrows, int MB, int G, const int* tl, const float* c, float* full);
void launch_tail_pack64(hipStream_t s, const DevMesh& M, int MB, int G, int n_layers, const int* tl,
                        const double* D64, const double* h, const double* mat, const double* pinv, double* cD,
                        double* ch, double* cmat, double* cpinv);
// nrows member-innermost FP64 rows, full <-> compact
void launch_tail_rows64(hipStream_t s, long nrows, int MB, int G, const int* tl, const double* src, double* dst,
                        bool unpack);
// operator A on the compact rows (the mixed path's inner operator, or the FP64
// one with D per point): G-wide rows, dashpot rows included, and partials of
// x . (A x) as G-wide rows of the listed members
void launch_ebe32_ctail(hipStream_t s, const DevMesh& M, int G, const int* tl, const uint32_t* cD, const double* ch,
                        const double* cmat, StepConst sc, const float* x, float* co, double dcoef, double* partial,
                        int* nblk);
void launch_ebe64_ctail(hipStream_t s, const DevMesh& M, int G, const int* tl, const double* cD, const double* ch,
                        const double* cmat, StepConst sc, const double* x, double* co, double dcoef, double* partial,
                        int* nblk);
// p = z + beta p on the compact rows
void launch_tail_p_update(hipStream_t s, long nrows, int nm, int G, const int* tl, const double* cz, double* cp,
                          const double* beta, const int* active);
// r_compact: r in the compact rows (the outer CG on compact rows), else full
void launch_tail_start(hipStream_t s, int nn, int MB, int nm, int G, const int* tl, const double* r, bool r_compact,
                       const float* cpinv, float* cir, float* ciz, float* cip, const int* active, double* partial,
                       int* nblk);
// the mixed path's outer flexible CG on the compact rows
void launch_tail_inner_out(hipStream_t s, long nrows, int MB, int nm, int G, const int* tl, const float* ciz,
                           double* cz, const double* cAp, const double* cr, const int* active, double* partial,
                           int* nblk);
// x += alpha p, then p = z + beta p, for the members of upd
template <typename T>
void launch_tail_pz(hipStream_t s, long nrows, int nm, int G, const int* tl, T* cx, T* cp, const T* cz,
                    const double* alpha, const double* beta, const int* upd);
// inner FP32 operator (A) with D in FP32 (D32) or bfloat16 pairs (D16, if non-null)
void launch_ebe32(hipStream_t s, const DevMesh& M, int MB, int nm, int e0, int e1, const float* D32,
                  const uint32_t* D16, const double* h, const double* mat, StepConst sc, const float* x, float* y,
                  const int* active, bool d16_mean);
void launch_theta_init(hipStream_t s, void* theta_chunk, long ecp, int ns, int MB);
void launch_law(hipStream_t s, const DevMesh& M, int MB, int nm, int e0, int ec, long ecp, const double* mat,
                int n_layers, const int* nonlinear, int ns, int depth, const double* dirs, const double* w,
                const double* du, void* theta_chunk, double* D, float* D32, uint32_t* D16, double* h,
                const int* stepping, bool d16_mean);

// ---- CG vectors (vec.hip): partial sums go to partial[(k*nblk + blk)*MB + m]
template <typename T>
void launch_dotsv(hipStream_t s, int nd, const T* a0, const T* b0, const T* a1, const T* b1, const T* a2,
                  const T* b2, long nrows, int MB, int nm, const int* flag, double* partial, int* nblk);

// inner CG iterations whose coefficients are kept for the spectrum estimate
constexpr int kLanczosMax = 64;
// law state per spring and integration point: 4 FP64 + one int32 of flags,
// plus two FP64 per older reversal point kept with a memory of depth > 1
constexpr int kThetaBytes = 36;
constexpr int kMaxMasingDepth = 8;  // the count of older points fits 3 bits of the flags
inline int theta_bytes(int depth) { return kThetaBytes + 16 * ((depth > 1 ? depth : 1) - 1); }
// Chebyshev degree limit; coefficient table cheb[(2 k + 0/1) * MB + m] =
// (c1_k, c2_k), k < kChebMax, and cheb[2 kChebMax * MB + m] = c0
constexpr int kChebMax = 64;

enum FinalizeStage {
    FIN_START = 0,   // (b.b, r.r, r.z): PCG start, active flags
    FIN_ALPHA,       // (p.Ap): alpha = rz / pAp
    FIN_BETA,        // (r.r, r.z): convergence, beta = rz_new / rz (PCG)
    FIN_FCG_START,   // (b.b, r.r): flexible CG start (outer)
    FIN_FCG_RZ,      // (z.Ap, z.r): rz = z.r after the first preconditioner call
    FIN_FCG_BETA,    // (z.Ap, z.r): beta = -alpha z.Ap / rz_old ; rz = z.r
    FIN_FCG_RR,      // (r.r): outer convergence check
    FIN_IN_START,    // (ir.ir, ir.w) inner start
    FIN_IN_ALPHA,    // (ip.iAp) inner alpha
    FIN_IN_BETA,     // (ir.ir, ir.w) inner convergence, beta
    FIN_CHEB_COUNT,  // (-): inner_total += degree for the outer-active members
    FIN_EST_START    // (ir.ir, ir.w) inner CG start on a random vector, for the members in this step
};
// per-member block partials of a compact kernel: lane k's sum over the block's
// rows (a fixed tree in LDS) goes to partial[(j * gridDim + blockIdx) * MB +
// tl[1 + k]], zero for the members not listed
template <int ND, int G>
__device__ __forceinline__ void tail_partials(double acc[ND], int MB, int m, double* __restrict__ partial, int boff,
                                              int nblk)
{
    __shared__ double sh[ND][256];
    __shared__ double pm[ND][256];
    const int t = threadIdx.x;
#pragma unroll
    for (int j = 0; j < ND; ++j) sh[j][t] = acc[j];
    __syncthreads();
    for (int s = 128; s >= G; s >>= 1) {  // s a multiple of G: lane k stays lane k
        if (t < s)
#pragma unroll
            for (int j = 0; j < ND; ++j) sh[j][t] += sh[j][t + s];
        __syncthreads();
    }
    if (t < MB)
#pragma unroll
        for (int j = 0; j < ND; ++j) pm[j][t] = 0.0;
    __syncthreads();
    if (t < G && m >= 0 && m < MB)
#pragma unroll
        for (int j = 0; j < ND; ++j) pm[j][m] = sh[j][t];  // listed members are distinct
    __syncthreads();
    if (t < MB)
#pragma unroll
        for (int j = 0; j < ND; ++j) partial[((size_t)j * nblk + boff + blockIdx.x) * MB + t] = pm[j][t];
}

void launch_fold(hipStream_t s, int nd, int MB, const double* partial, int nblk, int rows, double* fold);
void launch_finalize(hipStream_t s, FinalizeStage st, int nd, int MB, int nm, const double* partial, int nblk,
                     double* fold, const int* tl, int G, CgScalars cs, double tol2, int maxit);

void launch_pcg_start(hipStream_t s, int nn, int MB, int nm, const double* b, const double* Ap, const double* pinv,
                      double* r, double* z, double* p, const int* stepping, double* partial, int* nblk);
void launch_pcg_update(hipStream_t s, int nn, int MB, int nm, double* x, double* r, double* z, const double* p,
                       const double* Ap, const double* pinv, const double* alpha, const int* active, double* partial,
                       int* nblk);
template <typename T>
void launch_p_update(hipStream_t s, long nrows, int MB, int nm, const T* z, T* p, const double* beta, const int* active,
                     T* y);
void launch_xr_update(hipStream_t s, long nrows, int MB, int nm, double* x, double* r, const double* p, const double* Ap,
                      const double* alpha, const int* active, double* partial, int* nblk);
void launch_inner_start(hipStream_t s, int nn, int MB, int nm, const double* r, const float* pinv32, float* ir,
                        float* iz, float* ip, float* w, float* iAp, const int* active, double* partial, int* nblk);
void launch_inner_update(hipStream_t s, int nn, int MB, int nm, float* ir, float* w, const float* iAp,
                         const float* pinv32, const double* ialpha, const int* iactive, double* partial, int* nblk);
// x += alpha p, then p = z + beta p, for the members of upd
template <typename T>
void launch_pz(hipStream_t s, long nrows, int MB, int nm, T* x, T* p, const T* z, const double* alpha,
               const double* beta, const int* upd, const StageIn* fused = nullptr, const T* p_in = nullptr);
void launch_inner_out(hipStream_t s, long nrows, int MB, int nm, const float* iz, double* z, const double* Ap,
                      const double* r, const int* active, double* partial, int* nblk);
void launch_zero_if_b0(hipStream_t s, long nrows, int MB, int nm, double* x, const double* bb, const int* stepping);

// Chebyshev inner solve (preconditioner of the outer flexible CG)
void launch_cheb_bounds(hipStream_t s, int MB, int nm, CgScalars cs, int degree, double lo_scale, double hi_scale,
                        float* cheb, double* bounds);
void launch_cheb_hi_estimate(hipStream_t s, int MB, int nm, CgScalars cs, double scale, double* bounds);
void launch_fill_random(hipStream_t s, double* x, long n, uint64_t seed);
void launch_cheb_start(hipStream_t s, int nn, int MB, int nm, const double* r, const float* pinv32,
                       const float* cheb, float* ir, float* iz, float* id, const int* active);
void launch_cheb_update(hipStream_t s, int nn, int MB, int nm, int k, bool last, float* iz, float* ir,
                        const float* id, const float* iAp, float* id_next, const float* pinv32, const float* cheb,
                        const int* active);
void launch_gather_cheb(hipStream_t s, const DevMesh& M, int MB, int nm, int k, bool last, const float* rows,
                        float* iz, float* ir, const float* id, float* id_next, const float* pinv32,
                        const float* cheb, const int* active);

// Newmark state updates (Section 2.1) and receivers
void launch_newmark(hipStream_t s, long n, int MB, int nm, const double* du, double* u, double* v,
                    double* a, double dt, const int* stepping);
// CG initial guess extrapolated from the previous increments (order 0..2), history shifted
void launch_predict(hipStream_t s, long n, int MB, int nm, int order, double* du, double* d2, double* d3,
                    const int* stepping);
void launch_receivers(hipStream_t s, int nrecv, const int* recv, int MB, int nm, const double* v,
                      double* vel_hist, const int* member_step, int n_steps_max, double* vmax,
                      const int* stepping);
void launch_incident_velocity(hipStream_t s, int MB, int nm, int n_steps, const double* acc,
                              double* vI_all, double dt);
void launch_pick_vI(hipStream_t s, int MB, int nm, int n_steps, const double* vI_all,
                    const int* member_step, double* vI_cur);
void launch_response_spectra(hipStream_t s, const double* vel, int ns, int nt, double dt, const double* periods, int np,
                             double h, int kind, double* out);

}  // namespace nlth
