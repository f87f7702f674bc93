// Allocation-free form of the diagnostic operator application, for callers
// that cannot allocate device memory: code under HIP graph capture, tight
// serving loops, harnesses that forbid hipMalloc.  The caller passes device
// buffers for the inputs and the output; the intermediate (the operator's
// rows) lives in one file-scope device array of
// kScratchBytes that each device the library runs on holds until the process
// ends.  Its device address comes from hipGetSymbolAddress, taken once per
// device when a context is created on it (in host code the array's name is
// only a host-side stand-in).  The kernels are those of nlth_apply_operator's
// FP64 path for one member slot, which read D and h in input tet order and x in
// input node order, so the two entry points give the same results.  (Copying D,
// h, x and y between the orders took 5 launches more and moved D three times:
// with 58,080 tets 84 -> 29.5 us a call on the same buffers, whose 39 MB of D the
// last-level cache then holds, 99 -> 33 us on sixteen sets of buffers in turn, 255 ->
// 190 us for a first call on buffers not touched before.)
#include <math.h>
#include <string.h>

#include <cstdio>

#include "runtime.hpp"

namespace nlth {

constexpr size_t kScratchBytes = (size_t)64 << 20;  // per device
constexpr int kScratchDevices = 64;

static __device__ __align__(256) unsigned char scratch[kScratchBytes];

static std::mutex g_scratch_mu;
static void* g_scratch_ptr[kScratchDevices];

// Device address of `scratch` on `device`, which must be current; taken once
// per device and kept.
void scratch_setup(int device)
{
    if (device < 0 || device >= kScratchDevices) throw Error{NLTH_EDEVICE, "device index beyond the scratch table"};
    std::lock_guard<std::mutex> g(g_scratch_mu);
    if (g_scratch_ptr[device]) return;
    void* p = nullptr;
    const hipError_t e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
    if (e != hipSuccess || !p)
        throw Error{NLTH_EDEVICE, std::string("hipGetSymbolAddress(scratch): ") + hipGetErrorString(e)};
    g_scratch_ptr[device] = p;
}

static char* scratch_of(int device)
{
    std::lock_guard<std::mutex> g(g_scratch_mu);
    return (device >= 0 && device < kScratchDevices) ? (char*)g_scratch_ptr[device] : nullptr;
}

void rayleigh_coefficients(double f_lo, double f_hi, double* a, double* b);

}  // namespace nlth

using namespace nlth;

struct nlth_ctx : Ctx {};
struct nlth_mesh : Mesh {};

static size_t round256(size_t n) { return (n + 255) / 256 * 256; }

extern "C" int nlth_apply_operator_noalloc(nlth_ctx* ctx, const nlth_mesh* mesh, const nlth_problem* prob,
                                           int32_t which, const double* D_ip, const double* h, const double* x,
                                           double* y)
{
    Ctx* c = ctx;
    try {
        if (!ctx || !mesh || !prob || !D_ip || !x || !y) throw Error{NLTH_EINVAL, "NULL argument"};
        if (ctx->host_only) throw Error{NLTH_EDEVICE, "host-only context"};
        if (mesh->ctx != ctx) throw Error{NLTH_EINVAL, "mesh belongs to another context"};
        if (which < NLTH_OP_A || which > NLTH_OP_M) throw Error{NLTH_EINVAL, "which must be NLTH_OP_A/K/M"};
        const int nl = prob->n_layers;
        if (nl <= 0 || nl > kNoAllocMaxLayers)
            throw Error{NLTH_EINVAL, "problem: n_layers must be in 1..32 for the allocation-free apply"};
        if (nl <= mesh->max_layer) throw Error{NLTH_EINVAL, "problem: mesh uses a layer id >= n_layers"};
        if (!prob->rho || !prob->vs || !prob->nu || !prob->gamma_ref || !prob->h_max)
            throw Error{NLTH_EINVAL, "problem: a required array is NULL"};
        if (!(prob->dt > 0)) throw Error{NLTH_EINVAL, "problem: dt must be positive"};
        if (prob->damping_mode < NLTH_DAMPING_LAW || prob->damping_mode > NLTH_DAMPING_NONE)
            throw Error{NLTH_EINVAL, "problem: unknown damping mode"};
        if (prob->damping_mode != NLTH_DAMPING_NONE && !(prob->f_lo > 0 && prob->f_hi > prob->f_lo))
            throw Error{NLTH_EINVAL, "problem: Rayleigh band needs 0 < f_lo < f_hi"};
        const int ne = mesh->ne, nn = mesh->nn;
        const long n3 = 3L * nn;
        // the scratch holds the operator's rows, at most ten per element (2.6 on boxes)
        // and one per boundary node; the capacity that the entry point states is larger,
        // a material table, D, h, two nodal vectors and ten rows per element, and stays as
        // callers know it
        const size_t ne_pad = ((size_t)ne + 63) / 64 * 64;
        const size_t need = round256((size_t)nl * MAT_N * 8) + round256(ne_pad * 84 * 8) + round256(ne_pad * 8) + 2 * round256((size_t)n3 * 8) +
                            round256(ne_pad * 30 * 8);
        if (need > kScratchBytes) {
            char buf[200];
            snprintf(buf, sizeof buf,
                     "mesh of %d tets and %d nodes needs %.1f MiB of scratch; the allocation-free apply holds "
                     "at most %.0f MiB (about 67,000 tets)",
                     ne, nn, need / 1048576.0, kScratchBytes / 1048576.0);
            throw Error{NLTH_EINVAL, buf};
        }
        LayerMat lm{};
        for (int l = 0; l < nl; ++l) {
            const double rho = prob->rho[l], vs = prob->vs[l], nu = prob->nu[l], hm = prob->h_max[l];
            if (!(rho > 0 && vs > 0 && nu > -1.0 && nu < 0.5))
                throw Error{NLTH_EINVAL, "problem: layer needs rho > 0, vs > 0, -1 < nu < 0.5"};
            const double G0 = rho * vs * vs, lam = 2.0 * G0 * nu / (1.0 - 2.0 * nu);
            double* col = lm.v + (size_t)l * MAT_N;
            col[MAT_RHO] = rho;
            col[MAT_G0] = G0;
            col[MAT_KB] = lam + 2.0 * G0 / 3.0;
            col[MAT_VS] = vs;
            col[MAT_VP] = sqrt((lam + 2.0 * G0) / rho);
            col[MAT_GREF] = prob->gamma_ref[l];
            col[MAT_HMAX] = hm;
            col[MAT_BETA] = 2.0 * M_PI * hm / (2.0 - M_PI * hm);
        }
        StepConst sc{};
        sc.dt = prob->dt;
        sc.damping_mode = prob->damping_mode;
        sc.h0 = prob->h0;
        if (prob->damping_mode == NLTH_DAMPING_NONE) sc.ahat = sc.bhat = 0.0;
        else rayleigh_coefficients(prob->f_lo, prob->f_hi, &sc.ahat, &sc.bhat);
        sc.quotients();

        std::lock_guard<std::mutex> g(ctx->mu);
        NLTH_HIP(hipSetDevice(ctx->device));
        char* base = scratch_of(ctx->device);
        if (!base) throw Error{NLTH_EDEVICE, "scratch address not set up on this device"};
        double* rows = (double*)base;
        hipStream_t s = ctx->stream;
        const DevMesh dm = mesh->dev_input();
        const double dc = which == NLTH_OP_A ? 2.0 / prob->dt : 0.0;
        launch_op_input64(s, (OpMode)which, dm, mesh->order_d.as<int>(), D_ip, h, lm, sc, x, rows, dc);
        launch_gather<double>(s, dm, 1, 1, rows, dc != 0.0, nullptr, 0.0, y, nullptr, mesh->node_in.as<int>());
        NLTH_HIP(hipGetLastError());
        return NLTH_OK;
    } catch (const Error& e) {
        set_error(c, e);
        return e.code;
    }
}
