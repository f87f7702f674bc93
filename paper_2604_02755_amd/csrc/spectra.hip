// Velocity response spectra of receiver records (Section 3).
#include <hip/hip_runtime.h>

#include <cmath>

#include "nlth_impl.hpp"

namespace nlth {

// ---------------------------------------------------------------------------
// velocity response spectra of receiver records (Section 3, h = 0.05)
// ---------------------------------------------------------------------------

// One lane per (series, period), periods fastest (the lanes of a series read the
// same samples), a block of P wavefronts for 64 of them, each wavefront one
// part of the record.  The ground velocity is linear between samples, so
// the ground acceleration a_n = (v_n - v_{n-1}) / dt is constant on a step;
// over a step the oscillator x'' + 2 h w x' + w^2 x = -a moves as free damped
// vibration about its static offset -a / w^2, which gives the exact update of
// y = x + a / w^2 and x':
//   y(dt) = E ((C + q S) y + (S / wd) x'),  x'(dt) = E (-(w / r) S y + (C - q S) x'),
// with wd = w r, r = sqrt(1 - h^2), q = h / r, E = exp(-h w dt),
// C = cos(wd dt), S = sin(wd dt); y then changes by the change of the offset at
// the sample.  Carrying y instead of x makes a step two dependent operations
// instead of four.  With P > 1 a part is first run from rest; the
// states at the parts' ends follow from these and the same update over a
// part's length, and the part is run again from its state for the peaks.
//
// Bound by the chain of a step and by the vector loads: the samples are loaded
// sixteen ahead (a load a step, waited for, took 477 cycles a step), and where a
// wavefront's lanes cover at most four records (22 periods and more) they load
// sixteen samples of each at once and read them back from LDS.  Kernel: 867 series
// of 1,500 samples, 40 periods (542 wavefronts), 298 -> 88 us with one part, 83 with
// four, 58 through LDS; calls: 12 series of 2,000 samples, 20 periods, 362 -> 84 us
// (16 parts).
constexpr int kSpecAhead = 16;

struct Osc {
    double a11, a12, a21, a22;
};
__device__ __forceinline__ Osc osc_step(double w, double h, double t)
{
    const double r = sqrt(1.0 - h * h), q = h / r;
    const double E = exp(-h * w * t), C = cos(w * r * t), S = sin(w * r * t);
    return Osc{E * (C + q * S), E * S / (w * r), -E * w * S / r, E * (C - q * S)};
}

// samples n0 .. n1 of record v from (y, xd) just before sample n0, whose
// predecessors' velocity and offset are vp and op; PEAK: px, pv the largest |x|, |x'|.
// tile (64 doubles of LDS of the wavefront, or NULL): the lane's record is the ts-th of
// at most four of the wavefront, and the lane loads samples of record tv into it
template <bool PEAK>
__device__ __forceinline__ void osc_run(const double* __restrict__ v, int n0, int n1, const Osc& a, double scale,
                                        double& x, double& xd, double& px, double& pv, const double* __restrict__ tv,
                                        double* tile, int ts)
{
    // y = x + off; the offset of the last step is carried in `off`
    double vp = n0 > 0 ? v[n0 - 1] : 0.0, off = 0.0, y = x;
    auto step = [&](double vn) {
        const double on = (vn - vp) * scale;  // a_n / w^2
        vp = vn;
        y += on - off;
        off = on;
        const double y1 = fma(a.a11, y, a.a12 * xd);
        xd = fma(a.a21, y, a.a22 * xd);
        y = y1;
        if (PEAK) {
            px = fmax(px, fabs(y - off));
            pv = fmax(pv, fabs(xd));
        }
    };
    const int last = n1 - 1;
    int n = n0;
    if (tile) {
        // the lanes of at most four series: one load a tile, 16 samples of each
        double nx = n0 < n1 ? tv[min(n0 + (int)(threadIdx.x & 15), last)] : 0.0;
        for (; n + kSpecAhead <= n1; n += kSpecAhead) {
            tile[threadIdx.x & 63] = nx;
            __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
            nx = tv[min(n + kSpecAhead + (int)(threadIdx.x & 15), last)];
            double b[kSpecAhead];
#pragma unroll
            for (int k = 0; k < kSpecAhead; ++k) b[k] = tile[ts * kSpecAhead + k];
            __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
#pragma unroll
            for (int k = 0; k < kSpecAhead; ++k) step(b[k]);
        }
        for (; n < n1; ++n) step(v[n]);
        x = y - off;
        return;
    }
    double b[kSpecAhead];
#pragma unroll
    for (int k = 0; k < kSpecAhead; ++k) b[k] = n0 < n1 ? v[min(n0 + k, last)] : 0.0;
    for (; n + kSpecAhead <= n1; n += kSpecAhead) {
        double c[kSpecAhead];
#pragma unroll
        for (int k = 0; k < kSpecAhead; ++k) c[k] = v[min(n + kSpecAhead + k, last)];
#pragma unroll
        for (int k = 0; k < kSpecAhead; ++k) step(b[k]);
#pragma unroll
        for (int k = 0; k < kSpecAhead; ++k) b[k] = c[k];
    }
#pragma unroll
    for (int k = 0; k < kSpecAhead; ++k)
        if (n + k < n1) step(b[k]);
    x = y - off;
}

template <int P>
__global__ __launch_bounds__(64 * P) void k_response_spectra(const double* __restrict__ vel, int ns, int nt, double dt,
                                                            const double* __restrict__ periods, int np, double h,
                                                            int kind, double* __restrict__ out)
{
    const int lane = threadIdx.x & 63, part = threadIdx.x >> 6;
    const long t = blockIdx.x * 64l + lane, tc = min(t, (long)ns * np - 1);
    const int sr = (int)(tc / np), pk = (int)(tc % np);
    const double w = 2.0 * M_PI / periods[pk];
    const Osc a = osc_step(w, h, dt);
    const double scale = 1.0 / (dt * w * w);
    const double* v = vel + (size_t)sr * nt;
    double x = 0.0, xd = 0.0, px = 0.0, pv = 0.0;
    __shared__ double tiles[P][64];
    const int sr0 = (int)(min(blockIdx.x * 64l, (long)ns * np - 1) / np);
    const int srl = (int)(min(blockIdx.x * 64l + 63, (long)ns * np - 1) / np);
    double* tile = srl - sr0 < 4 ? tiles[part] : nullptr;
    const double* tv = vel + (size_t)min(sr0 + (lane >> 4), srl) * nt;
    const int ts = sr - sr0;
    const int len = (nt + P - 1) / P, n0 = min(part * len, nt), n1 = min(n0 + len, nt);
    if constexpr (P > 1) {
        __shared__ double end[P][2][64], peak[P][2][64];
        if (part < P - 1) osc_run<false>(v, n0, n1, a, scale, x, xd, px, pv, tv, tile, ts);
        end[part][0][lane] = x;
        end[part][1][lane] = xd;
        __syncthreads();
        const Osc l = osc_step(w, h, dt * len);
        x = xd = 0.0;
        for (int c = 0; c < part; ++c) {
            const double x1 = fma(l.a11, x, fma(l.a12, xd, end[c][0][lane]));
            xd = fma(l.a21, x, fma(l.a22, xd, end[c][1][lane]));
            x = x1;
        }
        osc_run<true>(v, n0, n1, a, scale, x, xd, px, pv, tv, tile, ts);
        peak[part][0][lane] = px;
        peak[part][1][lane] = pv;
        __syncthreads();
        if (part > 0) return;
        for (int c = 1; c < P; ++c) {
            px = fmax(px, peak[c][0][lane]);
            pv = fmax(pv, peak[c][1][lane]);
        }
    } else {
        osc_run<true>(v, n0, n1, a, scale, x, xd, px, pv, tv, tile, ts);
    }
    if (t < (long)ns * np) out[t] = kind == 0 ? pv : w * px;
}

void launch_response_spectra(hipStream_t s, const double* vel, int ns, int nt, double dt, const double* periods, int np,
                             double h, int kind, double* out)
{
    const long blocks = ((long)ns * np + 63) / 64;
    if (blocks <= 0) return;
    // parts double the work and divide its chain, which a wavefront alone leaves
    // two thirds idle: up to four wavefronts for each of the 1,024 SIMDs, and not below
    // 32 samples a part
    int P = 1;
    while (P < 16 && blocks * 2 * P <= 4096 && nt >= 64 * P) P *= 2;
#define NLTH_SPEC(PV)                                                                                               \
    hipLaunchKernelGGL((k_response_spectra<PV>), dim3((unsigned)blocks), dim3(64 * PV), 0, s, vel, ns, nt, dt, periods, \
                       np, h, kind, out)
    switch (P) {
    case 2: NLTH_SPEC(2); break;
    case 4: NLTH_SPEC(4); break;
    case 8: NLTH_SPEC(8); break;
    case 16: NLTH_SPEC(16); break;
    default: NLTH_SPEC(1); break;
    }
#undef NLTH_SPEC
}

}  // namespace nlth
