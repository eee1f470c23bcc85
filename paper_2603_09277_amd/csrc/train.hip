// Training-step terms around the rasterizer: the D-SSIM of the base loss
// (Sec. 3, Eq. 6) and a bias-corrected Adam step on raw parameters.
//
// SSIM follows the 3DGS lineage the paper builds on: per channel, local
// statistics over an 11x11 Gaussian window (sigma 1.5, normalised; zero outside
// the image), C1 = 0.01^2, C2 = 0.03^2,
//   S = (2 mx my + C1)(2 sxy + C2) / ((mx^2 + my^2 + C1)(sx^2 + sy^2 + C2)).
// The window is separable, so the statistics take a horizontal and a
// vertical 11-tap pass; the gradient runs the same two passes over the three
// per-pixel partials (dS/dmx, dS/dE[x^2], dS/dE[xy]) -- the window is symmetric,
// so the adjoint of each pass is the pass itself -- and combines them as
//   dS/dx_q = W*(dS/dmx) + 2 x_q W*(dS/dExx) + y_q W*(dS/dExy).
#include <cmath>

#include "internal.h"

namespace gsr {
namespace {

constexpr int kTaps = 11;
constexpr int kHalf = 5;
constexpr int kThr = 256;

__device__ __forceinline__ double block_sum_f64(double x)
{
    __shared__ double s[kThr];
    s[threadIdx.x] = x;
    __syncthreads();
    for (int o = kThr / 2; o > 0; o >>= 1) {
        if ((int)threadIdx.x < o) s[threadIdx.x] += s[threadIdx.x + o];
        __syncthreads();
    }
    return s[0];
}

// D-SSIM.  One launch covers every view, forward and gradient.  A workgroup owns a band
// of 64 pixel columns (192 floats: the interleaved channels are just a tap stride of
// 3) over a segment of rows and marches down it 8 rows at a time, so that the only
// traffic beyond the images, the gradient and their halos is LDS: per 8 rows
//   1. the rows' x and y (band + 10 pixels either side), loaded one step ahead, into LDS;
//   2. horizontal window sums of x^2 and y^2, then of x, y and xy, a thread per (row,
//      channel, 8-pixel strip): 18 values read for 8 outputs of 11 taps;
//   3. after each, vertical sums, a thread per float column, the 10 rows before the new ones
//      kept in registers; the SSIM map's terms and its three partials, zero outside the image;
//   4. horizontal sums of the partials, as 2;  5. vertical sums, as 3, and the gradient.
// Bound by its FMAs and LDS reads, not by memory.  The separable passes over whole
// images that this replaces (5 launches a view, 33 floats a pixel of scratch, every tap
// of an array of structures from L2) took 1.58 ms on 8 views of 9.76 Mpixel together and
// 0.23 ms on one 1296x840 image; this takes 0.43 ms (1.1 TB/s of images and gradient) and
// 0.077 ms, and on one of 148x96 23 us (24.5), with the same roundings in the same order.
// The five horizontal sums go through
// three planes of LDS in two parts, and loads are issued late, so that three workgroups
// fit a CU in LDS and registers (the prefetch before the first part: 0.62 ms, spilled).
// One window of x^2 + y^2 in place of two took 0.42 ms, but its last bits differ, and the
// scale and rotation gradients of some Gaussians, which cancel, showed that a thousandfold.
constexpr int kStep = 8;                       // rows a step
constexpr int kBandPx = 64;                    // output pixels across a band
constexpr int kOutF = 3 * kBandPx;             // its float columns
constexpr int kRS2 = kOutF + 3;                // row strides in LDS, 3 more than a multiple of 8: the lanes of a
                                               // strip pass read at 24 strip + channel + stride row
struct SsimView {
    int32_t W, H;
    uint32_t wg_base, bands;                   // first workgroup of the view; bands across
    int64_t off;                               // first float of the view
    float scale;                               // dloss/dSSIM-sum
};
constexpr int kSsimViews = 32;                 // views a launch
struct SsimArgs {
    SsimView v[kSsimViews];
    int32_t n_views, seg;                      // seg: output rows a workgroup
    float w[kHalf + 1];                        // the symmetric window: taps k and 10 - k are w[k]
};

// 8 outputs of the 11-tap window over 18 consecutive inputs
__device__ __forceinline__ void window8(const float* w, const float (&v)[kStep + 2 * kHalf], float (&o)[kStep])
{
#pragma unroll
    for (int j = 0; j < kStep; ++j) {
        float s = w[0] * v[j];
#pragma unroll
        for (int k = 1; k < kTaps; ++k) s = fmaf(w[k <= kHalf ? k : 2 * kHalf - k], v[j + k], s);
        o[j] = s;
    }
}

template <bool GRAD>
__global__ __launch_bounds__(kThr, 3) void ssim_kernel(const float* x, const float* y, SsimArgs a, float* grad,
                                                    double* block_sum)
{
    constexpr int kIn = kStep + 2 * kHalf;     // inputs of 8 outputs
    constexpr int kHalo1 = GRAD ? kHalf : 0;   // the map is needed this far around the outputs
    constexpr int kMapF = kOutF + 6 * kHalo1;  // its float columns
    constexpr int kInF = kMapF + 6 * kHalf;    // input float columns
    static_assert(kInF <= kThr, "one thread an input column");
    constexpr int kStrips1 = (kMapF + 23) / 24;
    constexpr int kRSin = GRAD ? 275 : 227, kRSh = GRAD ? 243 : 195, kRSp = 227;
    static_assert(24 * kStrips1 + 30 <= kRSin && 24 * kStrips1 <= kRSh && kOutF + 30 <= kRSp, "strips stay in a row");
    static_assert(kRS2 <= kRSh, "the second horizontal pass reuses the first one's rows");
    // the input rows and the partials' rows take turns in one array (three workgroups a CU)
    constexpr int kInWords = 2 * kStep * kRSin, kPWords = GRAD ? 3 * kStep * kRSp : 0;
    __shared__ float s_io[kInWords > kPWords ? kInWords : kPWords];
    __shared__ float s_h[3 * kStep * kRSh];
    __shared__ double s_sum[kThr / 64];
    const int t = (int)threadIdx.x;
    int v = 0;
    while (v + 1 < a.n_views && a.v[v + 1].wg_base <= blockIdx.x) ++v;
    const SsimView& vw = a.v[v];
    const int W = vw.W, H = vw.H;
    const uint32_t local = blockIdx.x - vw.wg_base;
    const int px0 = (int)(local % vw.bands) * kBandPx, r0 = (int)(local / vw.bands) * a.seg;
    const int r1 = r0 + a.seg < H ? r0 + a.seg : H;
    x += vw.off;
    y += vw.off;
    if (GRAD) grad += vw.off;
    const int64_t stride = 3 * (int64_t)W;
    // input column of this thread; map / output column (t < kMapF, t < kOutF)
    const int in_px = px0 - kHalo1 - kHalf + t / 3;
    const bool in_ok = t < kInF && in_px >= 0 && in_px < W;
    const int64_t in_c = 3 * (int64_t)(px0 - kHalo1 - kHalf) + t;
    const int map_px = px0 - kHalo1 + t / 3;
    const bool map_ok = t < kMapF && map_px >= 0 && map_px < W;
    const bool own_px = map_ok && map_px >= px0 && map_px < px0 + kBandPx;
    const int64_t out_c = 3 * (int64_t)px0 + t;
    const bool out_ok = t < kOutF && px0 + t / 3 < W;
    // strips: (row, strip, channel), the channel fastest
    const int h1_row = t / (3 * kStrips1), h1_rem = t % (3 * kStrips1), h1_c = 24 * (h1_rem / 3) + h1_rem % 3;
    const int h2_row = t / 24, h2_rem = t % 24, h2_c = 24 * (h2_rem / 3) + h2_rem % 3;

    float nx[kStep], ny[kStep];
    auto fetch = [&](int row) {
#pragma unroll
        for (int j = 0; j < kStep; ++j) {
            const bool ok = in_ok && row + j >= 0 && row + j < H;
            nx[j] = ok ? x[(row + j) * stride + in_c] : 0.f;
            ny[j] = ok ? y[(row + j) * stride + in_c] : 0.f;
        }
    };
    auto put = [&]() {
        if (t < kInF) {
#pragma unroll
            for (int j = 0; j < kStep; ++j) {
                s_io[j * kRSin + t] = nx[j];
                s_io[(kStep + j) * kRSin + t] = ny[j];
            }
        }
    };
    // horizontal window sums of this step's rows: x^2, y^2 (part 0), then x, y, xy (part 1)
    auto rows = [&](int part) {
        if (t >= 3 * kStrips1 * kStep) return;
        float xv[kIn], yv[kIn];
#pragma unroll
        for (int k = 0; k < kIn; ++k) {
            xv[k] = s_io[h1_row * kRSin + h1_c + 3 * k];
            yv[k] = s_io[(kStep + h1_row) * kRSin + h1_c + 3 * k];
        }
        float* h = s_h + h1_row * kRSh + h1_c;
        auto put_row = [&](int q, const float (&in)[kIn]) {
            float o[kStep];
            window8(a.w, in, o);
#pragma unroll
            for (int k = 0; k < kStep; ++k) h[q * kStep * kRSh + 3 * k] = o[k];
        };
        if (part == 0) {
#pragma unroll
            for (int k = 0; k < kIn; ++k) xv[k] *= xv[k];
            put_row(0, xv);
#pragma unroll
            for (int k = 0; k < kIn; ++k) yv[k] *= yv[k];
            put_row(1, yv);
        } else {
            put_row(0, xv);
            put_row(1, yv);
#pragma unroll
            for (int k = 0; k < kIn; ++k) xv[k] *= yv[k];
            put_row(2, xv);
        }
    };
    // vertical sums of row set q of s_h, `old` the 10 rows before it
    auto cols = [&](int q, float (&old)[2 * kHalf], float (&m)[kStep]) {
        float in[kIn];
#pragma unroll
        for (int k = 0; k < 2 * kHalf; ++k) in[k] = old[k];
#pragma unroll
        for (int j = 0; j < kStep; ++j) in[2 * kHalf + j] = s_h[(q * kStep + j) * kRSh + t];
        window8(a.w, in, m);
#pragma unroll
        for (int k = 0; k < 2 * kHalf; ++k) old[k] = in[kStep + k];
    };
    float old1[5][2 * kHalf], old2[GRAD ? 3 : 1][2 * kHalf];
#pragma unroll
    for (int q = 0; q < 5; ++q)
#pragma unroll
        for (int k = 0; k < 2 * kHalf; ++k) old1[q][k] = 0.f;
#pragma unroll
    for (int q = 0; q < (GRAD ? 3 : 1); ++q)
#pragma unroll
        for (int k = 0; k < 2 * kHalf; ++k) old2[q][k] = 0.f;
    double sacc = 0.0;
    int row = r0 - kHalo1 - kHalf;             // the step's first input row
    fetch(row);
    put();
    // the step of input rows [row, row + 8) completes map rows [row - 5, row + 3) and
    // output rows [row - 10, row - 2)
    for (; row - kHalf - kHalo1 < r1; row += kStep) {
        float m[5][kStep];
        __syncthreads();
        rows(0);
        __syncthreads();
        if (t < kMapF) {
#pragma unroll
            for (int q = 0; q < 2; ++q) cols(q, old1[q], m[q]);
        }
        __syncthreads();
        if (!GRAD) fetch(row + kStep);
        rows(1);
        __syncthreads();
        if (!GRAD) put();                       // (every read of this step's rows is done)
        if (t < kMapF) {
#pragma unroll
            for (int q = 0; q < 3; ++q) cols(q, old1[2 + q], m[2 + q]);
            const float C1 = 1e-4f, C2 = 9e-4f;
#pragma unroll
            for (int j = 0; j < kStep; ++j) {
                const int r = row - kHalf + j;
                const float mx = m[2][j], my = m[3][j];
                // (each rounding written out)
                const float ld = __fadd_rn(fmaf(mx, mx, __fmul_rn(my, my)), C1);
                const float cd = __fadd_rn(__fadd_rn(fmaf(-mx, mx, m[0][j]), fmaf(-my, my, m[1][j])), C2);
                const float cn = fmaf(2.f, fmaf(-mx, my, m[4][j]), C2);
                const float ln = fmaf(2.f * mx, my, C1);
                const float N = __fmul_rn(ln, cn), D = __fmul_rn(ld, cd);
                const float iD = 1.f / D, S = __fmul_rn(N, iD);
                if (own_px && r >= r0 && r < r1) sacc += (double)S;
                if (GRAD) {
                    const bool ok = map_ok && r >= 0 && r < H;
                    const float dD = __fmul_rn(2.f * mx, __fsub_rn(cd, ld));
                    const float g0 = __fmul_rn(iD, fmaf(2.f * my, __fsub_rn(cn, ln), -__fmul_rn(dD, S)));
                    const float g1 = __fmul_rn(iD, __fmul_rn(__fmul_rn(ld, -N), iD));
                    s_io[(0 * kStep + j) * kRSp + t] = ok ? g0 : 0.f;                          // dS/dmx
                    s_io[(1 * kStep + j) * kRSp + t] = ok ? g1 : 0.f;                          // dS/dExx
                    s_io[(2 * kStep + j) * kRSp + t] = ok ? __fmul_rn(2.f * ln, iD) : 0.f;     // dS/dExy
                }
            }
        }
        if constexpr (GRAD) {
            fetch(row + kStep);
            __syncthreads();
            // (no output needs the first step's map rows)
            if (t < 24 * kStep && row >= r0 - 2 * kHalf + kStep) {
#pragma unroll
                for (int q = 0; q < 3; ++q) {
                    float in[kIn], o[kStep];
#pragma unroll
                    for (int k = 0; k < kIn; ++k) in[k] = s_io[(q * kStep + h2_row) * kRSp + h2_c + 3 * k];
                    window8(a.w, in, o);
#pragma unroll
                    for (int k = 0; k < kStep; ++k) s_h[(q * kStep + h2_row) * kRS2 + h2_c + 3 * k] = o[k];
                }
            }
            __syncthreads();
            float gx[kStep], gy[kStep], gg[kStep];
#pragma unroll
            for (int j = 0; j < kStep; ++j) {   // in flight over the vertical pass
                const int r = row - 2 * kHalf + j;
                const bool ok = out_ok && r >= r0 && r < r1;
                gx[j] = ok ? x[r * stride + out_c] : 0.f;
                gy[j] = ok ? y[r * stride + out_c] : 0.f;
                gg[j] = ok ? grad[r * stride + out_c] : 0.f;
            }
            put();                              // (every read of the partials is done)
            if (t < kOutF && row >= r0 - 2 * kHalf + kStep) {
                float m2[3][kStep];
#pragma unroll
                for (int q = 0; q < 3; ++q) {
                    float in[kIn];
#pragma unroll
                    for (int k = 0; k < 2 * kHalf; ++k) in[k] = old2[q][k];
#pragma unroll
                    for (int j = 0; j < kStep; ++j) in[2 * kHalf + j] = s_h[(q * kStep + j) * kRS2 + t];
                    window8(a.w, in, m2[q]);
#pragma unroll
                    for (int k = 0; k < 2 * kHalf; ++k) old2[q][k] = in[kStep + k];
                }
#pragma unroll
                for (int j = 0; j < kStep; ++j) {
                    const int r = row - 2 * kHalf + j;
                    if (out_ok && r >= r0 && r < r1) {
                        const float d = fmaf(gy[j], m2[2][j], fmaf(2.f * gx[j], m2[1][j], m2[0][j]));
                        grad[r * stride + out_c] = fmaf(vw.scale, d, gg[j]);
                    }
                }
            }
        }
    }
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) sacc += __shfl_xor(sacc, o, 64);
    if ((t & 63) == 0) s_sum[t >> 6] = sacc;
    __syncthreads();
    if (t == 0) {
        double tot = 0.0;
#pragma unroll
        for (int w = 0; w < kThr / 64; ++w) tot += s_sum[w];
        block_sum[blockIdx.x] = tot;
    }
}

// one workgroup a view: weight (1 - SSIM) from its workgroups' sums, in a fixed order
__global__ __launch_bounds__(kThr) void ssim_loss_kernel(const double* block_sum, SsimArgs a, uint32_t n_wg,
                                                         float weight, float* loss)
{
    const int v = (int)blockIdx.x;
    const uint32_t b1 = v + 1 < a.n_views ? a.v[v + 1].wg_base : n_wg;
    double acc = 0.0;
    for (uint32_t b = a.v[v].wg_base + threadIdx.x; b < b1; b += kThr) acc += block_sum[b];
    const double tot = block_sum_f64(acc);
    if (threadIdx.x == 0)
        loss[v] = (float)((double)weight * (1.0 - tot / (3.0 * (double)((int64_t)a.v[v].W * a.v[v].H))));
}

// one bias-corrected Adam step on raw parameters; kind 0 identity, 1 exp, 2 sigmoid
struct AdamParams {
    float lr, b1, b2, eps, c1, c2;     // c1, c2: the bias corrections 1 / (1 - b^step)
    int kind;                          // 0 identity, 1 exp, 2 sigmoid
};

// The sigmoid and its derivative from e = exp(-|r|), which never cancels:
// sigmoid(r) = 1 / (1 + e) for r >= 0 and e / (1 + e) below; sigmoid' = e / (1 + e)^2.
__device__ __forceinline__ float act_of(float r, int kind)
{
    if (kind == 1) return expf(r);
    if (kind == 2) {
        const float e = expf(-fabsf(r)), q = 1.f / (1.f + e);
        return r >= 0.f ? q : e * q;
    }
    return r;
}

__device__ __forceinline__ float dact_of(float r, int kind)
{
    if (kind == 1) return expf(r);
    if (kind == 2) {
        const float e = expf(-fabsf(r)), q = 1.f / (1.f + e);
        return e * q * q;
    }
    return 1.f;
}

__device__ __forceinline__ void adam_one(float& r, float& m, float& v, float& a, float ga, const AdamParams& p)
{
    const float g = ga * dact_of(r, p.kind);
    m = p.b1 * m + (1.f - p.b1) * g;
    v = p.b2 * v + (1.f - p.b2) * g * g;
    r = r - p.lr * (m * p.c1) / (sqrtf(v * p.c2) + p.eps);
    a = act_of(r, p.kind);
}

// Element-wise, HBM-bound: 16 B read and 12-16 B written per parameter.  VEC moves
// four parameters per lane with 16-byte accesses (all pointers 16-byte aligned);
// the last n % 4 go one per lane.
template <bool VEC>
__global__ void __launch_bounds__(256) adam_kernel(float* raw, float* m, float* v, float* act, const float* grad_act,
                                                   int64_t n, AdamParams p)
{
    const int64_t stride = (int64_t)gridDim.x * blockDim.x;
    const int64_t t0 = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    int64_t done = 0;
    if (VEC) {
        const int64_t n4 = n >> 2;
        for (int64_t i = t0; i < n4; i += stride) {
            float4 r = reinterpret_cast<float4*>(raw)[i], mm = reinterpret_cast<float4*>(m)[i];
            float4 vv = reinterpret_cast<float4*>(v)[i];
            const float4 ga = reinterpret_cast<const float4*>(grad_act)[i];
            float4 a;
            adam_one(r.x, mm.x, vv.x, a.x, ga.x, p);
            adam_one(r.y, mm.y, vv.y, a.y, ga.y, p);
            adam_one(r.z, mm.z, vv.z, a.z, ga.z, p);
            adam_one(r.w, mm.w, vv.w, a.w, ga.w, p);
            reinterpret_cast<float4*>(raw)[i] = r;
            reinterpret_cast<float4*>(m)[i] = mm;
            reinterpret_cast<float4*>(v)[i] = vv;
            if (act) reinterpret_cast<float4*>(act)[i] = a;
        }
        done = n4 << 2;
    }
    for (int64_t i = done + t0; i < n; i += stride) {
        float r = raw[i], mm = m[i], vv = v[i], a;
        adam_one(r, mm, vv, a, grad_act[i], p);
        raw[i] = r;
        m[i] = mm;
        v[i] = vv;
        if (act) act[i] = a;
    }
}

uint32_t ssim_groups(int32_t W, int32_t H, int seg)
{
    return (uint32_t)((W + kBandPx - 1) / kBandPx) * (uint32_t)((H + seg - 1) / seg);
}

// rows a workgroup, of those whose marched rows (the segment and its halo) are whole
// steps: the one of the least time, rounds of workgroups (3 a CU, by LDS) times steps, where
// a step takes 5.9 us with one workgroup a CU, 7.9 with two and 10.3 with three: 3, 4 and 5 units for
// the last round.  (Counted as equal, 320x480 took three steps at 600 workgroups, 37 us, instead of
// four at 200, 30; 148x96 takes three at 72, 23, and four would take 31.)
int ssim_segment(const SsimSizes& z, int v0, int n, bool with_grad, uint64_t* groups)
{
    constexpr uint64_t kResident = 768;
    const int halo = with_grad ? 4 * kHalf : 2 * kHalf;
    int best = 0;
    uint64_t best_cost = 0;
    for (int steps : { 18, 14, 10, 8, 6, 4, 3 }) {
        const int seg = steps * kStep - halo;
        uint64_t wgs = 0;
        for (int v = v0; v < v0 + n; ++v) wgs += ssim_groups(z.w(v), z.h(v), seg);
        const uint64_t rest = wgs % kResident;
        const uint64_t cost = (5 * (wgs / kResident) + (rest == 0 ? 0 : rest <= 256 ? 3 : rest <= 512 ? 4 : 5)) * (uint64_t)steps;
        if (best == 0 || cost <= best_cost) { best = seg; best_cost = cost; *groups = wgs; }
    }
    return best;
}

}  // namespace

size_t ssim_tmp_bytes(const SsimSizes& z, bool with_grad)
{
    uint64_t most = 1;
    for (int v0 = 0; v0 < z.n; v0 += kSsimViews) {
        uint64_t g = 0;
        (void)ssim_segment(z, v0, z.n - v0 < kSsimViews ? z.n - v0 : kSsimViews, with_grad, &g);
        most = g > most ? g : most;
    }
    return (size_t)most * sizeof(double);
}

hipError_t launch_dssim(const float* x, const float* y, const SsimSizes& z, float weight, float* grad, float* loss,
                        void* tmp, hipStream_t s)
{
    SsimArgs a;
    double g[kTaps], gsum = 0.0;
    for (int k = 0; k < kTaps; ++k) { g[k] = std::exp(-(double)((k - kHalf) * (k - kHalf)) / (2.0 * 1.5 * 1.5)); gsum += g[k]; }
    for (int k = 0; k <= kHalf; ++k) a.w[k] = (float)(g[k] / gsum);
    double* bsum = (double*)tmp;
    int64_t off = 0;
    for (int v0 = 0; v0 < z.n; v0 += kSsimViews) {
        const int n = z.n - v0 < kSsimViews ? z.n - v0 : kSsimViews;
        uint64_t groups = 0;
        a.n_views = n;
        a.seg = ssim_segment(z, v0, n, grad != nullptr, &groups);
        uint32_t wg = 0;
        for (int v = 0; v < n; ++v) {
            SsimView& q = a.v[v];
            q.W = z.w(v0 + v);
            q.H = z.h(v0 + v);
            q.wg_base = wg;
            q.bands = (uint32_t)((q.W + kBandPx - 1) / kBandPx);
            q.off = 3 * off;
            // L = weight (1 - SSIM), SSIM = sum S / (3 M)
            const int64_t M = (int64_t)q.W * q.H;
            q.scale = -weight / (3.0f * (float)M);
            wg += ssim_groups(q.W, q.H, a.seg);
            off += M;
        }
        if (grad) hipLaunchKernelGGL(ssim_kernel<true>, dim3(wg), dim3(kThr), 0, s, x, y, a, grad, bsum);
        else hipLaunchKernelGGL(ssim_kernel<false>, dim3(wg), dim3(kThr), 0, s, x, y, a, grad, bsum);
        if (loss)
            hipLaunchKernelGGL(ssim_loss_kernel, dim3(n), dim3(kThr), 0, s, bsum, a, wg, weight, loss + v0);
    }
    return hipGetLastError();
}

hipError_t launch_adam(float* raw, float* m, float* v, float* act, const float* grad_act, int64_t n, int kind,
                       float lr, float b1, float b2, float eps, int64_t step, hipStream_t s)
{
    if (n <= 0) return hipSuccess;
    const float c1 = (float)(1.0 / (1.0 - std::pow((double)b1, (double)step)));
    const float c2 = (float)(1.0 / (1.0 - std::pow((double)b2, (double)step)));
    const AdamParams p{lr, b1, b2, eps, c1, c2, kind};
    auto a16 = [](const void* q) { return ((uintptr_t)q & 15) == 0; };
    const bool vec = a16(raw) && a16(m) && a16(v) && a16(grad_act) && (!act || a16(act));
    int64_t blocks = ((vec ? (n + 3) / 4 : n) + 255) / 256;
    if (blocks > 65536) blocks = 65536;
    if (vec)
        hipLaunchKernelGGL(adam_kernel<true>, dim3((unsigned)blocks), dim3(256), 0, s, raw, m, v, act, grad_act, n, p);
    else
        hipLaunchKernelGGL(adam_kernel<false>, dim3((unsigned)blocks), dim3(256), 0, s, raw, m, v, act, grad_act, n, p);
    return hipGetLastError();
}

}  // namespace gsr
