// EWA projection of 3D Gaussians (Sec. 3, Eq. 1-2) and its backward.
//
// Forward: one thread per Gaussian, which loops over the views of the launch so
// that parameters and SH coefficients are read from HBM once per Gaussian,
// not once per (view, Gaussian).  Backward: a workgroup owns 256 Gaussians and
// works on those of their views that blended them.  Everything is FP32 except the 2x2
// determinant / inverse / eigenvalue step, which runs in FP64: near-degenerate
// 2D covariances lose all significant digits of det = ac - b^2 in FP32.
#include "internal.h"

namespace gsr {
namespace {

constexpr uint32_t F_DILATE = 1u, F_JCLAMP = 2u, F_CCLAMP = 4u;

__device__ __forceinline__ float bf16_to_f32(uint16_t h) { return __uint_as_float((uint32_t)h << 16); }

__device__ __forceinline__ uint16_t f32_to_bf16_rne(float f)
{
    uint32_t b = __float_as_uint(f);
    if ((b & 0x7fffffffu) > 0x7f800000u) return (uint16_t)((b >> 16) | 0x40u);   // keep NaN quiet
    b += 0x7fffu + ((b >> 16) & 1u);
    return (uint16_t)(b >> 16);
}

// Real spherical harmonics without the Condon-Shortley phase, ordered
// k = l*l + l + m; the coefficients are sqrt((2l+1)/(4 pi) (l-|m|)!/(l+|m|)!)
// (times sqrt 2 for m != 0) folded into the polynomial of each (l, m).
constexpr float kC0 = 0.28209479177387814f;
constexpr float kC1 = 0.4886025119029199f;
constexpr float kC2a = 1.0925484305920792f;    // xy, yz, xz
constexpr float kC2b = 0.31539156525252005f;   // 3z^2 - 1
constexpr float kC2c = 0.5462742152960396f;    // x^2 - y^2
constexpr float kC3a = 0.5900435899266435f;    // y(3x^2 - y^2), x(x^2 - 3y^2)
constexpr float kC3b = 2.890611442640554f;     // xyz
constexpr float kC3c = 0.4570457994644658f;    // y(5z^2 - 1), x(5z^2 - 1)
constexpr float kC3d = 0.3731763325901154f;    // z(5z^2 - 3)
constexpr float kC3e = 1.445305721320277f;     // z(x^2 - y^2)

template <int DEG>
__device__ __forceinline__ void sh_basis(float x, float y, float z, float* Y)
{
    Y[0] = kC0;
    if constexpr (DEG >= 1) { Y[1] = kC1 * y; Y[2] = kC1 * z; Y[3] = kC1 * x; }
    if constexpr (DEG >= 2) {
        float xx = x * x, yy = y * y, zz = z * z;
        Y[4] = kC2a * x * y;
        Y[5] = kC2a * y * z;
        Y[6] = kC2b * (3.f * zz - 1.f);
        Y[7] = kC2a * x * z;
        Y[8] = kC2c * (xx - yy);
        if constexpr (DEG >= 3) {
            Y[9] = kC3a * y * (3.f * xx - yy);
            Y[10] = kC3b * x * y * z;
            Y[11] = kC3c * y * (5.f * zz - 1.f);
            Y[12] = kC3d * z * (5.f * zz - 3.f);
            Y[13] = kC3c * x * (5.f * zz - 1.f);
            Y[14] = kC3e * z * (xx - yy);
            Y[15] = kC3a * x * (xx - 3.f * yy);
        }
    }
}

// d/d(x, y, z) of sum_k w_k Y_k(x, y, z) (partials of the polynomials above)
template <int DEG>
__device__ __forceinline__ float3 sh_basis_grad(float x, float y, float z, const float* w)
{
    float gx = 0.f, gy = 0.f, gz = 0.f;
    if constexpr (DEG >= 1) { gy += kC1 * w[1]; gz += kC1 * w[2]; gx += kC1 * w[3]; }
    if constexpr (DEG >= 2) {
        gx += kC2a * y * w[4]; gy += kC2a * x * w[4];
        gy += kC2a * z * w[5]; gz += kC2a * y * w[5];
        gz += 6.f * kC2b * z * w[6];
        gx += kC2a * z * w[7]; gz += kC2a * x * w[7];
        gx += 2.f * kC2c * x * w[8]; gy -= 2.f * kC2c * y * w[8];
        if constexpr (DEG >= 3) {
            float xx = x * x, yy = y * y, zz = z * z;
            gx += 6.f * kC3a * x * y * w[9];          gy += 3.f * kC3a * (xx - yy) * w[9];
            gx += kC3b * y * z * w[10];               gy += kC3b * x * z * w[10];     gz += kC3b * x * y * w[10];
            gy += kC3c * (5.f * zz - 1.f) * w[11];    gz += 10.f * kC3c * y * z * w[11];
            gz += kC3d * (15.f * zz - 3.f) * w[12];
            gx += kC3c * (5.f * zz - 1.f) * w[13];    gz += 10.f * kC3c * x * z * w[13];
            gx += 2.f * kC3e * x * z * w[14];         gy -= 2.f * kC3e * y * z * w[14]; gz += kC3e * (xx - yy) * w[14];
            gx += 3.f * kC3a * (xx - yy) * w[15];     gy -= 6.f * kC3a * x * y * w[15];
        }
    }
    return make_float3(gx, gy, gz);
}

// Rotation matrix (row-major) of the unit quaternion (w, x, y, z).
__device__ __forceinline__ void quat_to_rot(float w, float x, float y, float z, float* R)
{
    R[0] = 1.f - 2.f * (y * y + z * z); R[1] = 2.f * (x * y - w * z);       R[2] = 2.f * (x * z + w * y);
    R[3] = 2.f * (x * y + w * z);       R[4] = 1.f - 2.f * (x * x + z * z); R[5] = 2.f * (y * z - w * x);
    R[6] = 2.f * (x * z - w * y);       R[7] = 2.f * (y * z + w * x);       R[8] = 1.f - 2.f * (x * x + y * y);
}

template <int K, bool BF16>
__device__ __forceinline__ void load_sh(const void* sh, uint32_t i, float* out)
{
    if constexpr (BF16) {
        const uint16_t* p = reinterpret_cast<const uint16_t*>(sh) + (size_t)i * (K * 3);
#pragma unroll
        for (int k = 0; k < K * 3; ++k) out[k] = bf16_to_f32(p[k]);
    } else {
        const float* p = reinterpret_cast<const float*>(sh) + (size_t)i * (K * 3);
#pragma unroll
        for (int k = 0; k < K * 3; ++k) out[k] = p[k];
    }
}

__device__ __forceinline__ bool finite3(float a, float b, float c) { return isfinite(a) && isfinite(b) && isfinite(c); }

// Per-Gaussian, view-independent state: normalised quaternion, rotation,
// 3D covariance (upper triangle 00 01 02 11 12 22).
struct Local {
    bool ok;
    float qn[4], qnorm;
    float R[9];
    float S[6];
};

__device__ __forceinline__ void local_state(const float* mu, const float* s, const float* q, float op,
                                            const float* sh, int nsh, Local& L)
{
    bool ok = finite3(mu[0], mu[1], mu[2]) && finite3(s[0], s[1], s[2]) && finite3(q[0], q[1], q[2]) &&
              isfinite(q[3]) && isfinite(op);
    for (int k = 0; k < nsh; ++k) ok = ok && isfinite(sh[k]);
    float qn2 = q[0] * q[0] + q[1] * q[1] + q[2] * q[2] + q[3] * q[3];
    ok = ok && qn2 > 0.f;
    float qn = sqrtf(qn2);
    L.qnorm = qn;
    float iq = ok ? 1.f / qn : 0.f;
    for (int k = 0; k < 4; ++k) L.qn[k] = q[k] * iq;
    quat_to_rot(L.qn[0], L.qn[1], L.qn[2], L.qn[3], L.R);
    float s2[3] = { s[0] * s[0], s[1] * s[1], s[2] * s[2] };
    const float* R = L.R;
    // Sigma = R diag(s^2) R^T  (Eq. 1)
    L.S[0] = R[0] * R[0] * s2[0] + R[1] * R[1] * s2[1] + R[2] * R[2] * s2[2];
    L.S[1] = R[0] * R[3] * s2[0] + R[1] * R[4] * s2[1] + R[2] * R[5] * s2[2];
    L.S[2] = R[0] * R[6] * s2[0] + R[1] * R[7] * s2[1] + R[2] * R[8] * s2[2];
    L.S[3] = R[3] * R[3] * s2[0] + R[4] * R[4] * s2[1] + R[5] * R[5] * s2[2];
    L.S[4] = R[3] * R[6] * s2[0] + R[4] * R[7] * s2[1] + R[5] * R[8] * s2[2];
    L.S[5] = R[6] * R[6] * s2[0] + R[7] * R[7] * s2[1] + R[8] * R[8] * s2[2];
    L.ok = ok;
}

// Per-(view, Gaussian) projection state shared by forward and backward.
struct ViewProj {
    bool ok;
    float tx, ty, tz, u, v, uc, vc;
    bool clx, cly;
    float J00, J02, J11, J12;
    float Tm[6];          // J Rc, 2x3
    float W[6];           // Tm Sigma, 2x3
    double a, b, c, det;  // dilated 2D covariance and its determinant
    double qA, qB, qC;    // conic (inverse)
    float mx, my;
};

__device__ __forceinline__ void view_proj(const CamDev& c, const float* mu, const Local& L, uint32_t flags,
                                          ViewProj& P)
{
    P.ok = false;
    // Camera transform, perspective divide and 2D mean in FP64 (unfused, in a
    // fixed order): the float32 results are then the correctly rounded values
    // of the exact ones, so the depth key and the tile rectangle of a Gaussian
    // do not depend on FP32 cancellation in R mu + t.
    double t3[3];
    for (int r = 0; r < 3; ++r)
        t3[r] = __dadd_rn(__dadd_rn(__dadd_rn(__dmul_rn((double)c.R[3 * r], (double)mu[0]),
                                              __dmul_rn((double)c.R[3 * r + 1], (double)mu[1])),
                                    __dmul_rn((double)c.R[3 * r + 2], (double)mu[2])),
                          (double)c.t[r]);
    P.tx = (float)t3[0]; P.ty = (float)t3[1]; P.tz = (float)t3[2];
    if (!L.ok || !(t3[2] > (double)c.near_z)) return;
    const double du = t3[0] / t3[2], dv = t3[1] / t3[2];
    P.u = (float)du;
    P.v = (float)dv;
    P.uc = P.u; P.vc = P.v; P.clx = false; P.cly = false;
    if (flags & F_JCLAMP) {
        if (du > c.limx_d) { P.uc = c.limx; P.clx = true; }
        if (du < -c.limx_d) { P.uc = -c.limx; P.clx = true; }
        if (dv > c.limy_d) { P.vc = c.limy; P.cly = true; }
        if (dv < -c.limy_d) { P.vc = -c.limy; P.cly = true; }
    }
    P.mx = (float)__dadd_rn(__dmul_rn((double)c.fx, du), (double)c.cx);
    P.my = (float)__dadd_rn(__dmul_rn((double)c.fy, dv), (double)c.cy);
    float iz = 1.f / P.tz;
    P.J00 = c.fx * iz; P.J02 = -c.fx * P.uc * iz;
    P.J11 = c.fy * iz; P.J12 = -c.fy * P.vc * iz;
    for (int j = 0; j < 3; ++j) {
        P.Tm[j] = P.J00 * c.R[j] + P.J02 * c.R[6 + j];
        P.Tm[3 + j] = P.J11 * c.R[3 + j] + P.J12 * c.R[6 + j];
    }
    const float* S = L.S;
    for (int r = 0; r < 2; ++r) {
        const float* T = P.Tm + 3 * r;
        P.W[3 * r + 0] = T[0] * S[0] + T[1] * S[1] + T[2] * S[2];
        P.W[3 * r + 1] = T[0] * S[1] + T[1] * S[3] + T[2] * S[4];
        P.W[3 * r + 2] = T[0] * S[2] + T[1] * S[4] + T[2] * S[5];
    }
    float dil = (flags & F_DILATE) ? 0.3f : 0.f;
    float ca = P.W[0] * P.Tm[0] + P.W[1] * P.Tm[1] + P.W[2] * P.Tm[2] + dil;
    float cb = P.W[0] * P.Tm[3] + P.W[1] * P.Tm[4] + P.W[2] * P.Tm[5];
    float cc = P.W[3] * P.Tm[3] + P.W[4] * P.Tm[4] + P.W[5] * P.Tm[5] + dil;
    // FP64: determinant and inverse of the 2x2 covariance
    P.a = ca; P.b = cb; P.c = cc;
    P.det = P.a * P.c - P.b * P.b;
    if (!(P.det > 0.0)) return;
    double id = 1.0 / P.det;
    P.qA = P.c * id; P.qB = -P.b * id; P.qC = P.a * id;
    P.ok = true;
}

// The forward reads the cameras of a launch from LDS, kCamChunk at a time: read
// from global memory in its view loop, a camera became vector loads, whose wait
// (the shared vector-memory counter) also waited for the previous view's stores.
// The backward's pairs name their views, so its lanes read the cameras from LDS as well.
constexpr int kCamChunk = 16;
static_assert(sizeof(CamDev) % 4 == 0, "cameras are copied in 4-byte words");

// cameras [v0, v0 + nv) into s_cam, by the whole workgroup (a barrier before and after)
__device__ __forceinline__ void stage_cams(CamDev* s_cam, const CamDev* cams, int v0, int nv)
{
    __syncthreads();
    const uint32_t* src = reinterpret_cast<const uint32_t*>(cams + v0);
    uint32_t* dst = reinterpret_cast<uint32_t*>(s_cam);
    const uint32_t words = (uint32_t)nv * (uint32_t)(sizeof(CamDev) / 4);
    for (uint32_t w = threadIdx.x; w < words; w += blockDim.x) dst[w] = src[w];
    __syncthreads();
}

// ONE: a launch of one view (a constant view count; fewer registers).  COUNT: every
// workgroup also leaves its tile count of each view in a.count, and only views from
// a.store_from on are stored (as if the launch had only them): the pair counts of several
// cameras from one read of the parameters.
template <int DEG, bool BF16, bool ONE, bool COUNT>
__global__ __launch_bounds__(256) void project_fwd_kernel(ProjectFwdArgs a)
{
    constexpr int K = (DEG + 1) * (DEG + 1);
    __shared__ CamDev s_cam[kCamChunk];
    const uint32_t i0 = blockIdx.x * 256u + threadIdx.x;
    const bool active = i0 < a.n;
    const uint32_t i = active ? i0 : a.n - 1u;               // past the end: only helps stage the cameras
    float mu[3] = { a.means[3 * (size_t)i], a.means[3 * (size_t)i + 1], a.means[3 * (size_t)i + 2] };
    float s[3] = { a.scales[3 * (size_t)i], a.scales[3 * (size_t)i + 1], a.scales[3 * (size_t)i + 2] };
    float q[4] = { a.quats[4 * (size_t)i], a.quats[4 * (size_t)i + 1], a.quats[4 * (size_t)i + 2], a.quats[4 * (size_t)i + 3] };
    float op = a.opac[i];
    float sh[K * 3];
    load_sh<K, BF16>(a.sh, i, sh);
    Local L;
    local_state(mu, s, q, op, sh, K * 3, L);
    const int tsx = a.tile_shift_x, tsy = a.tile_shift_y;
    const int n_views = ONE ? 1 : a.n_views;
    for (int v0 = 0; v0 < n_views; v0 += kCamChunk) {
    const int nv = n_views - v0 < kCamChunk ? n_views - v0 : kCamChunk;
    stage_cams(s_cam, a.cams, v0, nv);
    if (!COUNT && !active) continue;
    for (int v = v0; v < v0 + nv; ++v) {
        const CamDev& c = s_cam[v - v0];
        const bool store = !COUNT || (active && v >= a.store_from);
        size_t o = (size_t)(COUNT ? v - a.store_from : v) * a.n + i;
        ViewProj P;
        view_proj(c, mu, L, a.flags, P);
        uint32_t tt = 0;
        int32_t rad = 0;
        uint2 rc = make_uint2(1u, 1u);                      // empty: x1 < x0 and y1 < y0
        float4 r0 = make_float4(0.f, 0.f, 0.f, 0.f), r1 = r0, r2 = r0;
        if (P.ok) {
            double mid = 0.5 * (P.a + P.c);
            double disc = mid * mid - P.det;
            double lam = mid + sqrt(disc > 0.0 ? disc : 0.0);
            double rr = ceil(3.0 * sqrt(lam));
            rad = rr > 1073741824.0 ? 1073741824 : (int32_t)rr;
            // tile rectangle of [mean - r, mean + r]; floor(mean) is exact in FP32
            float fx = fminf(fmaxf(floorf(P.mx), -1e9f), 1e9f);
            float fy = fminf(fmaxf(floorf(P.my), -1e9f), 1e9f);
            int64_t ix = (int64_t)fx, iy = (int64_t)fy;
            int64_t x0 = (ix - rad) >> tsx, x1 = (ix + rad) >> tsx;
            int64_t y0 = (iy - rad) >> tsy, y1 = (iy + rad) >> tsy;
            x0 = x0 < 0 ? 0 : x0;
            y0 = y0 < 0 ? 0 : y0;
            x1 = x1 > c.gx - 1 ? c.gx - 1 : x1;
            y1 = y1 > c.gy - 1 ? c.gy - 1 : y1;
            if (rad > 0 && x0 <= x1 && y0 <= y1) {
                tt = (uint32_t)((x1 - x0 + 1) * (y1 - y0 + 1));
                rc = make_uint2((uint32_t)x0 | ((uint32_t)x1 << 16), (uint32_t)y0 | ((uint32_t)y1 << 16));
            }
            // colour along the viewing direction
            if (store) {
            float dx = mu[0] - c.campos[0], dy = mu[1] - c.campos[1], dz = mu[2] - c.campos[2];
            float idn = 1.f / sqrtf(dx * dx + dy * dy + dz * dz);
            float Y[K];
            sh_basis<DEG>(dx * idn, dy * idn, dz * idn, Y);
            float col[3];
            for (int ch = 0; ch < 3; ++ch) {
                float acc = 0.f;
#pragma unroll
                for (int k = 0; k < K; ++k) acc += Y[k] * sh[3 * k + ch];
                acc += 0.5f;
                if ((a.flags & F_CCLAMP) && acc < 0.f) acc = 0.f;
                col[ch] = acc;
            }
            const float A2 = (float)(-0.5 * kLog2e * P.qA), B2 = (float)(-kLog2e * P.qB);
            const float C2 = (float)(-0.5 * kLog2e * P.qC);
            r0 = make_float4(P.mx, P.my, A2, B2);
            r1 = make_float4(C2, op, col[0], col[1]);
            // Cull level for the blend: alpha < 1/255 wherever the exponent is
            // below -L, L = log2(255 opacity) + 1e-4; and the slopes of the exponent's
            // ridge lines, where its maximum along a pixel row / column lies (dy = k dx
            // with k = -B'/(2C'), dx = k' dy with k' = -B'/(2A')).
            const double Lc = op > 0.f ? log2(255.0 * (double)op) + 1e-4 : -HUGE_VAL;
            const float kr = (float)(-(double)B2 / (2.0 * (double)C2));
            const float kc = (float)(-(double)B2 / (2.0 * (double)A2));
            r2 = make_float4(col[2], (float)Lc, kr, kc);
            }
        }
        if (COUNT) {
            uint64_t sum = active ? tt : 0u;
#pragma unroll
            for (int w = 32; w > 0; w >>= 1) sum += __shfl_xor(sum, w, 64);
            if ((threadIdx.x & 63u) == 0u)
                a.count[(size_t)v * 4u * gridDim.x + 4u * blockIdx.x + (threadIdx.x >> 6)] = sum;
            if (!store) continue;
        }
        // 64 bytes a record, most of this kernel's traffic with several views: the sort's key
        // is the depth itself and the tile count follows from the rectangle (stored apart, 72
        // bytes: 8 views of 3M 0.52 -> 0.48 ms, four of 6M 0.58 -> 0.55)
        a.rec[3 * o + 0] = r0;
        a.rec[3 * o + 1] = r1;
        a.rec[3 * o + 2] = r2;
        a.depth[o] = P.tz;
        if (a.rect8)
            reinterpret_cast<uint32_t*>(a.trect)[o] = (rc.x & 0xffu) | ((rc.x >> 16) << 8) | (rc.y << 16) | ((rc.y >> 16) << 24);
        else
            a.trect[o] = rc;
        a.radius[o] = P.ok ? rad : 0;
    }
    }
}

// LDS rows of a wavefront's SH gradients: kWords 32-bit words a Gaussian, one more apart
// (an odd stride: no bank conflicts)
template <int K, bool BF16>
struct ShRows {
    static constexpr int kBytes = K * 3 * (BF16 ? 2 : 4);
    static constexpr bool kStaged = kBytes % 16 == 0;
    static constexpr int kWords = kBytes / 4, kStride = kWords + 1;
    static constexpr int kLds = kStaged ? 256 * kStride : 1;     // words a workgroup
};

// what one (view, Gaussian) adds to its Gaussian's gradient: 16 words of LDS, one more apart
struct PairGrad {
    float mu[3], S[6], op, col[3], dir[3];
};
constexpr int kPairWords = 16, kPairStride = kPairWords + 1;
static_assert(sizeof(PairGrad) == 4 * kPairWords, "a pair's record is 16 words");
constexpr int kBwdRound = 8;                   // views a round

// The gradient one view gives a Gaussian (mean mu, SH coefficients sh, state L): its 2D row g
// back through colour, conic and mean.  False where the view does not project it (nothing
// to add).
template <int DEG>
__device__ __forceinline__ bool project_bwd_pair(uint32_t flags, const float (&mu)[3], const float (&sh)[(DEG + 1) * (DEG + 1) * 3],
                                                 const Local& L, const float (&g)[kG2], const CamDev& c, PairGrad& o)
{
    constexpr int K = (DEG + 1) * (DEG + 1);
    ViewProj P;
    view_proj(c, mu, L, flags, P);
    if (!P.ok) return false;
    const float gmx = g[0], gmy = g[1], gA = g[2], gB = g[3], gC = g[4];
    o.op = g[5];
    // ---- colour -> SH coefficients (by the caller, from dir and col) and viewing direction
    const float dx = mu[0] - c.campos[0], dy = mu[1] - c.campos[1], dz = mu[2] - c.campos[2];
    const float idn = 1.f / sqrtf(dx * dx + dy * dy + dz * dz);
    const float d0 = dx * idn, d1 = dy * idn, d2 = dz * idn;
    o.dir[0] = d0; o.dir[1] = d1; o.dir[2] = d2;
    float Y[K];
    sh_basis<DEG>(d0, d1, d2, Y);
    for (int ch = 0; ch < 3; ++ch) {
        float acc = 0.f;
#pragma unroll
        for (int k = 0; k < K; ++k) acc += Y[k] * sh[3 * k + ch];
        acc += 0.5f;
        const bool clamped = (flags & F_CCLAMP) && acc < 0.f;
        o.col[ch] = clamped ? 0.f : g[6 + ch];
    }
    float gmu[3] = { 0.f, 0.f, 0.f };
    if constexpr (DEG > 0) {
        float wk[K];
#pragma unroll
        for (int k = 0; k < K; ++k) wk[k] = sh[3 * k] * o.col[0] + sh[3 * k + 1] * o.col[1] + sh[3 * k + 2] * o.col[2];
        const float3 gd = sh_basis_grad<DEG>(d0, d1, d2, wk);
        const float dd = d0 * gd.x + d1 * gd.y + d2 * gd.z;
        gmu[0] = (gd.x - d0 * dd) * idn;
        gmu[1] = (gd.y - d1 * dd) * idn;
        gmu[2] = (gd.z - d2 * dd) * idn;
    }
    // ---- conic -> 2D covariance (FP64): dL/dSigma' = -Q G Q, G the symmetric gradient of Q
    const double hB = 0.5 * (double)gB;
    const double QG00 = P.qA * gA + P.qB * hB, QG01 = P.qA * hB + P.qB * gC;
    const double QG10 = P.qB * gA + P.qC * hB, QG11 = P.qB * hB + P.qC * gC;
    const float g00 = (float)(-(QG00 * P.qA + QG01 * P.qB));
    const float g01 = (float)(-(QG00 * P.qB + QG01 * P.qC));
    const float g11 = (float)(-(QG10 * P.qB + QG11 * P.qC));
    // ---- Sigma' = Tm Sigma Tm^T: dL/dSigma += Tm^T GS Tm ; dL/dTm = 2 GS Tm Sigma = 2 GS W
    const float* T0 = P.Tm;
    const float* T1 = P.Tm + 3;
    int idx = 0;
    for (int k = 0; k < 3; ++k)
        for (int l = k; l < 3; ++l, ++idx)
            o.S[idx] = g00 * T0[k] * T0[l] + g01 * (T0[k] * T1[l] + T1[k] * T0[l]) + g11 * T1[k] * T1[l];
    float gTm[6];
    for (int j = 0; j < 3; ++j) {
        gTm[j] = 2.f * (g00 * P.W[j] + g01 * P.W[3 + j]);
        gTm[3 + j] = 2.f * (g01 * P.W[j] + g11 * P.W[3 + j]);
    }
    // dL/dJ = dL/dTm Rc^T (only the four non-zero entries of J matter)
    const float gJ00 = gTm[0] * c.R[0] + gTm[1] * c.R[1] + gTm[2] * c.R[2];
    const float gJ02 = gTm[0] * c.R[6] + gTm[1] * c.R[7] + gTm[2] * c.R[8];
    const float gJ11 = gTm[3] * c.R[3] + gTm[4] * c.R[4] + gTm[5] * c.R[5];
    const float gJ12 = gTm[3] * c.R[6] + gTm[4] * c.R[7] + gTm[5] * c.R[8];
    // ---- J and the 2D mean -> camera-space position
    const float iz = 1.f / P.tz, iz2 = iz * iz;
    float gtx = 0.f, gty = 0.f, gtz = 0.f;
    gtz += -(gJ00 * c.fx + gJ11 * c.fy) * iz2;
    if (!P.clx) { gtx += -gJ02 * c.fx * iz2; gtz += 2.f * gJ02 * c.fx * P.tx * iz2 * iz; }
    else        { gtz += gJ02 * c.fx * P.uc * iz2; }
    if (!P.cly) { gty += -gJ12 * c.fy * iz2; gtz += 2.f * gJ12 * c.fy * P.ty * iz2 * iz; }
    else        { gtz += gJ12 * c.fy * P.vc * iz2; }
    gtx += gmx * c.fx * iz;
    gty += gmy * c.fy * iz;
    gtz -= (gmx * c.fx * P.tx + gmy * c.fy * P.ty) * iz2;
    for (int k = 0; k < 3; ++k) o.mu[k] = gmu[k] + (c.R[k] * gtx + c.R[3 + k] * gty + c.R[6 + k] * gtz);
    return true;
}

// Gaussian i's parameters and their state
template <int DEG, bool BF16>
__device__ __forceinline__ void load_gaussian(const ProjectBwdArgs& a, uint32_t i, float (&mu)[3],
                                              float (&sh)[(DEG + 1) * (DEG + 1) * 3], Local& L)
{
    constexpr int K = (DEG + 1) * (DEG + 1);
    for (int k = 0; k < 3; ++k) mu[k] = a.means[3 * (size_t)i + k];
    const float s[3] = { a.scales[3 * (size_t)i], a.scales[3 * (size_t)i + 1], a.scales[3 * (size_t)i + 2] };
    const float q[4] = { a.quats[4 * (size_t)i], a.quats[4 * (size_t)i + 1], a.quats[4 * (size_t)i + 2], a.quats[4 * (size_t)i + 3] };
    load_sh<K, BF16>(a.sh, i, sh);
    local_state(mu, s, q, a.opac[i], sh, K * 3, L);
}

// the row of a (view, Gaussian)
__device__ __forceinline__ void load_row(const ProjectBwdArgs& a, uint32_t i, int v, float (&g)[kG2])
{
#pragma unroll
    for (int k = 0; k < kG2; ++k) g[k] = a.grad2d[(size_t)kG2 * ((size_t)v * a.n + i) + k];
}

// A workgroup owns 256 Gaussians.  Which of their (view, Gaussian) rows are this
// frame's (the others are zero: no pixel blended the record) is read from the row
// stamps, 8 views a round; the live pairs of a round are listed in LDS, Gaussian by
// Gaussian with the views in order, and worked on one a thread, 256 at a time; then each
// Gaussian's thread adds its pairs in that order.  So lanes are full whichever Gaussians
// and views are live, and a Gaussian with no live row reads nothing but its stamps: on 8
// views of 3M Gaussians 12 % of the pairs are live and 64 % of the Gaussians have none,
// while a thread a Gaussian that looped over the views ran at 0.29 of its lanes and read
// every parameter.  Bound by HBM, and with several views by the latency of its phases
// at two workgroups a CU (the 48 SH sums stay in registers over the rounds).  One view of
// 3.3M FP32 degree-3 Gaussians: 0.41 -> 0.20 ms (4.0 TB/s of what it has to move); 200k:
// 29 -> 21 us; 8 views of 3M, BF16: 0.53 -> 0.41 ms.
// EACH (several views of at most kBwdEach Gaussians): a Gaussian a thread after all, its
// parameters read once and the next live view's row a view ahead.
template <int DEG, bool BF16, bool ONE, bool EACH>
__global__ __launch_bounds__(256, ONE ? 3 : EACH ? 1 : 2) void project_bwd_kernel(ProjectBwdArgs a)
{
    constexpr int K = (DEG + 1) * (DEG + 1);
    constexpr int kBwdViews = ONE ? 1 : kBwdRound;
    using RL = ShRows<K, BF16>;
    constexpr int kPairLds = 256 * kPairStride;
    // the pairs' records, later the SH gradients' rows
    __shared__ uint32_t s_mem[kPairLds > RL::kLds ? kPairLds : RL::kLds];
    __shared__ uint16_t s_list[256 * kBwdViews];             // local Gaussian | view << 8
    __shared__ uint32_t s_wave[256 / 64];
    __shared__ CamDev s_cam[kBwdViews];
    const uint32_t tid = threadIdx.x, lane = tid & 63u, wid = tid >> 6;
    const uint32_t base = blockIdx.x * 256u, i = base + tid;
    const bool active = i < a.n;
    // the opacity regulariser's loss (Sec. 5.4 ablation): per-wavefront FP64 sums of
    // exp(-(sigma - 0.5)^2 / 0.05), in a fixed order, for a fixed-order final sum
    double e = 0.0;
    if (a.reg_partial && active) {
        const float d = a.opac[i] - 0.5f;
        e = (double)expf(-(d * d) * 20.0f);                  // 1 / 0.05 = 20
    }
    const uint32_t st = *a.stamp;

    float gmu[3] = { 0.f, 0.f, 0.f };
    float gS[6] = { 0.f, 0.f, 0.f, 0.f, 0.f, 0.f };   // symmetric dL/dSigma, upper triangle
    float gop = 0.f;
    float gsh[K * 3];
#pragma unroll
    for (int k = 0; k < K * 3; ++k) gsh[k] = 0.f;
    bool live = false;

    auto add = [&](const PairGrad& o) {
#pragma unroll
        for (int w = 0; w < 3; ++w) gmu[w] += o.mu[w];
#pragma unroll
        for (int w = 0; w < 6; ++w) gS[w] += o.S[w];
        gop += o.op;
        float Y[K];
        sh_basis<DEG>(o.dir[0], o.dir[1], o.dir[2], Y);
#pragma unroll
        for (int w = 0; w < K; ++w) {
            gsh[3 * w + 0] += Y[w] * o.col[0];
            gsh[3 * w + 1] += Y[w] * o.col[1];
            gsh[3 * w + 2] += Y[w] * o.col[2];
        }
    };
    float mu[3], sh[K * 3];                              // EACH
    Local L;
    const int n_views = ONE ? 1 : a.n_views;
    for (int v0 = 0; v0 < n_views; v0 += kBwdViews) {
        const int nv = n_views - v0 < kBwdViews ? n_views - v0 : kBwdViews;
        // this Gaussian's live views (every stamp in flight at once)
        uint32_t r[kBwdViews], mask = 0u;
#pragma unroll
        for (int k = 0; k < kBwdViews; ++k)
            r[k] = a.rec_stamp[(size_t)(v0 + (k < nv ? k : nv - 1)) * a.n + (active ? i : a.n - 1u)];
#pragma unroll
        for (int k = 0; k < kBwdViews; ++k)
            if (active && k < nv && r[k] == st) mask |= 1u << k;
        const uint32_t cnt = (uint32_t)__popc(mask);
        if constexpr (EACH) {
            __syncthreads();
            const uint32_t* src = reinterpret_cast<const uint32_t*>(a.cams + v0);
            for (uint32_t w = tid; w < (uint32_t)nv * (uint32_t)(sizeof(CamDev) / 4); w += 256u)
                reinterpret_cast<uint32_t*>(s_cam)[w] = src[w];
            __syncthreads();
            if (mask == 0u) continue;
            if (!live) load_gaussian<DEG, BF16>(a, i, mu, sh, L);
            live = true;
            float gn[kG2];
            load_row(a, i, v0 + (__ffs((int)mask) - 1), gn);
            for (uint32_t m = mask; m;) {
                const int v = __ffs((int)m) - 1;
                float g[kG2];
#pragma unroll
                for (int k = 0; k < kG2; ++k) g[k] = gn[k];
                m &= m - 1u;
                if (m) load_row(a, i, v0 + (__ffs((int)m) - 1), gn);     // (one view ahead)
                PairGrad o;
                if (project_bwd_pair<DEG>(a.flags, mu, sh, L, g, s_cam[v], o)) add(o);
            }
            continue;
        }
        live = live || cnt != 0u;
        uint32_t inc = cnt;
#pragma unroll
        for (int o = 1; o < 64; o <<= 1) {
            const uint32_t y = __shfl_up(inc, o, 64);
            if (lane >= (uint32_t)o) inc += y;
        }
        __syncthreads();                                     // (the last round's reads are done)
        if (lane == 63u) s_wave[wid] = inc;
        {   // the round's cameras
            const uint32_t* src = reinterpret_cast<const uint32_t*>(a.cams + v0);
            for (uint32_t w = tid; w < (uint32_t)nv * (uint32_t)(sizeof(CamDev) / 4); w += 256u)
                reinterpret_cast<uint32_t*>(s_cam)[w] = src[w];
        }
        __syncthreads();
        uint32_t first = inc - cnt, total = 0u;
#pragma unroll
        for (uint32_t w = 0; w < 256u / 64u; ++w) {
            if (w < wid) first += s_wave[w];
            total += s_wave[w];
        }
        uint32_t at = first;
        for (uint32_t m = mask; m; m &= m - 1u) s_list[at++] = (uint16_t)(tid | ((uint32_t)(__ffs(m) - 1) << 8));
        __syncthreads();
        for (uint32_t c0 = 0; c0 < (ONE ? 1u : total); c0 += 256u) {
            if (c0 + tid < total) {
                const uint32_t e2 = s_list[c0 + tid], v = e2 >> 8;
                const uint32_t own = base + (e2 & 0xffu);
                float g[kG2], pmu[3], psh[K * 3];
                Local pl;
                load_row(a, own, v0 + (int)v, g);
                load_gaussian<DEG, BF16>(a, own, pmu, psh, pl);
                PairGrad o;
                if (!project_bwd_pair<DEG>(a.flags, pmu, psh, pl, g, s_cam[v], o)) {
                    o = PairGrad{};
                    o.dir[2] = 1.f;
                }
                float* dst = reinterpret_cast<float*>(s_mem) + tid * kPairStride;
#pragma unroll
                for (int k = 0; k < kPairWords; ++k) dst[k] = reinterpret_cast<const float*>(&o)[k];
            }
            __syncthreads();
            const uint32_t k0 = ONE || first > c0 ? first : c0;
            const uint32_t k1 = ONE || first + cnt < c0 + 256u ? first + cnt : c0 + 256u;
            for (uint32_t k = k0; k < k1; ++k) {
                PairGrad o;
                const float* src = reinterpret_cast<const float*>(s_mem) + (k - c0) * kPairStride;
#pragma unroll
                for (int w = 0; w < kPairWords; ++w) reinterpret_cast<float*>(&o)[w] = src[w];
                add(o);
            }
            __syncthreads();
        }
    }

    float s[3] = { 0.f, 0.f, 0.f }, q[4] = { 0.f, 0.f, 0.f, 0.f };
    if (live) {
#pragma unroll
        for (int k = 0; k < 3; ++k) s[k] = a.scales[3 * (size_t)i + k];
#pragma unroll
        for (int k = 0; k < 4; ++k) q[k] = a.quats[4 * (size_t)i + k];
    }
    // a live row's Gaussian was projected, so its inputs are finite and its quaternion not zero
    const float qnorm = sqrtf(q[0] * q[0] + q[1] * q[1] + q[2] * q[2] + q[3] * q[3]);
    const float iq = live ? 1.f / qnorm : 0.f;
    const float w = q[0] * iq, x = q[1] * iq, y = q[2] * iq, z = q[3] * iq;
    float R[9];
    quat_to_rot(w, x, y, z, R);
    // ---- Sigma = M M^T with M = R diag(s):  dL/dM = 2 G M
    float G[9] = { gS[0], gS[1], gS[2], gS[1], gS[3], gS[4], gS[2], gS[4], gS[5] };
    float M[9];
    for (int r = 0; r < 3; ++r)
        for (int j = 0; j < 3; ++j) M[3 * r + j] = R[3 * r + j] * s[j];
    // (the sums that cancel are written as the multiply-adds they are, so that their
    // rounding is not the compiler's choice of what to fuse)
    float gR[9], gs[3] = { 0.f, 0.f, 0.f }, gm = 0.f;
    for (int r = 0; r < 3; ++r)
        for (int j = 0; j < 3; ++j) {
            gm = 2.f * fmaf(G[3 * r + 2], M[6 + j], fmaf(G[3 * r + 1], M[3 + j], G[3 * r] * M[j]));
            gs[j] += gm * R[3 * r + j];
            gR[3 * r + j] = gm * s[j];
        }
    const float gR48 = fmaf(gm, s[2], gR[4]);                // gR[4] + gR[8]
    // ---- rotation -> normalised quaternion -> raw quaternion
    float gw = 2.f * (-z * gR[1] + y * gR[2] + z * gR[3] - x * gR[5] - y * gR[6] + x * gR[7]);
    float gx = 2.f * (fmaf(y, gR[1], z * gR[2]) + y * gR[3] - w * gR[5] + z * gR[6] + w * gR[7]) -
               4.f * x * gR48;
    float gy = 2.f * (fmaf(x, gR[1], w * gR[2]) + x * gR[3] + z * gR[5] - w * gR[6] + z * gR[7]) -
               4.f * y * (gR[0] + gR[8]);
    float gz = 2.f * (-w * gR[1] + x * gR[2] + w * gR[3] + y * gR[5] + x * gR[6] + y * gR[7]) -
               4.f * z * (gR[0] + gR[4]);
    float qd = w * gw + x * gx + y * gy + z * gz;

    // Every lane stores: a Gaussian without a live row its zeros, with its neighbours'
    // gradients (stored apart, the lines they share went to memory twice: 0.53 -> 0.81 ms
    // on 8 views).
    if (active) {
        a.g_means[3 * (size_t)i + 0] = live ? gmu[0] : 0.f;
        a.g_means[3 * (size_t)i + 1] = live ? gmu[1] : 0.f;
        a.g_means[3 * (size_t)i + 2] = live ? gmu[2] : 0.f;
        a.g_scales[3 * (size_t)i + 0] = live ? gs[0] : 0.f;
        a.g_scales[3 * (size_t)i + 1] = live ? gs[1] : 0.f;
        a.g_scales[3 * (size_t)i + 2] = live ? gs[2] : 0.f;
        a.g_quats[4 * (size_t)i + 0] = live ? (gw - w * qd) * iq : 0.f;
        a.g_quats[4 * (size_t)i + 1] = live ? (gx - x * qd) * iq : 0.f;
        a.g_quats[4 * (size_t)i + 2] = live ? (gy - y * qd) * iq : 0.f;
        a.g_quats[4 * (size_t)i + 3] = live ? (gz - z * qd) * iq : 0.f;
        float go = live ? gop : 0.f;
        if (a.reg_w != 0.f) {                                // + dL_O/dsigma, as a separate pass would add it
            const float d = a.opac[i] - 0.5f;
            const float ex = expf(-(d * d) * 20.0f);
            go += (a.reg_w / (float)a.n) * ex * (-40.0f * d);
        }
        a.g_opac[i] = go;
    }
    // SH gradients: through LDS, so that the workgroup stores its Gaussians' range as
    // consecutive 16-byte words (from the lanes' own rows, 16 bytes each at a stride of a
    // row, every store touched 64 lines in part: 0.35 instead of 0.27 ms at 3.3M, one view)
    const bool staged = RL::kStaged && (reinterpret_cast<uintptr_t>(a.g_sh) & 15u) == 0u;
    if (staged) {
        uint32_t* row = s_mem + tid * RL::kStride;
#pragma unroll
        for (int k = 0; k < RL::kWords; ++k) {
            if constexpr (BF16)
                row[k] = (uint32_t)f32_to_bf16_rne(gsh[2 * k]) | ((uint32_t)f32_to_bf16_rne(gsh[2 * k + 1]) << 16);
            else
                row[k] = __float_as_uint(gsh[k]);
        }
        __syncthreads();
        const uint32_t n_own = base < a.n ? (a.n - base < 256u ? a.n - base : 256u) : 0u;
        constexpr uint32_t kQ = RL::kWords / 4 > 0 ? RL::kWords / 4 : 1;         // 16-byte words a Gaussian
        uint4* dst = reinterpret_cast<uint4*>(a.g_sh) + (size_t)base * kQ;
#pragma unroll
        for (uint32_t r = 0; r < kQ; ++r) {
            const uint32_t f = r * 256u + tid, g = f / kQ;
            const uint32_t* src = s_mem + g * RL::kStride + 4u * (f - g * kQ);
            if (g < n_own) dst[f] = make_uint4(src[0], src[1], src[2], src[3]);
        }
    } else if (active) {
        if constexpr (BF16) {
            uint16_t* p = reinterpret_cast<uint16_t*>(a.g_sh) + (size_t)i * (K * 3);
#pragma unroll
            for (int k = 0; k < K * 3; ++k) p[k] = f32_to_bf16_rne(gsh[k]);
        } else {
            float* p = reinterpret_cast<float*>(a.g_sh) + (size_t)i * (K * 3);
#pragma unroll
            for (int k = 0; k < K * 3; ++k) p[k] = gsh[k];
        }
    }
    if (a.reg_partial) {
#pragma unroll
        for (int o = 32; o > 0; o >>= 1) e += __shfl_xor(e, o, 64);
        if (lane == 0u) a.reg_partial[4u * blockIdx.x + wid] = e;
    }
}

// one workgroup a view: the sum of its n counts
__global__ __launch_bounds__(256) void count_reduce_kernel(const uint64_t* count, uint32_t n, uint64_t* total)
{
    __shared__ uint64_t s_w[256 / 64];
    const uint64_t* c = count + (size_t)blockIdx.x * n;
    uint64_t sum = 0;
    for (uint32_t b0 = threadIdx.x; b0 < n; b0 += 8u * 256u) {
        uint64_t v[8];
#pragma unroll
        for (uint32_t k = 0; k < 8u; ++k) v[k] = b0 + k * 256u < n ? c[b0 + k * 256u] : 0u;
#pragma unroll
        for (uint32_t k = 0; k < 8u; ++k) sum += v[k];
    }
#pragma unroll
    for (int w = 32; w > 0; w >>= 1) sum += __shfl_xor(sum, w, 64);
    if ((threadIdx.x & 63u) == 0u) s_w[threadIdx.x >> 6] = sum;
    __syncthreads();
    if (threadIdx.x == 0) total[blockIdx.x] = s_w[0] + s_w[1] + s_w[2] + s_w[3];
}

template <int DEG, bool BF16>
hipError_t fwd_dispatch(const ProjectFwdArgs& a, hipStream_t s)
{
    dim3 grid((a.n + 255u) / 256u);
    if (a.count) {
        hipLaunchKernelGGL((project_fwd_kernel<DEG, BF16, false, true>), grid, dim3(256), 0, s, a);
        hipLaunchKernelGGL(count_reduce_kernel, dim3((unsigned)a.n_views), dim3(256), 0, s, a.count, 4u * grid.x,
                           a.count_total);
    } else if (a.n_views == 1) hipLaunchKernelGGL((project_fwd_kernel<DEG, BF16, true, false>), grid, dim3(256), 0, s, a);
    else hipLaunchKernelGGL((project_fwd_kernel<DEG, BF16, false, false>), grid, dim3(256), 0, s, a);
    return hipGetLastError();
}

// several views: a Gaussian a thread, or its live pairs compacted?  The first while the launch is
// short of wavefronts or most pairs are live, the second where it reads the parameters of few
// of many.  Both sides, first / second in us: 8 views of 400x300, 2k Gaussians 19 / 45, 60k 22 /
// 47, 300k 71 / 102, 1M 190 / 190; of 972x648, 1M 218 / 238; two views of 972x648, 1M 105 / 113, 3M
// 302 / 280; 8 views of 9.76 Mpixel, 3M in BF16 493 / 408.
constexpr uint32_t kBwdEach = 1u << 20;
template <int DEG, bool BF16>
hipError_t bwd_dispatch(const ProjectBwdArgs& a, hipStream_t s)
{
    dim3 grid((a.n + 255u) / 256u);
    if (a.n_views == 1) hipLaunchKernelGGL((project_bwd_kernel<DEG, BF16, true, false>), grid, dim3(256), 0, s, a);
    else if (a.n <= kBwdEach) hipLaunchKernelGGL((project_bwd_kernel<DEG, BF16, false, true>), grid, dim3(256), 0, s, a);
    else hipLaunchKernelGGL((project_bwd_kernel<DEG, BF16, false, false>), grid, dim3(256), 0, s, a);
    return hipGetLastError();
}

}  // namespace

hipError_t launch_project_fwd(const ProjectFwdArgs& a, int deg, bool bf16, hipStream_t s)
{
    if (a.n == 0) return hipSuccess;
    switch (deg * 2 + (bf16 ? 1 : 0)) {
        case 0: return fwd_dispatch<0, false>(a, s);
        case 1: return fwd_dispatch<0, true>(a, s);
        case 2: return fwd_dispatch<1, false>(a, s);
        case 3: return fwd_dispatch<1, true>(a, s);
        case 4: return fwd_dispatch<2, false>(a, s);
        case 5: return fwd_dispatch<2, true>(a, s);
        case 6: return fwd_dispatch<3, false>(a, s);
        case 7: return fwd_dispatch<3, true>(a, s);
    }
    return hipErrorInvalidValue;
}

hipError_t launch_project_bwd(const ProjectBwdArgs& a, int deg, bool bf16, hipStream_t s)
{
    if (a.n == 0) return hipSuccess;
    switch (deg * 2 + (bf16 ? 1 : 0)) {
        case 0: return bwd_dispatch<0, false>(a, s);
        case 1: return bwd_dispatch<0, true>(a, s);
        case 2: return bwd_dispatch<1, false>(a, s);
        case 3: return bwd_dispatch<1, true>(a, s);
        case 4: return bwd_dispatch<2, false>(a, s);
        case 5: return bwd_dispatch<2, true>(a, s);
        case 6: return bwd_dispatch<3, false>(a, s);
        case 7: return bwd_dispatch<3, true>(a, s);
    }
    return hipErrorInvalidValue;
}

}  // namespace gsr
