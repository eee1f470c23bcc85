// Front-to-back alpha blending with the entropy of the blending weights
// (Sec. 3, Eq. 3-5; Sec. 4.3, Eq. 8-11) and the back-to-front backward with
// the O(N) entropy gradient of Alg. 1 (Sec. 4.4, Eq. 13-15; Suppl. C).
//
// Work decomposition.  Every 64-lane wavefront owns one 8x8 pixel block (one
// pixel per lane) and walks the Gaussian list of the tile that contains it.
// Wave blocks are numbered tile-major: a 16x16 or 32x8 tile is one workgroup
// of 4 wavefronts (its 4 blocks), an 8x8 tile is one wavefront.  The tile
// shape sets the sort granularity; the wavefront sets the blend granularity.
//
// Forward, four forms with the same outputs.  Per block: each wavefront stages its list in LDS in
// batches of B records (its own LDS region: no workgroup barrier, and a
// wavefront whose 64 pixels have all stopped leaves at the next batch
// boundary).  Shared (16x16 and 32x8 tiles, long lists): the 4 wavefronts of a
// tile stage each batch once, one entry per thread, and the tile's batch loop
// ends when none of its pixels is open.  Slotted (few blocks): four wavefronts a
// block, four list entries a step.  Mixed (mid-sized launches of short lists): the
// longest tiles slotted, the others per block.
//
// Culling: while staging, every wavefront drops the Gaussians that cannot
// reach alpha >= 1/255 at any pixel centre of its 8x8 block: the exact maximum
// of the (concave) exponent over the block's pixel-centre rectangle, plus a
// bound on the FP32 evaluation error, is below the skip threshold.  Those
// entries would be skipped by every lane anyway, so results are unchanged;
// the list walk only visits the survivors, compacted in list order.
//
// Backward: list windows of B entries are walked from the back (in the slotted form
// too, with 4x4 blocks and four entries a step).  In a 16x16
// or 32x8 tile the 4 wavefronts share each window's records.  An entry that
// no lane of a wavefront blended is skipped by that wavefront.  Per Gaussian,
// every wavefront sums its 9 partial gradients over its 64 lanes (half and
// row lane swaps, then DPP) and writes them to its own LDS slot; the window's
// slots (one per wavefront) are summed in a fixed order and stored once per
// (tile, Gaussian) pair, in the pair's emission slot.  A segmented reduction
// over each Gaussian's contiguous emission range then yields its 2D gradient.
// No float atomics touch global memory, so gradients are bit-reproducible.
//
// The conic is stored pre-scaled by -log2(e)/2 (-log2(e) for B) so the
// exponent is in log2 units: alpha = min(0.99, opacity * 2^p); the entropy is
// accumulated in log2 units and scaled by ln 2 once per pixel.
#include "internal.h"

namespace gsr {
namespace {

constexpr float kAlphaMax = 0.99f;
constexpr float kAlphaMin = 1.0f / 255.0f;
constexpr float kTStop = 1e-4f;
constexpr float kLn2 = 0.6931471805599453f;
constexpr int kWavesPerGroup = 4;
constexpr int kAccF = 10;            // floats per backward accumulator row: 9 sums and a hit flag
constexpr int kFwdRecF4 = kRecF4 + 1; // a staged forward entry: the record and its list position

__device__ __forceinline__ void wave_lds_sync()
{
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// exponent (log2 units) of the 2D Gaussian at offset (dx, dy) = mean - pixel:
//   p = A' dx^2 + B' dx dy + C' dy^2  with the pre-scaled conic (A', B', C');
// explicit FMAs so forward and backward produce bit-identical alphas.
__device__ __forceinline__ float gauss_p2(float A2, float B2, float C2, float dx, float dy)
{
    return fmaf(dx, fmaf(A2, dx, B2 * dy), (C2 * dy) * dy);
}

template <int CTRL, int ROW_MASK>
__device__ __forceinline__ float dpp_f(float v)
{
    return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), CTRL, ROW_MASK, 0xf, true));
}

// Wavefront sums of the 9 per-pixel gradient terms of one list entry, by
// folding registers in pairs so that one add serves two values: the gfx950
// lane swaps between the two 32-lane halves and between neighbouring 16-lane
// rows, then inside each row a rotation by 8 lanes, a half-row mirror and a
// quad sum.  Fixed order: bit-reproducible.  The total of o[c] ends in lane
// tot_lane(c): lanes 16 r and 16 r + 8 hold o[row_comp(r)] and
// o[4 + row_comp(r)], lane 4 holds o[8] (see wave_sum9).
__device__ __forceinline__ int row_comp(uint32_t r) { return (int)(((r & 1u) << 1) | (r >> 1)); }

// the component whose wavefront total wave_sum9 leaves in this lane, or -1
__device__ __forceinline__ int tot_comp(uint32_t lane)
{
    const uint32_t q = lane & 15u;
    return q == 0u ? row_comp(lane >> 4) : (q == 8u ? 4 + row_comp(lane >> 4) : (lane == 4u ? 8 : -1));
}

// lanes 0-31: x[l] + x[l + 32]; lanes 32-63: y[l - 32] + y[l]
__device__ __forceinline__ float fold_halves(float x, float y)
{
    const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(y), false, false);
    return __uint_as_float(r[0]) + __uint_as_float(r[1]);
}

// rows (0, 1, 2, 3) <- (x.r0 + x.r1, y.r0 + y.r1, x.r2 + x.r3, y.r2 + y.r3), lane by lane
__device__ __forceinline__ float fold_rows(float x, float y)
{
    const auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(x), __float_as_uint(y), false, false);
    return __uint_as_float(r[0]) + __uint_as_float(r[1]);
}

// LDS_FOLD: o[8], which has no partner, has its halves and rows added through the LDS
// crossbar (ds_bpermute, no register copy), else by lane swaps with a copy of itself
// (two VALU operations more, one LDS round trip less: the per-block backward, which
// runs at three wavefronts a SIMD, is faster so; the shared one, at eight, is not)
template <bool LDS_FOLD>
__device__ __forceinline__ float wave_sum9(const float* o, uint32_t lane)
{
    const float u0 = fold_halves(o[0], o[1]), u1 = fold_halves(o[2], o[3]);
    const float u2 = fold_halves(o[4], o[5]), u3 = fold_halves(o[6], o[7]);
    const float u4 = LDS_FOLD ? o[8] + __shfl_xor(o[8], 32, 64) : fold_halves(o[8], o[8]);
    // row r: x0 holds 16 partial sums of o[row_comp(r)], x1 of o[4 + row_comp(r)], x2 of o[8]
    const float x0 = fold_rows(u0, u1), x1 = fold_rows(u2, u3);
    const float x2 = LDS_FOLD ? u4 + __shfl_xor(u4, 16, 64) : fold_rows(u4, u4);
    // row_ror:8 adds lane l ^ 8: 8 partials in each half row
    const float a0 = x0 + dpp_f<0x128, 0xf>(x0);
    const float a1 = x1 + dpp_f<0x128, 0xf>(x1);
    const float a2 = x2 + dpp_f<0x128, 0xf>(x2);
    const float y0 = (lane & 8u) ? a1 : a0;         // lanes 0-7: o[rc], lanes 8-15: o[4 + rc]
    // row_half_mirror adds lane 7 - l of the same half row: 4 partials
    const float b0 = y0 + dpp_f<0x141, 0xf>(y0);
    const float b2 = a2 + dpp_f<0x141, 0xf>(a2);
    const float z = (lane & 4u) ? b2 : b0;          // quads: o[rc], o[8], o[4 + rc], o[8]
    float t = z + dpp_f<0xb1, 0xf>(z);              // quad_perm [1,0,3,2]
    t += dpp_f<0x4e, 0xf>(t);                       // quad_perm [2,3,0,1]
    return t;
}

__device__ __forceinline__ int wave_max_i32(int x)
{
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) {
        int y = __shfl_xor(x, o, 64);
        x = x > y ? x : y;
    }
    return x;
}

__device__ __forceinline__ int wave_sum_all_i(int x)
{
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) x += __shfl_xor(x, o, 64);
    return x;
}

__device__ __forceinline__ float wave_sum_all(float x)
{
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) x += __shfl_xor(x, o, 64);
    return x;
}

struct BlockGeom {
    int view;
    uint32_t tx, ty;                 // tile coordinates in the view
    int px, py;
    bool inside;
    uint32_t tile;
    int64_t pix;
    float cx0, cx1, cy0, cy1;        // pixel-centre rectangle of the block's in-image pixels
};

// max over v in [v0, v1] of the concave f(v) = a u^2 + b u v + c v^2 (c < 0), whose
// stationary point is v = k u with k = -b / (2 c)
__device__ __forceinline__ float edge_max(float a, float b, float c, float u, float v0, float v1, float k)
{
    const float v = fminf(fmaxf(k * u, v0), v1);
    return fmaf(u, fmaf(a, u, b * v), (c * v) * v);
}

// true if the Gaussian cannot reach alpha >= 1/255 at any pixel centre of the
// block: r0 = (mean, A', B'), c2 = C', r2 = (blue, L, -B'/(2C'), -B'/(2A')) with
// L = log2(255 opacity) + 1e-4.  The exponent is concave with its maximum 0 at the
// mean; over a rectangle that does not contain the mean its maximum lies on a side
// that faces the mean (the mean is outside that side's half-plane), and at most one
// side per axis faces it.  So two edge maxima give the exact maximum: the facing
// side of each axis, or, for an axis whose range holds the mean, any side of it
// (a value inside the rectangle, which cannot exceed the maximum).  The blend
// evaluates the exponent in FP32 with an error below 1e-6 (|A'|+|B'|+|C'|) |d|^2;
// the test adds twice that bound (and 1.5 % more) to the maximum.
__device__ __forceinline__ bool culled(const BlockGeom& g, float4 r0, float c2, float4 r2)
{
    const float a = r0.z, b = r0.w, c = c2;
    const float eps = 2.03e-6f * (fabsf(a) + fabsf(b) + fabsf(c));
    const float u0 = g.cx0 - r0.x, u1 = g.cx1 - r0.x;       // pixel - mean
    const float v0 = g.cy0 - r0.y, v1 = g.cy1 - r0.y;
    const float uf = u0 > 0.f ? u0 : u1;                    // the side facing the mean (if any)
    const float vf = v0 > 0.f ? v0 : v1;
    float qmax = fmaxf(edge_max(a, b, c, uf, v0, v1, r2.z), edge_max(c, b, a, vf, u0, u1, r2.w));
    if (u0 <= 0.f && u1 >= 0.f && v0 <= 0.f && v1 >= 0.f) qmax = 0.f;    // the mean lies over the block
    const float um = fmaxf(fabsf(u0), fabsf(u1)), vm = fmaxf(fabsf(v0), fabsf(v1));
    const float dmax2 = fmaf(um, um, vm * vm);
    return qmax + eps * dmax2 < -r2.y;
}

// wave block id -> view, tile, pixel of this lane (tile-major numbering,
// `spt` = 8x8 blocks per tile: 1 or 4)
__device__ __forceinline__ BlockGeom block_geom(const CamDev* cams, int n_views, uint32_t wb, uint32_t lane,
                                                int tsx, int tsy, int spt)
{
    BlockGeom g;
    const uint32_t tile = wb / (uint32_t)spt, sub = wb % (uint32_t)spt;
    int v = 0;
    while (v + 1 < n_views && cams[v + 1].tile_base <= tile) ++v;
    const CamDev& c = cams[v];
    const uint32_t lt = tile - c.tile_base;
    const uint32_t tx = lt % (uint32_t)c.gx, ty = lt / (uint32_t)c.gx;
    uint32_t sx = 0, sy = 0;
    if (spt == 4) {
        if (tsx == 4) { sx = sub & 1u; sy = sub >> 1; }   // 16x16: 2x2 blocks
        else { sx = sub; sy = 0; }                         // 32x8: 4x1 blocks
    }
    g.view = v;
    g.tx = tx;
    g.ty = ty;
    g.tile = tile;
    g.px = (int)((tx << tsx) + sx * kBlockPx + (lane & 7u));
    g.py = (int)((ty << tsy) + sy * kBlockPx + (lane >> 3));
    g.inside = g.px < c.W && g.py < c.H;
    g.pix = c.pix_base + (int64_t)g.py * c.W + g.px;
    const int bx0 = (int)((tx << tsx) + sx * kBlockPx), by0 = (int)((ty << tsy) + sy * kBlockPx);
    g.cx0 = (float)bx0 + 0.5f;
    g.cy0 = (float)by0 + 0.5f;
    g.cx1 = (float)min(bx0 + kBlockPx - 1, c.W - 1) + 0.5f;
    g.cy1 = (float)min(by0 + kBlockPx - 1, c.H - 1) + 0.5f;
    return g;
}

// Persistent scheduling.  The n items (in tile-major, i.e. spatial, order) are
// split into kQueues contiguous ranges, one per XCD: workgroups are dispatched
// to the XCDs round-robin, so workgroup b serves queue b % kQueues first and
// neighbouring tiles, which share most of their Gaussians, meet in one XCD's
// L2.  A drained queue sends its workgroups to the next queues.  Each queue
// head is its own 128-byte line; a claim takes `count` consecutive items.
// Returns [first, end) of the claim, or (n, n) when every queue is drained.
__device__ __forceinline__ uint2 claim_items(uint32_t* queues, uint32_t n, uint32_t count)
{
    const uint32_t home = blockIdx.x % kQueues;
    for (uint32_t t = 0; t < kQueues; ++t) {
        const uint32_t k = (home + t) % kQueues;
        const uint32_t lo = (uint32_t)((uint64_t)n * k / kQueues), hi = (uint32_t)((uint64_t)n * (k + 1) / kQueues);
        if (lo >= hi) continue;
        const uint32_t v = atomicAdd(queues + k * kQueueStride, count);
        if (v < hi - lo) return make_uint2(lo + v, lo + v + count < hi ? lo + v + count : hi);
    }
    return make_uint2(n, n);
}

// items of a persistent wavefront, claimed kClaim at a time
constexpr uint32_t kClaim = 4;

struct WaveQueue {
    uint32_t cur = 0, end = 0;
};

__device__ __forceinline__ uint32_t next_item_wave(WaveQueue& q, uint32_t* queues, uint32_t n, uint32_t lane)
{
    if (q.cur >= q.end) {
        uint2 r = make_uint2(0u, 0u);
        if (lane == 0) r = claim_items(queues, n, kClaim);
        q.cur = __shfl(r.x, 0, 64);
        q.end = __shfl(r.y, 0, 64);
        if (q.cur >= q.end) return n;
    }
    return q.cur++;
}


// Per-lane state of the front-to-back walk of one pixel.
struct FwdPix {
    float T, Cr, Cg, Cb, H2;         // transmittance, colour, entropy in log2 units
    int32_t last;                    // n_contrib
    int32_t stop_pos;                // list position of the stopping entry; -1 while the
                                     // pixel is open (0 from the start outside the image)
};

// Wavefront-uniform state of a block's walk (scalar registers): the mask of its
// open pixels (lane l's bit set while stop_pos of lane l is -1), and the alpha
// tests made (a surviving entry visited by a pixel still open) and the entries
// blended, summed over the wavefront.
struct FwdWave {
    uint64_t open;
    uint32_t tested, blended;
};

__device__ __forceinline__ void fwd_init(FwdPix& q, FwdWave& wc, bool inside)
{
    q.T = 1.f; q.Cr = q.Cg = q.Cb = q.H2 = 0.f;
    q.last = 0; q.stop_pos = inside ? -1 : 0;
    wc.open = __builtin_amdgcn_ballot_w64(inside);
    wc.tested = wc.blended = 0u;
}

__device__ __forceinline__ bool fwd_open(const FwdPix& q) { return q.stop_pos < 0; }

// Alpha of one list entry at this lane's pixel (Eq. 3): g0 = (mean, A', B'),
// g1 = (C', opacity, ...).  A pure function of the record and the pixel, so the
// alphas of consecutive entries can be evaluated together.
__device__ __forceinline__ float fwd_alpha(float4 g0, float4 g1, float fpx, float fpy)
{
    const float p = gauss_p2(g0.z, g0.w, g1.x, g0.x - fpx, g0.y - fpy);
    return fminf(kAlphaMax, g1.y * __builtin_amdgcn_exp2f(p));
}

// One surviving list entry for one pixel, given its alpha: the transmittance stop,
// colour (Eq. 5) and the entropy term -w log2 w (Eq. 10).  pos1: the entry's list
// position + 1.  Whether a lane is open, and the counts, are lane masks and their
// sums (scalar work); the ray stops once per pixel, so its bookkeeping sits in a
// branch the wavefront almost always skips.
template <bool RENDER>
__device__ __forceinline__ void fwd_apply(FwdPix& q, FwdWave& wc, float alpha, float cr, float cg, float cb,
                                          int32_t pos1)
{
    const float Tn = q.T * (1.f - alpha);
    // lane masks: open pixels the entry reaches; of those, the ones it would take below
    // T = 1e-4 (they stop) and the rest (they blend)
    const uint64_t hit = wc.open & __builtin_amdgcn_ballot_w64(alpha >= kAlphaMin);
    const uint64_t low = __builtin_amdgcn_ballot_w64(Tn < kTStop);
    const uint64_t stop = hit & low, blend = hit & ~low;
    wc.tested += (uint32_t)__popcll(wc.open);
    wc.blended += (uint32_t)__popcll(blend);
    wc.open &= ~stop;
    if (__builtin_expect(__builtin_amdgcn_inverse_ballot_w64(stop), 0)) q.stop_pos = pos1 - 1;
    if (__builtin_amdgcn_inverse_ballot_w64(blend)) {
        const float w = alpha * q.T;
        q.Cr = fmaf(w, cr, q.Cr);
        q.Cg = fmaf(w, cg, q.Cg);
        q.Cb = fmaf(w, cb, q.Cb);
        if (!RENDER) q.H2 = fmaf(-w, __builtin_amdgcn_logf(w), q.H2);    // -w log2 w   (Eq. 10)
        q.T = Tn;
        q.last = pos1;
    }
}

template <bool RENDER>
__device__ __forceinline__ void fwd_step(FwdPix& q, FwdWave& wc, float4 g0, float4 g1, float b, float fpx, float fpy,
                                         int32_t pos1)
{
    fwd_apply<RENDER>(q, wc, fwd_alpha(g0, g1, fpx, fpy), g1.z, g1.w, b, pos1);
}

// Outputs of one pixel and the work counts of its 8x8 block.
template <bool RENDER>
__device__ __forceinline__ void fwd_store(const BlendFwdArgs& a, const BlockGeom& g, const FwdPix& q,
                                          const FwdWave& wc, uint2 rg, uint32_t wb, uint32_t lane)
{
    // background weight T_{N+1} (Eq. 9-10), then natural-log units
    const float H = RENDER ? 0.f : kLn2 * fmaf(-q.T, __builtin_amdgcn_logf(q.T), q.H2);
    if (g.inside) {
        a.out_rgb[3 * g.pix + 0] = q.Cr;
        a.out_rgb[3 * g.pix + 1] = q.Cg;
        a.out_rgb[3 * g.pix + 2] = q.Cb;
        if (!RENDER) {
            a.out_H[g.pix] = H;
            a.out_T[g.pix] = q.T;
            a.out_nc[g.pix] = q.last;
        }
    }
    // list positions this pixel visited (the stopping entry included), culled ones counted
    const int32_t n_eval = !g.inside ? 0 : (!fwd_open(q) ? q.stop_pos + 1 : (int32_t)(rg.y - rg.x));
    const uint32_t ne = (uint32_t)wave_sum_all_i(n_eval);
    const uint32_t nc = (uint32_t)wave_sum_all_i(q.last);
    const uint32_t nb = wc.blended;
    // alpha tests at list positions that survived the block cull that this kernel
    // made (until the ray stopped); the backward adds its own count (up to the last
    // contributor) in the next word
    const uint32_t tf = wc.tested;
    const float hs = RENDER ? 0.f : wave_sum_all(g.inside ? H : 0.f);
    if (lane == 0) {
        if (!RENDER) a.block_H[wb] = hs;
        a.block_cnt[2 * wb] = make_uint4(ne, nc, nb, 0u);
        a.block_cnt[2 * wb + 1] = make_uint4(tf, 0u, 0u, 0u);
    }
}

// One wavefront per 8x8 block with its own batches: a wavefront whose pixels
// have all stopped leaves at once, which pays on short lists; on long ones the
// four blocks of a tile restage the same entries (blend_fwd_shared_kernel
// below stages them once).  RENDER: colour only (test-time rendering): no
// entropy, no per-pixel saved state.
template <int B>
struct FwdLds {
    float4 g0[kWavesPerGroup][B];                // mean x, mean y, A', B'
    float4 g1[kWavesPerGroup][B];                // C', opacity, red, green
    float2 bp[kWavesPerGroup][B];                // blue, position in the tile list + 1 (int bits)
};

// workgroup wg of the launch; `from`: the first place of the tile order it serves
template <int B, bool PERSIST, bool RENDER>
__device__ __forceinline__ void fwd_blocks(const BlendFwdArgs& a, uint32_t wg, uint32_t from, FwdLds<B>& lds)
{
    auto& s_g0 = lds.g0;
    auto& s_g1 = lds.g1;
    auto& s_bp = lds.bp;
    const uint32_t lane = threadIdx.x & 63u, wid = threadIdx.x >> 6;
    WaveQueue wq;
    uint32_t item;
    if (PERSIST) {
        item = next_item_wave(wq, a.queues, a.n_blocks, lane);
    } else if (a.tile_order) {                   // hardware dispatch, longest tiles first
        if (a.spt == 4) {
            item = a.tile_order[from + wg] * kWavesPerGroup + wid;  // one tile per workgroup
        } else {
            const uint32_t i = from + wg * kWavesPerGroup + wid;     // one tile per wavefront
            item = i < a.n_blocks ? a.tile_order[i] : a.n_blocks;
        }
    } else {
        item = wg * kWavesPerGroup + wid;
    }
    for (; item < a.n_blocks; item = PERSIST ? next_item_wave(wq, a.queues, a.n_blocks, lane) : a.n_blocks) {
    const uint32_t wb = item;
    const BlockGeom g = block_geom(a.cams, a.n_views, wb, lane, a.tile_shift_x, a.tile_shift_y, a.spt);
    const uint2 rg = a.ranges[g.tile];
    const float fpx = (float)g.px + 0.5f, fpy = (float)g.py + 0.5f;
    const uint64_t lt_mask = (1ull << lane) - 1ull;
    FwdPix q;
    FwdWave wc;
    fwd_init(q, wc, g.inside);
    // a batch's records are loaded into registers one batch ahead (in flight while the
    // previous batch blends), their record indices (two dependent loads) two batches
    // ahead, 64 entries a register
    constexpr int NH = (B + kWave - 1) / kWave;
    uint32_t pv[NH];
    float4 c0[NH], c1[NH], c2[NH];
#pragma unroll
    for (int h = 0; h < NH; ++h) {
        const uint32_t jh = (uint32_t)h * kWave + lane;
        const uint32_t e = rg.x + jh;
        pv[h] = jh < (uint32_t)B && e < rg.y ? a.emit_vg[a.pair_vals[e]] : 0u;
        c0[h] = c1[h] = c2[h] = make_float4(0.f, 0.f, 0.f, 0.f);
        if (jh < (uint32_t)B && e < rg.y) {
            const float4* r = a.rec + (size_t)kRecF4 * pv[h];
            c0[h] = r[0];
            c1[h] = r[1];
            c2[h] = r[2];
        }
        const uint32_t e2 = rg.x + B + jh;
        if (jh < (uint32_t)B && e2 < rg.y) pv[h] = a.emit_vg[a.pair_vals[e2]];
    }
    for (uint32_t bs = rg.x; bs < rg.y; bs += B) {
        if (wc.open == 0ull) break;
        const uint32_t cnt = (rg.y - bs) < (uint32_t)B ? (rg.y - bs) : (uint32_t)B;
        // stage the batch, keeping (in list order) only Gaussians that can reach this block
        uint32_t m = 0;
#pragma unroll
        for (int h = 0; h < NH; ++h) {
            const uint32_t j0 = (uint32_t)h * kWave;
            if (j0 >= cnt) continue;                           // (uniform; no break, so the registers stay)
            const uint32_t j = j0 + lane;
            const bool keep = j < cnt && !culled(g, c0[h], c1[h].x, c2[h]);
            const uint64_t bal = __ballot(keep);
            if (keep) {
                const uint32_t k = m + (uint32_t)__popcll(bal & lt_mask);
                s_g0[wid][k] = c0[h];
                s_g1[wid][k] = c1[h];
                s_bp[wid][k] = make_float2(c2[h].x, __int_as_float((int32_t)(bs + j - rg.x) + 1));
            }
            m += (uint32_t)__popcll(bal);
        }
        // the next batch's records, the record indices of the one after
#pragma unroll
        for (int h = 0; h < NH; ++h) {
            const uint32_t jh = (uint32_t)h * kWave + lane;
            if (jh < (uint32_t)B && bs + B + jh < rg.y) {
                const float4* r = a.rec + (size_t)kRecF4 * pv[h];
                c0[h] = r[0];
                c1[h] = r[1];
                c2[h] = r[2];
            }
            if (jh < (uint32_t)B && bs + 2 * B + jh < rg.y) pv[h] = a.emit_vg[a.pair_vals[bs + 2 * B + jh]];
        }
        wave_lds_sync();
        m = (uint32_t)__builtin_amdgcn_readfirstlane((int)m);   // wavefront-uniform: a scalar loop
        // two entries a step: both alphas evaluated before either is applied
        for (uint32_t k = 0; k < m; k += 2) {
            const uint32_t k1 = k + 1 < m ? k + 1 : k;           // an entry that can be read
            const float4 a1 = s_g1[wid][k], b1 = s_g1[wid][k1];
            const float aa = fwd_alpha(s_g0[wid][k], a1, fpx, fpy);
            const float ab = fwd_alpha(s_g0[wid][k1], b1, fpx, fpy);
            const float2 pa = s_bp[wid][k];
            fwd_apply<RENDER>(q, wc, aa, a1.z, a1.w, pa.x, __float_as_int(pa.y));
            if (k + 1 < m) {
                const float2 pb = s_bp[wid][k1];
                fwd_apply<RENDER>(q, wc, ab, b1.z, b1.w, pb.x, __float_as_int(pb.y));
            }
        }
        wave_lds_sync();
    }
    fwd_store<RENDER>(a, g, q, wc, rg, wb, lane);
    }
}

template <int B, bool PERSIST, bool RENDER>
__global__ __launch_bounds__(256) void blend_fwd_kernel(BlendFwdArgs a)
{
    __shared__ FwdLds<B> s_lds;
    fwd_blocks<B, PERSIST, RENDER>(a, blockIdx.x, 0u, s_lds);
}

// The 4 wavefronts of a workgroup are the 4 8x8 blocks of one 16x16 or 32x8
// tile: each batch of the tile's list is staged once for all four (one entry per
// thread), then every wavefront keeps the entries that can reach its block (the
// exact cull, into its own index list) and blends them.  The batch loop ends when
// no pixel of the tile is still open.
template <int B, bool PERSIST, bool RENDER>
__global__ __launch_bounds__(256) void blend_fwd_shared_kernel(BlendFwdArgs a)
{
    static_assert(B <= 256, "one staged entry per thread");
    // a batch entry j: s_rec[0][j] = (mean x, mean y, A', B'), s_rec[1][j] = (C', opacity,
    // red, green), s_rec[2][j] = (blue, L, -B'/(2C'), -B'/(2A')), s_rec[3][j].x = list
    // position + 1 (int bits); one array per part, so that the lanes of the cull, one
    // entry each, read 16-byte strides (no bank conflicts), and the blend loop reads all
    // four parts of entry j at one offset, 16 j
    __shared__ float4 s_rec[kFwdRecF4][B];
    // each wavefront's surviving batch entries (byte offsets), in list order, and after
    // the last of them a valid offset; read two at a time, so a row holds one pair more
    // than a batch needs
    __shared__ int2 s_idx2[kWavesPerGroup][B / 2 + 1];
    __shared__ uint32_t s_item;
    const uint32_t lane = threadIdx.x & 63u, wid = threadIdx.x >> 6, tid = threadIdx.x;
    const uint32_t n_items = a.n_blocks / kWavesPerGroup;      // tiles
    auto next = [&]() -> uint32_t {
        if (!PERSIST) return n_items;
        __syncthreads();
        if (tid == 0) s_item = claim_items(a.queues, n_items, 1u).x;
        __syncthreads();
        return s_item;
    };
    uint32_t item;
    if (PERSIST) item = next();
    else item = a.tile_order ? a.tile_order[blockIdx.x] : blockIdx.x;   // longest tiles first
    for (; item < n_items; item = next()) {
    const uint32_t wb = item * kWavesPerGroup + wid;
    const BlockGeom g = block_geom(a.cams, a.n_views, wb, lane, a.tile_shift_x, a.tile_shift_y, a.spt);
    const uint2 rg = a.ranges[g.tile];
    const float fpx = (float)g.px + 0.5f, fpy = (float)g.py + 0.5f;
    const uint64_t lt_mask = (1ull << lane) - 1ull;
    FwdPix q;
    FwdWave wc;
    fwd_init(q, wc, g.inside);
    // each thread stages one entry of a batch: its record is loaded into registers one
    // batch ahead (in flight while the previous batch blends), its record index (two
    // dependent loads) two batches ahead
    uint32_t pv = 0;
    float4 n0 = make_float4(0.f, 0.f, 0.f, 0.f), n1 = n0, n2 = n0;
    if (tid < (uint32_t)B && rg.x + tid < rg.y) {
        pv = a.emit_vg[a.pair_vals[rg.x + tid]];
        const float4* r = a.rec + (size_t)kRecF4 * pv;
        n0 = r[0];
        n1 = r[1];
        n2 = r[2];
    }
    if (tid < (uint32_t)B && rg.x + B + tid < rg.y) pv = a.emit_vg[a.pair_vals[rg.x + B + tid]];
    for (uint32_t bs = rg.x; bs < rg.y; bs += B) {
        // (also orders this batch's staging after every wavefront's reads of the last one)
        if (!__syncthreads_or(wc.open != 0ull ? 1 : 0)) break;  // every pixel of the tile has stopped
        const uint32_t cnt = (rg.y - bs) < (uint32_t)B ? (rg.y - bs) : (uint32_t)B;
        if (tid < cnt) {
            s_rec[0][tid] = n0;
            s_rec[1][tid] = n1;
            s_rec[2][tid] = n2;
            s_rec[3][tid] = make_float4(__int_as_float((int32_t)(bs - rg.x + tid) + 1), 0.f, 0.f, 0.f);
        }
        __syncthreads();
        if (tid < (uint32_t)B && bs + B + tid < rg.y) {
            const float4* r = a.rec + (size_t)kRecF4 * pv;
            n0 = r[0];
            n1 = r[1];
            n2 = r[2];
        }
        if (tid < (uint32_t)B && bs + 2 * B + tid < rg.y) pv = a.emit_vg[a.pair_vals[bs + 2 * B + tid]];
        uint32_t m = 0;
        if (wc.open != 0ull) {                                   // this block still has open pixels
            for (uint32_t j0 = 0; j0 < cnt; j0 += kWave) {
                const uint32_t j = j0 + lane;
                const bool keep = j < cnt && !culled(g, s_rec[0][j], s_rec[1][j].x, s_rec[2][j]);
                const uint64_t bal = __ballot(keep);
                if (keep) {
                    const uint32_t k = m + (uint32_t)__popcll(bal & lt_mask);
                    reinterpret_cast<int32_t*>(&s_idx2[wid][0])[k] = (int32_t)(sizeof(float4) * j);
                }
                m += (uint32_t)__popcll(bal);
            }
        }
        // the slot after the last survivor holds a valid offset (entry 0), so that a step's
        // second entry can always be read
        if (lane == 0) reinterpret_cast<int32_t*>(&s_idx2[wid][0])[m] = 0;
        wave_lds_sync();
        m = (uint32_t)__builtin_amdgcn_readfirstlane((int)m);   // wavefront-uniform: a scalar loop
        // two entries a step: their offsets read together, both alphas evaluated before
        // either is applied (independent chains), then applied in list order
        for (uint32_t k = 0; k < m; k += 2) {
            const int2 off = s_idx2[wid][k / 2];                 // k + 1 <= B: inside the row
            const float4* ra = reinterpret_cast<const float4*>(reinterpret_cast<const char*>(&s_rec[0][0]) + off.x);
            const float4* rb = reinterpret_cast<const float4*>(reinterpret_cast<const char*>(&s_rec[0][0]) + off.y);
            const float4 a1 = ra[B], b1 = rb[B];
            const float aa = fwd_alpha(ra[0], a1, fpx, fpy);
            const float ab = fwd_alpha(rb[0], b1, fpx, fpy);
            fwd_apply<RENDER>(q, wc, aa, a1.z, a1.w, ra[2 * B].x, __float_as_int(ra[3 * B].x));
            if (k + 1 < m) fwd_apply<RENDER>(q, wc, ab, b1.z, b1.w, rb[2 * B].x, __float_as_int(rb[3 * B].x));
        }
    }
    fwd_store<RENDER>(a, g, q, wc, rg, wb, lane);
    }
}

// ---------------------------------------------------------------------------
// The slotted forms, forward and backward: four list entries a step.
//
// A launch of few tiles ends with its longest list's walk, one entry after another, on
// a chip that is mostly idle by then.  Here a wavefront owns a 4x4 pixel block and the
// four lanes of a quad take four consecutive surviving entries of one pixel: everything
// that does not depend on the entries before runs four entries wide, and the walk's serial
// part (the transmittance, backward also Q) is four multiply steps over the quad by DPP,
// in list order, with the arithmetic of the plain forms: alphas, transmittances, stops
// and n_contrib are bit-identical to theirs, and so are colour and entropy (a quad's lanes
// accumulate one channel each, the fourth the entropy, in list order).  The 16 wavefronts of a 16x16 / 32x8 tile
// (4 of an 8x8 tile) share the staged records.  A step of 4 entries at 16 pixels costs 1.3
// times the instructions of one entry at 64 pixels and its latency is about that of
// one; the finer cull gives most of the throughput back.  Bound by the latency of the
// longest list's steps (LDS reads, exp, the quad's chain), forward / backward at 16x16
// tiles, plain -> slotted: 2k Gaussians at 128x128, 27 -> 13 / 52 -> 25 us; 200k at 256x160,
// 718 -> 170 / 955 -> 425 us; 200k at 640x416, 207 -> 79 / 347 -> 167 us; 150k at 801x533 in
// 8x8 tiles, 118 -> 55 / 187 -> 79 us.
// ---------------------------------------------------------------------------
constexpr int kSlotBatch = 256;          // entries a forward batch

// value of quad lane I in every lane of the quad
template <int I>
__device__ __forceinline__ float quad_f(float v)
{
    return dpp_f<0x55 * I, 0xf>(v);
}

template <int I>
__device__ __forceinline__ int32_t quad_i(int32_t v)
{
    return __builtin_amdgcn_update_dpp(0, v, 0x55 * I, 0xf, 0xf, true);
}

// v[slot], slot = this lane's place in its quad
__device__ __forceinline__ float by_slot(uint32_t slot, float v0, float v1, float v2, float v3)
{
    const float lo = slot & 1u ? v1 : v0, hi = slot & 1u ? v3 : v2;
    return slot & 2u ? hi : lo;
}

// Geometry of a wavefront's 4x4 block: quarter wid % 4 of 8x8 block wb.  g8: the 8x8 block
// (its rectangle); g: the 4x4 block's rectangle and this lane's pixel.
__device__ __forceinline__ void slot_geom(const CamDev* cams, int n_views, uint32_t wb, uint32_t wid, uint32_t lane,
                                          int tsx, int tsy, int spt, BlockGeom& g8, BlockGeom& g)
{
    const uint32_t q = wid & 3u, p = lane >> 2;
    g8 = block_geom(cams, n_views, wb, 0u, tsx, tsy, spt);
    const CamDev& c = cams[g8.view];
    g = g8;
    const int x0 = g8.px + 4 * (int)(q & 1u), y0 = g8.py + 4 * (int)(q >> 1);
    g.px = x0 + (int)(p & 3u);
    g.py = y0 + (int)(p >> 2);
    g.inside = g.px < c.W && g.py < c.H;
    g.pix = c.pix_base + (int64_t)g.py * c.W + g.px;
    g.cx0 = (float)x0 + 0.5f;
    g.cy0 = (float)y0 + 0.5f;
    g.cx1 = (float)min(x0 + 3, c.W - 1) + 0.5f;
    g.cy1 = (float)min(y0 + 3, c.H - 1) + 0.5f;
}

// the entries of a slotted walk whose colours are not finite: taken by the lanes that
// blend them only (a zero weight times infinity must not reach the others)
__device__ __forceinline__ bool odd_colour(float r, float g, float b)
{
    return !(fabsf(r) + fabsf(g) + fabsf(b) < __builtin_inff());
}

// Forward: a workgroup of 4 wavefronts an 8x8 block, also where a tile has 4 of them (each
// stages the tile's list for itself: the blocks of a tile need not wait for each other, and
// five workgroups a CU hide more than one of 16 wavefronts did: 200k Gaussians at 640x416,
// 79 against 104 us)
template <int B>
struct FwdSlotLds {
    float4 rec[2][3 * (B + 1)];                              // a part's last record is empty (opacity 0)
    // each wavefront's surviving entries (byte offsets in a part), in list order, and up to 8
    // empty ones (read a step ahead)
    int32_t idx[4][B + 8];
    uint64_t keep[4];                                        // the 8x8 block's survivors, entries 64 w ..
    uint32_t open[4];
    uint32_t cnt[4][4];
    float h[64];                                             // entropy of the 8x8 block's pixels
};

template <int B, bool RENDER>
__device__ __forceinline__ void fwd_slots(const BlendFwdArgs& a, uint32_t wg, FwdSlotLds<B>& lds)
{
    constexpr int NW = 4;
    constexpr int kPart = B + 1;
    constexpr int kEmptyOff = 16 * B;
    auto& s_rec = lds.rec;
    auto& s_idx = lds.idx;
    auto& s_keep = lds.keep;
    auto& s_open = lds.open;
    auto& s_cnt = lds.cnt;
    auto& s_h = lds.h;
    const uint32_t tid = threadIdx.x, lane = tid & 63u, wid = tid >> 6, slot = lane & 3u;
    const uint32_t item = wg / (uint32_t)a.spt;              // longest tiles first
    const uint32_t wb = (a.tile_order ? a.tile_order[item] : item) * (uint32_t)a.spt + wg % (uint32_t)a.spt;
    BlockGeom g8, g;
    slot_geom(a.cams, a.n_views, wb, wid, lane, a.tile_shift_x, a.tile_shift_y, a.spt, g8, g);
    const uint2 rg = a.ranges[g8.tile];
    const float fpx = (float)g.px + 0.5f, fpy = (float)g.py + 0.5f;
    const uint64_t lt_mask = (1ull << lane) - 1ull;
    if (tid < 6u) s_rec[tid / 3u][(tid % 3u) * kPart + B] = make_float4(0.f, 0.f, 0.f, 0.f);
    // byte offset, from an entry's first part, of the colour channel this lane accumulates
    const int32_t ch_off = slot == 0u ? 16 * kPart + 8 : (slot == 1u ? 16 * kPart + 12 : 32 * kPart);
    float T = 1.f, C = 0.f;                                  // C: channel `slot`, of slot 3 the entropy (log2 units)
    int32_t last = 0, stop_pos = g.inside ? -1 : 0;
    uint64_t open = __builtin_amdgcn_ballot_w64(g.inside);
    uint32_t tested = 0u, blended = 0u;
    // records one batch ahead in registers, record indices two
    uint32_t pv = 0;
    float4 n0 = make_float4(0.f, 0.f, 0.f, 0.f), n1 = n0, n2 = n0;
    if (tid < (uint32_t)B && rg.x + tid < rg.y) {
        pv = a.emit_vg[a.pair_vals[rg.x + tid]];
        const float4* r = a.rec + (size_t)kRecF4 * pv;
        n0 = r[0];
        n1 = r[1];
        n2 = r[2];
    }
    if (tid < (uint32_t)B && rg.x + B + tid < rg.y) pv = a.emit_vg[a.pair_vals[rg.x + B + tid]];
    uint32_t buf = 0u;
    for (uint32_t bs = rg.x; bs < rg.y; bs += B, buf ^= 1u) {
        const uint32_t cnt = (rg.y - bs) < (uint32_t)B ? (rg.y - bs) : (uint32_t)B;
        float4* rec = s_rec[buf];
        if (tid < cnt) {
            rec[tid] = n0;
            rec[kPart + tid] = n1;
            rec[2 * kPart + tid] = n2;
        }
        __syncthreads();
        if (tid < (uint32_t)B && bs + B + tid < rg.y) {
            const float4* r = a.rec + (size_t)kRecF4 * pv;
            n0 = r[0];
            n1 = r[1];
            n2 = r[2];
        }
        if (tid < (uint32_t)B && bs + 2 * B + tid < rg.y) pv = a.emit_vg[a.pair_vals[bs + 2 * B + tid]];
        // a quarter of the batch against this wavefront's 8x8 block
        {
            const uint32_t j = tid;
            const bool keep = j < cnt && !culled(g8, rec[j], rec[kPart + j].x, rec[2 * kPart + j]);
            const uint64_t bal = __builtin_amdgcn_ballot_w64(keep);
            if (lane == 0u) {
                s_keep[wid] = bal;
                s_open[wid] = open != 0ull ? 1u : 0u;
            }
        }
        __syncthreads();
        if ((s_open[0] | s_open[1] | s_open[2] | s_open[3]) == 0u) break;          // every pixel has stopped
        if (open == 0ull) continue;
        // the batch's entries that can reach the 4x4 block
        uint32_t m = 0, m8 = 0;
        bool odd = false;
#pragma unroll
        for (uint32_t h = 0; h < (uint32_t)B / 64u; ++h) {
            const uint64_t k8 = s_keep[h];
            const uint32_t j = 64u * h + lane;
            bool keep = (k8 >> lane) & 1ull;
            if (keep) {
                const float4 r1 = rec[kPart + j], r2 = rec[2 * kPart + j];
                keep = !culled(g, rec[j], r1.x, r2);
                odd |= keep && odd_colour(r1.z, r1.w, r2.x);
            }
            const uint64_t bal = __builtin_amdgcn_ballot_w64(keep);
            if (keep) s_idx[wid][m + (uint32_t)__popcll(bal & lt_mask)] = (int32_t)(16u * j);
            m += (uint32_t)__popcll(bal);
            m8 += (uint32_t)__popcll(k8);
        }
        if (lane < 8u) s_idx[wid][m + lane] = kEmptyOff;
        wave_lds_sync();
        m = (uint32_t)__builtin_amdgcn_readfirstlane((int)m);
        const bool any_odd = __builtin_amdgcn_ballot_w64(odd) != 0ull;
        const char* base = reinterpret_cast<const char*>(rec);
        const int32_t pos0 = (int32_t)(bs - rg.x) + 1;
        // a step's operands, loaded a step ahead
        int32_t off = s_idx[wid][slot];
        float4 e0 = *reinterpret_cast<const float4*>(base + off);
        float2 e1 = *reinterpret_cast<const float2*>(base + off + 16 * kPart);
        float c0 = *reinterpret_cast<const float*>(base + quad_i<0>(off) + ch_off);
        float c1 = *reinterpret_cast<const float*>(base + quad_i<1>(off) + ch_off);
        float c2 = *reinterpret_cast<const float*>(base + quad_i<2>(off) + ch_off);
        float c3 = *reinterpret_cast<const float*>(base + quad_i<3>(off) + ch_off);
        for (uint32_t k = 0; k < m; k += 4u) {
            const int32_t noff = s_idx[wid][k + 4u + slot];
            const float p = gauss_p2(e0.z, e0.w, e1.x, e0.x - fpx, e0.y - fpy);
            const float alpha = fminf(kAlphaMax, e1.y * __builtin_amdgcn_exp2f(p));
            const uint64_t hit = open & __builtin_amdgcn_ballot_w64(alpha >= kAlphaMin);
            float al = __builtin_amdgcn_inverse_ballot_w64(hit) ? alpha : 0.f;
            const float4 f0 = *reinterpret_cast<const float4*>(base + noff);
            const float2 f1 = *reinterpret_cast<const float2*>(base + noff + 16 * kPart);
            const float d0 = *reinterpret_cast<const float*>(base + quad_i<0>(noff) + ch_off);
            const float d1 = *reinterpret_cast<const float*>(base + quad_i<1>(noff) + ch_off);
            const float d2 = *reinterpret_cast<const float*>(base + quad_i<2>(noff) + ch_off);
            const float d3 = *reinterpret_cast<const float*>(base + quad_i<3>(noff) + ch_off);
            // the transmittance before and after each of the four entries, in list order
            float om = 1.f - al;
            float t1 = T * quad_f<0>(om), t2 = t1 * quad_f<1>(om), t3 = t2 * quad_f<2>(om), t4 = t3 * quad_f<3>(om);
            uint64_t blend = hit;
            const int32_t pos1 = pos0 + (off >> 4);
            if (__builtin_expect(__builtin_amdgcn_ballot_w64(t4 < kTStop) != 0ull, 0)) {
                // some pixel stops at one of them: the first hit that would take T below the
                // threshold, and nothing after it, blends
                const uint64_t low = __builtin_amdgcn_ballot_w64(by_slot(slot, t1, t2, t3, t4) < kTStop);
                blend = hit & ~low;
                uint64_t stop = hit & low;                   // the stopping entry and hits after it
                al = __builtin_amdgcn_inverse_ballot_w64(blend) ? alpha : 0.f;
                om = 1.f - al;
                t1 = T * quad_f<0>(om);
                t2 = t1 * quad_f<1>(om);
                t3 = t2 * quad_f<2>(om);
                t4 = t3 * quad_f<3>(om);
                const uint32_t mine = (uint32_t)(stop >> (lane & ~3u)) & 0xfu;   // this quad's
                if (mine != 0u) {
                    const int first = __ffs((int)mine) - 1;
                    const int32_t so = first == 0 ? quad_i<0>(off) : first == 1 ? quad_i<1>(off)
                                       : first == 2 ? quad_i<2>(off) : quad_i<3>(off);
                    const int32_t j = so >> 4;
                    stop_pos = pos0 + j - 1;
                    // the 8x8 block's survivors up to and including the stopping entry
                    uint32_t t = 0u;
#pragma unroll
                    for (int h = 0; h < B / 64; ++h) {
                        const uint64_t k8 = s_keep[h];
                        const int32_t r = j - 64 * h;
                        if (r >= 0) t += (uint32_t)__popcll(r >= 63 ? k8 : k8 & ((2ull << r) - 1ull));
                    }
                    if (slot == 0u) tested += t;
                }
                open &= ~__builtin_amdgcn_ballot_w64(mine != 0u);
            }
            const float w = al * by_slot(slot, T, t1, t2, t3);
            if (!RENDER) {                                   // -w log2 w (Eq. 10): slot 3's "channel"
                const float lw = -__builtin_amdgcn_logf(fmaxf(w, 1e-30f));
                // (moved before the choice: a lane move reads only lanes that execute it)
                const float l0 = quad_f<0>(lw), l1 = quad_f<1>(lw), l2 = quad_f<2>(lw), l3 = quad_f<3>(lw);
                c0 = slot == 3u ? l0 : c0;
                c1 = slot == 3u ? l1 : c1;
                c2 = slot == 3u ? l2 : c2;
                c3 = slot == 3u ? l3 : c3;
            }
            const float w0 = quad_f<0>(w), w1 = quad_f<1>(w), w2 = quad_f<2>(w), w3 = quad_f<3>(w);
            if (__builtin_expect(any_odd, 0)) {              // (a zero weight takes no part)
                if (w0 != 0.f) C = fmaf(w0, c0, C);
                if (w1 != 0.f) C = fmaf(w1, c1, C);
                if (w2 != 0.f) C = fmaf(w2, c2, C);
                if (w3 != 0.f) C = fmaf(w3, c3, C);
            } else {
                C = fmaf(w0, c0, C);
                C = fmaf(w1, c1, C);
                C = fmaf(w2, c2, C);
                C = fmaf(w3, c3, C);
            }
            if (__builtin_amdgcn_inverse_ballot_w64(blend)) last = pos1;
            blended += (uint32_t)__popcll(blend);
            T = t4;
            off = noff;
            e0 = f0;
            e1 = f1;
            c0 = d0; c1 = d1; c2 = d2; c3 = d3;
        }
        // pixels still open tested every survivor of the 8x8 block
        if (slot == 0u && __builtin_amdgcn_inverse_ballot_w64(open)) tested += m8;
        wave_lds_sync();
    }
    // the quad's entropy and last position
    const float H = RENDER ? 0.f : kLn2 * fmaf(-T, __builtin_amdgcn_logf(T), quad_f<3>(C));
    last = max(last, __builtin_amdgcn_update_dpp(0, last, 0xb1, 0xf, 0xf, true));
    last = max(last, __builtin_amdgcn_update_dpp(0, last, 0x4e, 0xf, 0xf, true));
    if (g.inside) {
        if (slot < 3u) a.out_rgb[3 * g.pix + slot] = C;
        else if (!RENDER) {
            a.out_H[g.pix] = H;
            a.out_T[g.pix] = T;
            a.out_nc[g.pix] = last;
        }
    }
    // the 8x8 block's work counts, and its entropy, summed as the plain forms sum it
    const bool count = slot == 0u && g.inside;
    const int32_t n_eval = !count ? 0 : (stop_pos >= 0 ? stop_pos + 1 : (int32_t)(rg.y - rg.x));
    const uint32_t ne = (uint32_t)wave_sum_all_i(n_eval), nc = (uint32_t)wave_sum_all_i(count ? last : 0);
    const uint32_t tf = (uint32_t)wave_sum_all_i((int32_t)tested);
    if (!RENDER && slot == 0u)
        s_h[8 * (g.py & 7) + (g.px & 7)] = g.inside ? H : 0.f;
    if (lane == 0u) {
        s_cnt[wid][0] = ne;
        s_cnt[wid][1] = nc;
        s_cnt[wid][2] = blended;
        s_cnt[wid][3] = tf;
    }
    __syncthreads();
    if (wid == 0u) {
        const float h = RENDER ? 0.f : wave_sum_all(s_h[lane]);
        if (lane == 0u) {
            uint32_t s[4] = { 0u, 0u, 0u, 0u };
#pragma unroll
            for (int w = 0; w < NW; ++w)
#pragma unroll
                for (int k = 0; k < 4; ++k) s[k] += s_cnt[w][k];
            if (!RENDER) a.block_H[wb] = h;
            a.block_cnt[2 * wb] = make_uint4(s[0], s[1], s[2], 0u);
            a.block_cnt[2 * wb + 1] = make_uint4(s[3], 0u, 0u, 0u);
        }
    }
}

template <bool RENDER>
__global__ __launch_bounds__(256) void blend_fwd_slot_kernel(BlendFwdArgs a)
{
    __shared__ FwdSlotLds<kSlotBatch> s_lds;
    fwd_slots<kSlotBatch, RENDER>(a, blockIdx.x, s_lds);
}

// A mid-sized launch of short lists ends with the walks of its longest tiles too: of 200k
// Gaussians at 1296x840 VALU instructions were active for 0.79 of the plain form's busy cycles, of
// 1M with longer lists for 1.00.  The first workgroups take the 128 longest tiles in the slotted
// form, the others the rest of the tile order in the plain one, in the same launch; the outputs
// are those of either form.  90 -> 78 us, active for 0.91; its registers are the slotted form's (five
// wavefronts a SIMD instead of seven), which larger launches would feel (mixed_blend).
constexpr int kMixedBatch = 128;
template <int B, bool RENDER>
__global__ __launch_bounds__(256) void blend_fwd_mixed_kernel(BlendFwdArgs a)
{
    __shared__ union {
        FwdSlotLds<kMixedBatch> slot;
        FwdLds<B> plain;
    } s_lds;
    const uint32_t n_slot = kMixedTiles * (uint32_t)a.spt;
    if (blockIdx.x < n_slot) fwd_slots<kMixedBatch, RENDER>(a, blockIdx.x, s_lds.slot);
    else fwd_blocks<B, false, RENDER>(a, blockIdx.x - n_slot, kMixedTiles, s_lds.plain);
}

// Per-lane state of the backward walk of one pixel.  The per-pixel sums the
// backward needs, S_{i+1} = sum_{k>i} w_k c_k (colour, Eq. 13-14) and Alg. 1's
// R_{i+1} = sum_{k>i} (ln w_k + 1) w_k + (ln T + 1) T (entropy, Eq. 15), only
// ever enter dL/dalpha_i through Q_{i+1} = gh R_{i+1} - dL/dC . S_{i+1}, so one
// running scalar carries both:
//   dL/dalpha_i = T_i D_i + Q_{i+1} / (1 - alpha_i),
//   D_i = dL/dC . c_i - gh (ln w_i + 1),   Q_i = Q_{i+1} - w_i D_i,
// with gh = dL/dH of the pixel and Q_{N+1} = gh (ln T_final + 1) T_final.
struct BwdPix {
    int32_t n;                       // list positions to walk (n_contrib)
    float T;                         // T_{i+1} while walking back; starts at T_final
    float gCr, gCg, gCb;             // dL/dC of this pixel
    float gh, ghl;                   // dL/dH of this pixel, and gh ln 2 (weights' logs are in log2 units)
    float Q;                         // Q_{i+1}
    float fpx, fpy;
};

// Backward of one list entry for one pixel.  Branch-free per lane: every lane
// evaluates the entry and a lane whose pixel did not blend it (position past its
// last contributor, or alpha < 1/255) contributes zero and keeps its state.
// bwd_alpha evaluates alpha; bwd_grad, run only if some lane of the wavefront
// blended the entry, updates the walk state and returns the 9 per-pixel terms
// whose sums over pixels give the entry's gradient:
//   o[0] = e2 dg          (-> opacity; e2 = 2^p, dg = dL/dalpha in the unclamped branch)
//   o[1] = o[0] dx,  o[2] = o[0] dy                     (-> mean, with the conic)
//   o[3] = o[1] dx,  o[4] = o[1] dy,  o[5] = o[2] dy     (-> conic A, B, C)
//   o[6..8] = w dL/dC                                   (-> colour)
// The per-Gaussian factors (opacity, conic, ln 2) are applied once per
// (tile, Gaussian) after the sum, by finish_row.
struct BwdAlpha {
    float dx, dy, e2, a_raw, alpha;
    bool act;
};

// j: the entry's index in the window, nrel = n - (the window's first list position),
// both scaled by the same positive factor (the record's byte size)
__device__ __forceinline__ BwdAlpha bwd_alpha(const BwdPix& q, int32_t j, int32_t nrel, float4 g0, float4 g1)
{
    BwdAlpha r;
    r.dx = g0.x - q.fpx;
    r.dy = g0.y - q.fpy;
    r.e2 = __builtin_amdgcn_exp2f(gauss_p2(g0.z, g0.w, g1.x, r.dx, r.dy));
    r.a_raw = g1.y * r.e2;
    r.alpha = fminf(kAlphaMax, r.a_raw);
    r.act = (j < nrel) & (r.alpha >= kAlphaMin);
    return r;
}

__device__ __forceinline__ void bwd_grad(BwdPix& q, const BwdAlpha& r, float4 g1, float cb, float* o)
{
    const bool act = r.act;
    const float rom = __builtin_amdgcn_rcpf(1.f - r.alpha);
    const float Ti = q.T * rom;                              // T_i = T_{i+1} / (1 - alpha_i)
    const float w = r.alpha * Ti;
    const float lw2 = __builtin_amdgcn_logf(act ? w : 1.f);  // log2 w_i
    const float D = fmaf(-q.ghl, lw2, fmaf(q.gCr, g1.z, fmaf(q.gCg, g1.w, fmaf(q.gCb, cb, -q.gh))));
    const float dal = rom * fmaf(q.T, D, q.Q);              // (T_{i+1} D_i + Q_{i+1}) / (1 - alpha_i)
    const float wa = act ? w : 0.f;
    const float dg = (act & (r.a_raw <= kAlphaMax)) ? dal : 0.f;   // zero in the clamped branch
    o[0] = r.e2 * dg;
    o[1] = o[0] * r.dx;
    o[2] = o[0] * r.dy;
    o[3] = o[1] * r.dx;
    o[4] = o[1] * r.dy;
    o[5] = o[2] * r.dy;
    o[6] = wa * q.gCr;
    o[7] = wa * q.gCg;
    o[8] = wa * q.gCb;
    q.Q = fmaf(-wa, D, q.Q);                                 // Q_i = Q_{i+1} - w_i D_i
    q.T = act ? Ti : q.T;
}

// Gradient row of one (tile, Gaussian) pair from the summed terms S[0..8] of
// bwd_grad, with g0 = (mean, A', B'), g1 = (C', opacity, ...):  alpha = opacity 2^p and
// p = A' dx^2 + B' dx dy + C' dy^2 (log2 units), so dalpha/dp = alpha ln 2 and
// dalpha/d(natural-log exponent) = alpha.
__device__ __forceinline__ void finish_row(const float* S, float4 g0, float4 g1, float* G)
{
    const float sig = g1.y;
    const float sl = kLn2 * sig;
    G[0] = sl * fmaf(2.f * g0.z, S[1], g0.w * S[2]);         // mean x
    G[1] = sl * fmaf(2.f * g1.x, S[2], g0.w * S[1]);         // mean y
    G[2] = -0.5f * sig * S[3];                               // conic A, B, C (unscaled)
    G[3] = -sig * S[4];
    G[4] = -0.5f * sig * S[5];
    G[5] = S[0];                                             // opacity
    G[6] = S[6];                                             // colour
    G[7] = S[7];
    G[8] = S[8];
}

__device__ __forceinline__ void bwd_init(const BlendBwdArgs& a, const BlockGeom& g, int32_t len, BwdPix& q)
{
    q.n = 0; q.T = 1.f; q.gCr = q.gCg = q.gCb = q.gh = 0.f;
    if (g.inside) {
        int32_t n = a.n_contrib[g.pix];
        q.n = n < 0 ? 0 : (n > len ? len : n);               // never walk past this tile's list
        q.T = a.T_final[g.pix];
        q.gCr = a.grad_rgb[3 * g.pix + 0];
        q.gCg = a.grad_rgb[3 * g.pix + 1];
        q.gCb = a.grad_rgb[3 * g.pix + 2];
        if (a.grad_H) q.gh = a.grad_H[g.pix];
        if (a.grad_LE) {
            const CamDev& c = a.cams[g.view];
            q.gh += a.grad_LE[g.view] / (float)((int64_t)c.W * c.H);
        }
    }
    q.ghl = q.gh * kLn2;
    q.Q = q.gh * ((logf(q.T) + 1.f) * q.T);                 // gh R_{N+1}, Alg. 1's initialisation
    q.fpx = (float)g.px + 0.5f;
    q.fpy = (float)g.py + 0.5f;
}

// SHARED: the 4 wavefronts of the workgroup are the 4 blocks of one tile and
// share each window; otherwise every wavefront has its own tile and window.
//
// Window records in LDS.  SHARED: two buffers (the next window is loaded while this
// one is walked), each as three arrays of one 16-byte part of every entry (part k of
// entry j at s_rec[buffer][k B + j]), filled straight from global memory by direct
// loads to LDS (global_load_lds_dwordx4: lane l's 16 bytes land at the wavefront's
// LDS base + 16 l), so no register holds a record in flight.  Otherwise: per
// wavefront slot, whole 48-byte entries (entry j at s_rec[slot][3 j]) staged through
// registers.
// 16 bytes per lane from global memory straight into LDS: lane l's land at lds + 16 l
// (lds is the wavefront's base; a device function, so that only the device pass sees
// the builtin)
__device__ __forceinline__ void lds_direct_load16(const float4* src, float4* lds)
{
    __builtin_amdgcn_global_load_lds(src, lds, 16, 0, 0);
}

template <int B, bool SHARED>
struct BwdRecLayout {
    static constexpr int kBytes = SHARED ? (int)sizeof(float4) : (int)sizeof(float4) * kRecF4;  // per entry
    static constexpr int kPart = SHARED ? B : 1;               // float4s between an entry's parts
    __device__ static int idx(int j, int k) { return SHARED ? k * B + j : kRecF4 * j + k; }
};

template <int B, bool SHARED, bool PERSIST>
__global__ __launch_bounds__(256, (SHARED && B <= 64 && !PERSIST) ? 8 : 1) void blend_bwd_kernel(BlendBwdArgs a)
{
    using RL = BwdRecLayout<B, SHARED>;
    constexpr int NS = SHARED ? 1 : kWavesPerGroup;          // LDS slots
    // window entries' records (see above) and emission indices (SHARED: s_rec / s_e hold
    // one buffer, s_rec2 / s_e2 the other; two arrays, so that the compiler sees that
    // the direct loads into one never alias the reads of the other and makes those reads
    // wait for nothing), and, per wavefront, each entry's accumulator row (the 9
    // wavefront sums, then 1 where the wavefront blended it)
    __shared__ float4 s_rec[NS][B * kRecF4];
    __shared__ uint32_t s_e[NS][B];
    __shared__ float4 s_rec2[SHARED ? B * kRecF4 : 1];
    __shared__ uint32_t s_e2[SHARED ? B : 1];
    __shared__ float s_acc[kWavesPerGroup][B * kAccF];   // per-wavefront sums of each window entry
    // surviving window entries of each wavefront, as the offsets of their record
    // (float4 index) and of their accumulator row (float index)
    // surviving entries' record offsets and accumulator offsets, entry k at [.][k + 1]
    // (the same row shape, so that one address serves both; the first slot is never used)
    __shared__ int32_t s_idx[kWavesPerGroup][B + 1];
    __shared__ int32_t s_aidx[kWavesPerGroup][B + 1];
    __shared__ int32_t s_max[kWavesPerGroup];
    __shared__ uint32_t s_item;
    const uint32_t lane = threadIdx.x & 63u, wid = threadIdx.x >> 6;
    const uint32_t stamp = *a.stamp;
    const int tcomp = tot_comp(lane);
    // work items: tiles (SHARED: one per workgroup; else one per wavefront), claimed from the per-XCD queues
    const uint32_t n_items = SHARED ? a.n_blocks / kWavesPerGroup : a.n_blocks;
    WaveQueue wq;
    auto next = [&]() -> uint32_t {
        if (!PERSIST) return n_items;
        if (SHARED) {
            __syncthreads();
            if (threadIdx.x == 0) s_item = claim_items(a.queues, n_items, 1u).x;
            __syncthreads();
            return s_item;
        }
        return next_item_wave(wq, a.queues, n_items, lane);
    };
    uint32_t item;
    if (PERSIST) item = next();
    else if (a.tile_order) {                     // hardware dispatch, longest tiles first
        const uint32_t i = SHARED ? blockIdx.x : blockIdx.x * kWavesPerGroup + wid;
        item = i < n_items ? a.tile_order[i] : n_items;
    } else item = SHARED ? blockIdx.x : blockIdx.x * kWavesPerGroup + wid;
    for (; item < n_items; item = next()) {
    const uint32_t tile_id = item;
    const uint32_t wb = SHARED ? tile_id * kWavesPerGroup + wid : tile_id;
    const BlockGeom g = block_geom(a.cams, a.n_views, wb, lane, a.tile_shift_x, a.tile_shift_y, a.spt);
    const uint2 rg = a.ranges[g.tile];
    const int32_t len = (int32_t)(rg.y - rg.x);
    BwdPix q;
    bwd_init(a, g, len, q);
    // wavefront-uniform loop bounds live in scalar registers
    const int32_t wave_n = __builtin_amdgcn_readfirstlane(wave_max_i32(q.n));
    int32_t maxn = wave_n;
    if (SHARED) {
        if (lane == 0) s_max[wid] = wave_n;
        __syncthreads();
        maxn = __builtin_amdgcn_readfirstlane(max(max(s_max[0], s_max[1]), max(s_max[2], s_max[3])));
    }
    const int32_t nthr = SHARED ? 256 : 64;
    const int32_t tid = SHARED ? (int32_t)threadIdx.x : (int32_t)lane;
    // only the hit flags start at zero: a slot's sums are read only where its flag is set
    for (int32_t i = (int32_t)lane; i < B; i += kWave) s_acc[wid][kAccF * i + kG2] = 0.f;
    uint32_t tested = 0;                     // alpha tests (list positions before a pixel's n_contrib)

    // window x covers list positions [lo(x), lo(x) + cnt(x)), from the back
    const int32_t nwin = (maxn + B - 1) / B;
    auto win_lo = [&](int32_t x) { const int32_t l = maxn - (x + 1) * B; return l > 0 ? l : 0; };
    auto win_cnt = [&](int32_t x) { const int32_t c = maxn - x * B; return c < B ? c : B; };
    // per-block: each thread stages entries tid, tid + 64, ... of its wavefront's window
    // through registers; their emission and record indices (two dependent loads) are
    // fetched one window ahead
    constexpr int NW = SHARED ? 1 : (B + kWave - 1) / kWave;
    uint32_t pe[NW], pv[NW];
#pragma unroll
    for (int h = 0; h < NW; ++h) pe[h] = pv[h] = 0u;
    auto fetch_indices = [&](int32_t x) {
        const int32_t lo_x = win_lo(x), cnt_x = win_cnt(x);
#pragma unroll
        for (int h = 0; h < NW; ++h) {
            const int32_t j = tid + h * nthr;
            if (j < cnt_x) {
                pe[h] = a.pair_vals[rg.x + (uint32_t)(lo_x + j)];
                pv[h] = a.emit_vg[pe[h]];
            }
        }
    };
    // SHARED: thread tid < cnt(x) holds entry tid of window x.  A window's records are
    // loaded into the other buffer while the one before it is walked, by direct loads
    // (one instruction per 16-byte part for the wavefront's 64 entries); its record
    // indices one window earlier, its emission indices one earlier again, so that every
    // load waits only at the barrier that ends a window (the wait count of vector memory
    // is in order: a dependent load issued after the direct loads would wait for them).
    // e1, v1: emission and record index of the next window; e2: emission index of the
    // one after.
    uint32_t e1 = 0u, v1 = 0u, e2 = 0u;
    auto load_window = [&](float4* rec_b, uint32_t* e_b, int32_t x) {
        if (tid < win_cnt(x)) {
            const float4* r = a.rec + (size_t)kRecF4 * v1;
            const int w0 = tid & ~(kWave - 1);               // the wavefront's first entry
#pragma unroll
            for (int k = 0; k < kRecF4; ++k) lds_direct_load16(r + k, &rec_b[RL::idx(w0, k)]);
            e_b[tid] = e1;
        }
    };
    // one window: its records and emission indices in rec_w / e_w; SHARED: the next
    // window's go to rec_n / e_n
    auto window = [&](float4* rec_w, uint32_t* e_w, float4* rec_n, uint32_t* e_n, int32_t w) {
        const int32_t lo = win_lo(w);
        const int32_t cnt = win_cnt(w);
        if (SHARED) {
            // (the barrier that ended the last window also ended every read of rec_n)
            if (w + 1 < nwin) load_window(rec_n, e_n, w + 1);
            if (w + 2 < nwin && tid < win_cnt(w + 2)) {
                v1 = a.emit_vg[e2];
                e1 = e2;
            }
            if (w + 3 < nwin && tid < win_cnt(w + 3)) e2 = a.pair_vals[rg.x + (uint32_t)(win_lo(w + 3) + tid)];
        } else {
#pragma unroll
            for (int h = 0; h < NW; ++h) {
                const int32_t j = tid + h * nthr;
                if (j < cnt) {
                    const float4* r = a.rec + (size_t)kRecF4 * pv[h];
                    e_w[j] = pe[h];
                    rec_w[kRecF4 * j + 0] = r[0];
                    rec_w[kRecF4 * j + 1] = r[1];
                    rec_w[kRecF4 * j + 2] = r[2];
                }
            }
            wave_lds_sync();
            if (w + 1 < nwin) fetch_indices(w + 1);
        }
        // this wavefront's surviving entries of the window, in list order
        const int32_t jtop = (wave_n - lo) < cnt ? (wave_n - lo) : cnt;
        int32_t m = 0;
        for (int32_t j0 = 0; j0 < jtop; j0 += kWave) {
            const int32_t j = j0 + (int32_t)lane;
            bool keep = false;
            if (j < jtop)
                keep = !culled(g, rec_w[RL::idx(j, 0)], rec_w[RL::idx(j, 1)].x, rec_w[RL::idx(j, 2)]);
            const uint64_t bal = __ballot(keep);
            if (keep) {
                const int32_t k = m + (int32_t)__popcll(bal & ((1ull << lane) - 1ull));
                s_idx[wid][k + 1] = RL::kBytes * j;
                s_aidx[wid][k + 1] = kAccF * j;
            }
            m += (int32_t)__popcll(bal);
        }
        wave_lds_sync();
        // window entries j < nrel lie in this pixel's list (compared as the byte offset
        // of the entry's record in s_rec)
        const int32_t nrel = RL::kBytes * (q.n - lo);
        // walk them back to front, two entries a step (their offsets read together); per
        // Gaussian, the wavefront sums go to this wavefront's slot
        auto entry = [&](int32_t kk, int32_t j3) {
            const float4* r = reinterpret_cast<const float4*>(reinterpret_cast<const char*>(rec_w) + j3);
            const float4 g1 = r[RL::kPart];
            const BwdAlpha al = bwd_alpha(q, j3, nrel, r[0], g1);
            tested += (uint32_t)__popcll(__builtin_amdgcn_ballot_w64(j3 < nrel));
            if (__builtin_amdgcn_ballot_w64(al.act) != 0ull) {   // else no lane of this wavefront blended it
                float o[kG2];
                bwd_grad(q, al, g1, r[2 * RL::kPart].x, o);
                const float tot = wave_sum9<SHARED>(o, lane);
                if (tcomp >= 0) {
                    float* acc = &s_acc[wid][s_aidx[wid][kk + 1]];
                    acc[tcomp] = tot;
                    acc[kG2] = 1.f;                          // (every total's lane writes the same flag)
                }
            }
        };
        int32_t kk = m - 1;
        for (; kk >= 1; kk -= 2) {
            const int32_t oa = s_idx[wid][kk + 1], ob = s_idx[wid][kk];   // entries kk, kk - 1
            entry(kk, oa);
            entry(kk - 1, ob);
        }
        if (kk == 0) entry(0, s_idx[wid][1]);
        if (SHARED) __syncthreads(); else wave_lds_sync();
        // store the rows of the window's blended entries (emission slots),
        // summing the flagged wavefront slots in a fixed order and clearing their flags
        // (a slot without its flag holds stale sums and adds nothing); entries no pixel
        // blended keep no row (their stamp is not this frame's)
        for (int32_t j = tid; j < cnt; j += nthr) {
            constexpr int32_t nsl = SHARED ? kWavesPerGroup : 1;
            const int32_t s0 = SHARED ? 0 : (int32_t)wid;
            bool f[nsl];
            bool hit = false;
#pragma unroll
            for (int32_t r = 0; r < nsl; ++r) {
                f[r] = s_acc[s0 + r][kAccF * j + kG2] != 0.f;
                hit |= f[r];
            }
            if (!hit) continue;
            float S[kG2], G[kG2];
#pragma unroll
            for (int k = 0; k < kG2; ++k) S[k] = 0.f;
#pragma unroll
            for (int32_t r = 0; r < nsl; ++r) {
                if (!f[r]) continue;
                const float* src = &s_acc[s0 + r][kAccF * j];
#pragma unroll
                for (int k = 0; k < kG2; ++k) S[k] += src[k];
                s_acc[s0 + r][kAccF * j + kG2] = 0.f;
            }
            finish_row(S, rec_w[RL::idx(j, 0)], rec_w[RL::idx(j, 1)], G);
            float* row = a.pair_grad + (size_t)kRowF * e_w[j];
#pragma unroll
            for (int k = 0; k < kG2; ++k) row[k] = G[k];
            a.pair_stamp[e_w[j]] = stamp;
        }
        if (SHARED) {
            __builtin_amdgcn_s_waitcnt(0);                   // the next window's direct loads have landed
            __syncthreads();
        } else {
            wave_lds_sync();
        }
    };
    if (SHARED) {
        if (nwin > 0) {
            if (tid < win_cnt(0)) {
                e1 = a.pair_vals[rg.x + (uint32_t)(win_lo(0) + tid)];
                v1 = a.emit_vg[e1];
            }
            load_window(s_rec[0], s_e[0], 0);
        }
        if (nwin > 1 && tid < win_cnt(1)) {
            e1 = a.pair_vals[rg.x + (uint32_t)(win_lo(1) + tid)];
            v1 = a.emit_vg[e1];
        }
        if (nwin > 2 && tid < win_cnt(2)) e2 = a.pair_vals[rg.x + (uint32_t)(win_lo(2) + tid)];
        __builtin_amdgcn_s_waitcnt(0);                       // this thread's direct loads have landed
        __syncthreads();
        // two windows an iteration, so that each buffer is one named array in each
        for (int32_t w = 0; w < nwin; w += 2) {
            window(s_rec[0], s_e[0], s_rec2, s_e2, w);
            if (w + 1 < nwin) window(s_rec2, s_e2, s_rec[0], s_e[0], w + 1);
        }
    } else {
        if (nwin > 0) fetch_indices(0);
        for (int32_t w = 0; w < nwin; ++w) window(s_rec[wid], s_e[wid], nullptr, nullptr, w);
    }
    if (lane == 0) reinterpret_cast<uint32_t*>(a.block_cnt + 2 * wb + 1)[1] = tested;
    }
}

// The slotted backward: windows of 64 entries from the back, the slots of a quad in walk
// order.  T and Q pass from slot to slot by DPP (T with the plain form's arithmetic); the 9
// terms of the four entries are summed over the 16 pixels together, by lane swaps and row
// rotations, into one row of LDS an entry and wavefront.
// DENSE: held to 64 VGPRs (19 of them spill, 80 bytes of scratch a lane), so that two
// workgroups of 16 wavefronts share a CU.
template <int SPT, bool DENSE>
__global__ __launch_bounds__(256 * SPT, DENSE ? 8 : 1) void blend_bwd_slot_kernel(BlendBwdArgs a)
{
    constexpr int B = 64, NW = 4 * SPT;
    constexpr int kPart = B + 1;                             // records a part: the last is empty (opacity 0)
    constexpr int kEmptyOff = 16 * B;
    __shared__ float4 s_rec[3 * kPart];                      // two buffers, as two arrays (see blend_bwd_kernel)
    __shared__ float4 s_rec2[3 * kPart];
    __shared__ uint32_t s_e[B], s_e2[B];
    __shared__ float s_acc[NW][(B + 4) * kG2];               // each wavefront's sums of its surviving entries
    __shared__ int32_t s_idx[NW][B + 8];                     // their byte offsets, last first, and empty ones
    __shared__ uint64_t s_keep[NW], s_hit[NW];               // surviving entries; of those, the blended ones
    __shared__ uint64_t s_keep8[SPT];                        // the 8x8 blocks' survivors (work counts)
    __shared__ int32_t s_max[NW];
    __shared__ uint32_t s_tested[NW];
    const uint32_t tid = threadIdx.x, lane = tid & 63u, wid = tid >> 6, slot = lane & 3u;
    const uint32_t stamp = *a.stamp;
    const uint32_t tile = a.tile_order ? a.tile_order[blockIdx.x] : blockIdx.x;
    BlockGeom g8, g;
    slot_geom(a.cams, a.n_views, tile * SPT + (SPT == 4 ? wid >> 2 : 0u), wid, lane, a.tile_shift_x, a.tile_shift_y, SPT,
              g8, g);
    const uint2 rg = a.ranges[tile];
    BwdPix q;
    bwd_init(a, g, (int32_t)(rg.y - rg.x), q);
    const int32_t wave_n = __builtin_amdgcn_readfirstlane(wave_max_i32(q.n));
    if (lane == 0u) s_max[wid] = wave_n;
    if (tid < 3u) s_rec[tid * kPart + B] = s_rec2[tid * kPart + B] = make_float4(0.f, 0.f, 0.f, 0.f);
    __syncthreads();
    const int32_t maxn = __builtin_amdgcn_readfirstlane(wave_max_i32(s_max[lane % NW]));
    uint32_t tested = 0u;

    const int32_t nwin = (maxn + B - 1) / B;
    auto win_lo = [&](int32_t x) { const int32_t l = maxn - (x + 1) * B; return l > 0 ? l : 0; };
    auto win_cnt = [&](int32_t x) { const int32_t c = maxn - x * B; return c < B ? c : B; };
    // the first wavefront fetches the windows, as in blend_bwd_kernel
    uint32_t e1 = 0u, v1 = 0u, e2 = 0u;
    const int32_t t = (int32_t)tid;
    auto load_window = [&](float4* rec_b, uint32_t* e_b, int32_t x) {
        if (t < win_cnt(x)) {
            const float4* r = a.rec + (size_t)kRecF4 * v1;
#pragma unroll
            for (int k = 0; k < kRecF4; ++k) lds_direct_load16(r + k, &rec_b[k * kPart]);
            e_b[t] = e1;
        }
    };
    auto window = [&](float4* rec_w, uint32_t* e_w, float4* rec_n, uint32_t* e_n, int32_t w) {
        const int32_t lo = win_lo(w), cnt = win_cnt(w);
        if (w + 1 < nwin) load_window(rec_n, e_n, w + 1);
        if (w + 2 < nwin && t < win_cnt(w + 2)) {
            v1 = a.emit_vg[e2];
            e1 = e2;
        }
        if (w + 3 < nwin && t < win_cnt(w + 3)) e2 = a.pair_vals[rg.x + (uint32_t)(win_lo(w + 3) + t)];
        // this wavefront's surviving entries, last first; each 8x8 block's by one of its wavefronts in turn
        const int32_t jtop = (wave_n - lo) < cnt ? (wave_n - lo) : cnt;
        const float4 r0 = rec_w[lane], r2 = rec_w[2 * kPart + lane];
        const float rc = rec_w[kPart + lane].x;
        const bool kept = (int32_t)lane < jtop && !culled(g, r0, rc, r2);
        const uint64_t keep = __builtin_amdgcn_ballot_w64(kept);
        const int32_t m = (int32_t)__popcll(keep);
        if (kept) s_idx[wid][__popcll((keep >> lane) >> 1)] = 16 * (int32_t)lane;
        if (lane < 8u) s_idx[wid][m + (int32_t)lane] = kEmptyOff;
        if ((wid & 3u) == ((uint32_t)w & 3u)) {
            const uint64_t k8 = __builtin_amdgcn_ballot_w64((int32_t)lane < cnt && !culled(g8, r0, rc, r2));
            if (lane == 0u) s_keep8[wid >> 2] = k8;
        }
        wave_lds_sync();
        const int32_t nrel = 16 * (q.n - lo);                // entries below it lie in this pixel's list
        uint64_t hits = 0ull;
        if (m > 0) {
            const char* base = reinterpret_cast<const char*>(rec_w);
            int32_t off = s_idx[wid][slot];
            float4 g0 = *reinterpret_cast<const float4*>(base + off);
            float4 g1 = *reinterpret_cast<const float4*>(base + off + 16 * kPart);
            float cb = *reinterpret_cast<const float*>(base + off + 32 * kPart);
            for (int32_t k = 0; k < m; k += 4) {
                const int32_t noff = s_idx[wid][k + 4 + (int32_t)slot];
                const BwdAlpha al = bwd_alpha(q, off, nrel, g0, g1);
                const uint64_t act = __builtin_amdgcn_ballot_w64(al.act);
                const float4 h0 = *reinterpret_cast<const float4*>(base + noff);
                const float4 h1 = *reinterpret_cast<const float4*>(base + noff + 16 * kPart);
                const float hb = *reinterpret_cast<const float*>(base + noff + 32 * kPart);
                if (act != 0ull) {
                    const float alpha = al.act ? al.alpha : 0.f;
                    const float rom = __builtin_amdgcn_rcpf(1.f - alpha);
                    // T_{i+1} and T_i = T_{i+1} / (1 - alpha_i) of every slot, in walk order
                    const float t1 = q.T * quad_f<0>(rom), t2 = t1 * quad_f<1>(rom);
                    const float t3 = t2 * quad_f<2>(rom), t4 = t3 * quad_f<3>(rom);
                    const float wt = alpha * by_slot(slot, t1, t2, t3, t4);
                    const float lw2 = __builtin_amdgcn_logf(al.act ? wt : 1.f);
                    const float D = fmaf(-q.ghl, lw2, fmaf(q.gCr, g1.z, fmaf(q.gCg, g1.w, fmaf(q.gCb, cb, -q.gh))));
                    // (an entry that this pixel did not blend may have a colour past the largest float)
                    const float wd = al.act ? wt * D : 0.f;
                    const float q1 = q.Q - quad_f<0>(wd), q2 = q1 - quad_f<1>(wd);
                    const float q3 = q2 - quad_f<2>(wd), q4 = q3 - quad_f<3>(wd);
                    const float dal = rom * fmaf(by_slot(slot, q.T, t1, t2, t3), D, by_slot(slot, q.Q, q1, q2, q3));
                    const float dg = (al.act & (al.a_raw <= kAlphaMax)) ? dal : 0.f;
                    q.T = t4;
                    q.Q = q4;
                    float o[kG2];
                    o[0] = al.e2 * dg;
                    o[1] = o[0] * al.dx;
                    o[2] = o[0] * al.dy;
                    o[3] = o[1] * al.dx;
                    o[4] = o[1] * al.dy;
                    o[5] = o[2] * al.dy;
                    o[6] = wt * q.gCr;
                    o[7] = wt * q.gCg;
                    o[8] = wt * q.gCb;
                    // sums over the 16 pixels, a slot a lane: halves and rows fold in pairs (row r ends
                    // with o[row_comp(r)] in x0, o[4 + row_comp(r)] in x1, o[8] in x2), then lanes 4
                    // and 8 apart
                    const float u0 = fold_halves(o[0], o[1]), u1 = fold_halves(o[2], o[3]);
                    const float u2 = fold_halves(o[4], o[5]), u3 = fold_halves(o[6], o[7]);
                    const float u4 = fold_halves(o[8], o[8]);
                    float x0 = fold_rows(u0, u1), x1 = fold_rows(u2, u3), x2 = fold_rows(u4, u4);
                    x0 += dpp_f<0x128, 0xf>(x0);
                    x1 += dpp_f<0x128, 0xf>(x1);
                    x2 += dpp_f<0x128, 0xf>(x2);
                    x0 += dpp_f<0x124, 0xf>(x0);
                    x1 += dpp_f<0x124, 0xf>(x1);
                    x2 += dpp_f<0x124, 0xf>(x2);
                    if ((lane & 15u) < 4u) {
                        float* dst = &s_acc[wid][(k + (int32_t)slot) * kG2];
                        dst[row_comp(lane >> 4)] = x0;
                        dst[4 + row_comp(lane >> 4)] = x1;
                        if (lane < 4u) dst[8] = x2;
                    }
                    uint64_t b = act | (act >> 32);          // the slots some pixel blended
                    b |= b >> 16;
                    b |= b >> 8;
                    b |= b >> 4;
                    hits |= (b & 0xfull) << k;
                }
                off = noff;
                g0 = h0;
                g1 = h1;
                cb = hb;
            }
        }
        if (lane == 0u) {
            s_keep[wid] = keep;
            s_hit[wid] = hits;
        }
        __syncthreads();
        if (slot == 0u) {
            const int32_t nw = q.n - lo;
            const uint64_t k8 = s_keep8[wid >> 2];
            tested += nw <= 0 ? 0u : (uint32_t)__popcll(nw >= B ? k8 : k8 & ((1ull << nw) - 1ull));
        }
        // the rows of the window's blended entries: NW lanes an entry, lane r for wavefront
        // r's sums, added in a fixed order (the tree of the lanes)
        {
            const int32_t j = (int32_t)(tid / (uint32_t)NW);
            const uint32_t r = tid % (uint32_t)NW;
            const uint64_t kr = s_keep[r] >> j;
            float S[kG2 + 1];
#pragma unroll
            for (int k = 0; k <= kG2; ++k) S[k] = 0.f;
            if (kr & 1ull) {
                const int32_t c = (int32_t)__popcll(kr >> 1);
                if ((s_hit[r] >> c) & 1ull) {
                    const float* src = &s_acc[r][c * kG2];
#pragma unroll
                    for (int k = 0; k < kG2; ++k) S[k] = src[k];
                    S[kG2] = 1.f;
                }
            }
#pragma unroll
            for (int k = 0; k <= kG2; ++k) {
                S[k] += dpp_f<0xb1, 0xf>(S[k]);              // quad_perm [1,0,3,2]
                S[k] += dpp_f<0x4e, 0xf>(S[k]);              // quad_perm [2,3,0,1]
                if (NW == 16) {
                    S[k] += dpp_f<0x141, 0xf>(S[k]);         // row_half_mirror
                    S[k] += dpp_f<0x140, 0xf>(S[k]);         // row_mirror
                }
            }
            if (S[kG2] != 0.f) {
                float G[kG2];
                finish_row(S, rec_w[j], rec_w[kPart + j], G);
                const uint32_t e = e_w[j];
                float* row = a.pair_grad + (size_t)kRowF * e;
                if (r < 4u) {
                    const float2 part = r == 0u ? make_float2(G[0], G[1]) : r == 1u ? make_float2(G[2], G[3])
                                        : r == 2u ? make_float2(G[4], G[5]) : make_float2(G[6], G[7]);
                    reinterpret_cast<float2*>(row)[r] = part;
                    if (r == 0u) row[8] = G[8];
                    if (r == 1u) a.pair_stamp[e] = stamp;
                }
            }
        }
        __builtin_amdgcn_s_waitcnt(0);                       // the next window's direct loads have landed
        __syncthreads();
    };
    if (nwin > 0) {
        if (t < win_cnt(0)) {
            e1 = a.pair_vals[rg.x + (uint32_t)(win_lo(0) + t)];
            v1 = a.emit_vg[e1];
        }
        load_window(s_rec, s_e, 0);
    }
    if (nwin > 1 && t < win_cnt(1)) {
        e1 = a.pair_vals[rg.x + (uint32_t)(win_lo(1) + t)];
        v1 = a.emit_vg[e1];
    }
    if (nwin > 2 && t < win_cnt(2)) e2 = a.pair_vals[rg.x + (uint32_t)(win_lo(2) + t)];
    __builtin_amdgcn_s_waitcnt(0);                           // this thread's direct loads have landed
    __syncthreads();
    for (int32_t w = 0; w < nwin; w += 2) {
        window(s_rec, s_e, s_rec2, s_e2, w);
        if (w + 1 < nwin) window(s_rec2, s_e2, s_rec, s_e, w + 1);
    }
    const uint32_t nt = (uint32_t)wave_sum_all_i((int)tested);
    if (lane == 0u) s_tested[wid] = nt;
    __syncthreads();
    if (tid < (uint32_t)SPT)
        reinterpret_cast<uint32_t*>(a.block_cnt + 2 * (tile * SPT + tid) + 1)[1] =
            s_tested[4u * tid] + s_tested[4u * tid + 1u] + s_tested[4u * tid + 2u] + s_tested[4u * tid + 3u];
}

// Debug check of Eq. 9 (GSR_DEBUG_INVARIANTS): the weights of the blended Gaussians and
// the background weight T_final sum to one.  An independent per-pixel walk: one thread
// per pixel re-evaluates its tile's list from the front, with the forward's alpha
// arithmetic, sums the weights of the entries it blends up to the forward's n_contrib,
// and compares sum w + T_final (the forward's) with 1.  Each blended step rounds w and T
// within 2u T_i and the running sum within u per add, so |sum w + T - 1| <= 3u n_contrib;
// the check counts pixels beyond 4u (n_contrib + 1).  Debug speed: uncoalesced walks.
__global__ __launch_bounds__(256) void invariant_kernel(InvArgs a)
{
    const int64_t p = (int64_t)blockIdx.x * 256 + threadIdx.x;   // packed pixel index
    float err = 0.f;
    bool bad = false;
    if (p < a.n_pix) {
        int v = 0;
        while (v + 1 < a.n_views && a.cams[v + 1].pix_base <= p) ++v;
        const CamDev& c = a.cams[v];
        const int64_t q = p - c.pix_base;
        const int px = (int)(q % c.W), py = (int)(q / c.W);
        const uint32_t tile = c.tile_base + (uint32_t)((py >> a.tile_shift_y) * c.gx + (px >> a.tile_shift_x));
        const uint2 rg = a.ranges[tile];
        int32_t n = a.n_contrib[p];
        n = n < 0 ? 0 : (n > (int32_t)(rg.y - rg.x) ? (int32_t)(rg.y - rg.x) : n);
        const float fpx = (float)px + 0.5f, fpy = (float)py + 0.5f;
        float T = 1.f, S = 0.f;
        for (int32_t i = 0; i < n; ++i) {
            const float4* r = a.rec + (size_t)kRecF4 * a.emit_vg[a.pair_vals[rg.x + (uint32_t)i]];
            const float4 g0 = r[0], g1 = r[1];
            const float alpha =
                fminf(kAlphaMax, g1.y * __builtin_amdgcn_exp2f(gauss_p2(g0.z, g0.w, g1.x, g0.x - fpx, g0.y - fpy)));
            if (alpha < kAlphaMin) continue;
            S = fmaf(alpha, T, S);
            T *= 1.f - alpha;
        }
        err = fabsf(S + a.T_final[p] - 1.f);
        bad = !(err <= 4.f * 5.9604645e-8f * (float)(n + 1));     // NaN counts as a violation
        if (!(err == err)) err = __uint_as_float(0x7f800000u);      // reported as +inf
    }
    const uint32_t nbad = (uint32_t)__popcll(__ballot(bad));
    float m = err;
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) m = fmaxf(m, __shfl_xor(m, o, 64));
    if ((threadIdx.x & 63u) == 0u) {
        if (nbad) atomicAdd(&a.counters[7], nbad);
        atomicMax(&a.counters[6], __float_as_uint(m));           // non-negative floats order as their bits
    }
}

__device__ __forceinline__ double block_sum_f64(double x)
{
    __shared__ double s[256];
    s[threadIdx.x] = x;
    __syncthreads();
    for (int o = 128; o > 0; o >>= 1) {
        if ((int)threadIdx.x < o) s[threadIdx.x] += s[threadIdx.x + o];
        __syncthreads();
    }
    return s[0];
}

// level 1: one workgroup per chunk of kRedChunk wave blocks of one view
__global__ __launch_bounds__(256) void entropy_chunk_kernel(const float* block_H, const CamDev* cams, int n_views,
                                                            double* chunk_sum)
{
    const uint32_t ch = blockIdx.x;
    int v = 0;
    while (v + 1 < n_views && cams[v + 1].hred_base <= ch) ++v;
    const CamDev& c = cams[v];
    const uint32_t nb = c.n_wblocks;
    const uint32_t b0 = (ch - c.hred_base) * kRedChunk;
    // all loads first (clamped index), then the sum in the same order as a plain loop
    constexpr int kPer = kRedChunk / 256;
    static_assert(kRedChunk % 256 == 0, "whole rounds of 256");
    float hv[kPer];
#pragma unroll
    for (int j = 0; j < kPer; ++j) {
        const uint32_t b = b0 + threadIdx.x + 256u * (uint32_t)j;
        hv[j] = block_H[c.block_base + (b < nb ? b : nb - 1u)];
    }
    double acc = 0.0;
#pragma unroll
    for (int j = 0; j < kPer; ++j)
        if (b0 + threadIdx.x + 256u * (uint32_t)j < nb) acc += (double)hv[j];
    const double tot = block_sum_f64(acc);
    if (threadIdx.x == 0) chunk_sum[ch] = tot;
}

// level 2: one workgroup per view, L_E = sum of its chunks / (W H)   (Eq. 11)
__global__ __launch_bounds__(256) void entropy_mean_kernel(const double* chunk_sum, const CamDev* cams, int n_views,
                                                           uint32_t n_chunks, float* out)
{
    const int v = blockIdx.x;
    if (v >= n_views) return;
    const CamDev& c = cams[v];
    const uint32_t c0 = c.hred_base, c1 = (v + 1 < n_views) ? cams[v + 1].hred_base : n_chunks;
    double acc = 0.0;
    for (uint32_t k = c0 + threadIdx.x; k < c1; k += 256) acc += chunk_sum[k];
    const double tot = block_sum_f64(acc);
    if (threadIdx.x == 0) out[v] = (float)(tot / ((double)c.W * (double)c.H));
}

// views of at most kOneBlocks blocks: one workgroup a view, one launch instead of two.  Both sides
// as a step's time in us, one launch / two: 4,000 blocks 114 / 120, 10,240 124 / 127, 17,172 136.5 /
// 136.8, 20,520 143.0 / 142.4, 22,800 147 / 146, 26,800 155 / 152, 32,640 166 / 162.
constexpr uint32_t kOneThreads = 1024, kOneBlocks = 20u * kOneThreads;

__global__ __launch_bounds__(kOneThreads) void entropy_one_kernel(const float* block_H, const CamDev* cams, float* out)
{
    __shared__ double s_w[kOneThreads / 64];
    const CamDev& c = cams[blockIdx.x];
    const uint32_t nb = c.n_wblocks;
    double acc = 0.0;
    for (uint32_t b0 = threadIdx.x; b0 < nb; b0 += 8u * kOneThreads) {
        float h[8];                                          // in flight together
#pragma unroll
        for (uint32_t k = 0; k < 8u; ++k) {
            const uint32_t b = b0 + k * kOneThreads;
            h[k] = b < nb ? block_H[c.block_base + b] : 0.f;
        }
#pragma unroll
        for (uint32_t k = 0; k < 8u; ++k) acc += (double)h[k];
    }
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) acc += __shfl_xor(acc, o, 64);
    if ((threadIdx.x & 63u) == 0u) s_w[threadIdx.x >> 6] = acc;
    __syncthreads();
    if (threadIdx.x == 0) {
        double tot = 0.0;
#pragma unroll
        for (uint32_t w = 0; w < kOneThreads / 64u; ++w) tot += s_w[w];
        out[blockIdx.x] = (float)(tot / ((double)c.W * (double)c.H));
    }
}

// persistent grids: as many workgroups as fit on the device at once
template <typename K>
uint32_t resident_groups(K kernel, uint32_t want)
{
    int dev = 0, cus = 0, per_cu = 0;
    (void)hipGetDevice(&dev);
    (void)hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev);
    (void)hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, kernel, 256, 0);
    uint32_t g = (uint32_t)(cus > 0 ? cus : 256) * (uint32_t)(per_cu > 0 ? per_cu : 1);
    return g < want ? g : want;
}

template <int B, bool RENDER>
hipError_t fwd_launch(const BlendFwdArgs& a, hipStream_t s)
{
    const uint32_t groups = (a.n_blocks + kWavesPerGroup - 1) / kWavesPerGroup;
    if (a.slotted) {                       // one 8x8 block per workgroup, a wavefront per 4x4 block
        hipLaunchKernelGGL(blend_fwd_slot_kernel<RENDER>, dim3(a.n_blocks), dim3(256), 0, s, a);
    } else if (a.spt == 4 && a.shared_batches) {  // one tile per workgroup, batches shared by its 4 blocks
        if (a.queues)
            hipLaunchKernelGGL((blend_fwd_shared_kernel<B, true, RENDER>),
                               dim3(resident_groups(blend_fwd_shared_kernel<B, true, RENDER>, groups)), dim3(256), 0,
                               s, a);
        else
            hipLaunchKernelGGL((blend_fwd_shared_kernel<B, false, RENDER>), dim3(groups), dim3(256), 0, s, a);
    } else {                               // one 8x8 block per wavefront, its own batches
        if (a.queues)
            hipLaunchKernelGGL((blend_fwd_kernel<B, true, RENDER>),
                               dim3(resident_groups(blend_fwd_kernel<B, true, RENDER>, groups)), dim3(256), 0, s, a);
        else if (a.tile_order && a.mixed) {
            const uint32_t n_slot = kMixedTiles * (uint32_t)a.spt, rest = a.n_blocks - n_slot;
            hipLaunchKernelGGL((blend_fwd_mixed_kernel<B, RENDER>),
                               dim3(n_slot + (rest + kWavesPerGroup - 1) / kWavesPerGroup), dim3(256), 0, s, a);
        } else
            hipLaunchKernelGGL((blend_fwd_kernel<B, false, RENDER>), dim3(groups), dim3(256), 0, s, a);
    }
    return hipGetLastError();
}

template <int B>
hipError_t fwd_b(const BlendFwdArgs& a, hipStream_t s)
{
    return a.render_only ? fwd_launch<B, true>(a, s) : fwd_launch<B, false>(a, s);
}

template <int B>
hipError_t bwd_b(const BlendBwdArgs& a, hipStream_t s)
{
    static_assert(B <= 128, "the backward window is limited by LDS");
    const uint32_t groups = (a.n_blocks + kWavesPerGroup - 1) / kWavesPerGroup;
    if (a.queues) {
        if (a.spt == 4)
            hipLaunchKernelGGL((blend_bwd_kernel<B, true, true>),
                               dim3(resident_groups(blend_bwd_kernel<B, true, true>, groups)), dim3(256), 0, s, a);
        else
            hipLaunchKernelGGL((blend_bwd_kernel<B, false, true>),
                               dim3(resident_groups(blend_bwd_kernel<B, false, true>, groups)), dim3(256), 0, s, a);
    } else {
        if (a.spt == 4) hipLaunchKernelGGL((blend_bwd_kernel<B, true, false>), dim3(groups), dim3(256), 0, s, a);
        else hipLaunchKernelGGL((blend_bwd_kernel<B, false, false>), dim3(groups), dim3(256), 0, s, a);
    }
    return hipGetLastError();
}

}  // namespace

hipError_t launch_blend_fwd(const BlendFwdArgs& a, int lds_batch, hipStream_t s)
{
    if (a.n_blocks == 0) return hipSuccess;
    switch (lds_batch) {
        case 32: return fwd_b<32>(a, s);
        case 64: return fwd_b<64>(a, s);
        case 128: return fwd_b<128>(a, s);
        case 256: return fwd_b<256>(a, s);
    }
    return hipErrorInvalidValue;
}

hipError_t launch_blend_bwd(const BlendBwdArgs& a, int lds_batch, hipStream_t s)
{
    if (a.n_blocks == 0) return hipSuccess;
    if (a.slotted) {
        // dense from 6 tiles a CU (640x416, 200k Gaussians, 4,160 blocks: 167 us, dense 207;
        // 960x640, 9,600 blocks: 204 us, dense 162; at 6,600 blocks alike)
        if (a.spt == 4 && a.n_blocks > 6144u)
            hipLaunchKernelGGL((blend_bwd_slot_kernel<4, true>), dim3(a.n_blocks / 4u), dim3(1024), 0, s, a);
        else if (a.spt == 4)
            hipLaunchKernelGGL((blend_bwd_slot_kernel<4, false>), dim3(a.n_blocks / 4u), dim3(1024), 0, s, a);
        else
            hipLaunchKernelGGL((blend_bwd_slot_kernel<1, false>), dim3(a.n_blocks), dim3(256), 0, s, a);
        return hipGetLastError();
    }
    switch (lds_batch) {
        case 32: return bwd_b<32>(a, s);
        case 64: return bwd_b<64>(a, s);
        case 128: return bwd_b<128>(a, s);
    }
    return hipErrorInvalidValue;
}

hipError_t launch_invariants(const InvArgs& a, hipStream_t s)
{
    if (a.n_pix <= 0) return hipSuccess;
    const uint32_t blocks = (uint32_t)((a.n_pix + 255) / 256);
    hipLaunchKernelGGL(invariant_kernel, dim3(blocks), dim3(256), 0, s, a);
    return hipGetLastError();
}

hipError_t launch_entropy_mean(const float* block_H, const CamDev* cams, int n_views, uint32_t n_chunks,
                               uint32_t max_blocks, double* tmp, float* out, hipStream_t s)
{
    if (n_views == 0 || n_chunks == 0) return hipSuccess;
    if (max_blocks <= kOneBlocks) {
        hipLaunchKernelGGL(entropy_one_kernel, dim3(n_views), dim3(kOneThreads), 0, s, block_H, cams, out);
        return hipGetLastError();
    }
    hipLaunchKernelGGL(entropy_chunk_kernel, dim3(n_chunks), dim3(256), 0, s, block_H, cams, n_views, tmp);
    hipLaunchKernelGGL(entropy_mean_kernel, dim3(n_views), dim3(256), 0, s, tmp, cams, n_views, n_chunks, out);
    return hipGetLastError();
}

}  // namespace gsr
