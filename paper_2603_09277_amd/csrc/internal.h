// Internal declarations of the gfx950 rasterizer library: device-side camera
// record, kernel argument blocks and the host launchers each .hip file
// provides.  Not part of the public ABI (include/gsr.h is).
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace gsr {

constexpr int kWave = 64;          // CDNA wavefront width
constexpr int kBlockPx = 8;        // every wavefront blends one 8x8 pixel block
constexpr int kMaxViews = 64;

// Per-view camera and layout record, resident in device memory.
struct CamDev {
    int32_t W, H;
    float fx, fy, cx, cy;
    float R[9];
    float t[3];
    float near_z;
    float campos[3];               // camera centre in world space, -R^T t
    float limx, limy;              // 1.3 x half field of view (tan), Jacobian clamp
    int32_t gx, gy;                // tile grid of this view
    uint32_t tile_base;            // first global tile id of this view
    uint32_t n_wblocks;            // 8x8 wave blocks of this view (tiles x blocks per tile)
    uint32_t block_base;           // first global wave block of this view (tile-major numbering)
    uint32_t pad0, pad1;
    int64_t pix_base;              // first pixel of this view in the packed outputs
    double limx_d, limy_d;         // the clamp bounds in FP64 (the clamp decision is taken in FP64)
    uint32_t hred_base;            // first entropy-reduction chunk of this view (kRedChunk blocks each)
    uint32_t l1_base;              // first L1 block of this view (kL1Block pixels each)
};

// cameras handed to a kernel by value (its arguments hold 4 KB)
constexpr int kCamPack = 16;
struct CamPack {
    CamDev c[kCamPack];
};

constexpr int kRedChunk = 1024;    // 8x8 blocks summed per entropy-reduction chunk
constexpr int kL1Block = 256;      // threads per L1 block
constexpr int kL1Pix = 4 * kL1Block;   // pixels per L1 block (4 a thread)

// Projected record of one (view, Gaussian): three float4
//   r0 = (mean x, mean y, A', B')
//   r1 = (C', opacity, red, green)
//   r2 = (blue, L, kr, kc)  (L: cull level; kr = -B'/(2C'), kc = -B'/(2A'): where the
//        exponent's maximum along a pixel row / column lies)
// with the conic pre-scaled to log2 units: A' = -A log2(e)/2, B' = -B log2(e),
// C' = -C log2(e)/2, so that the exponent is A' dx^2 + B' dx dy + C' dy^2.
constexpr double kLog2e = 1.4426950408889634;
constexpr int kRecF4 = 3;
// mean per-tile list length from which the forward stages each batch once per
// 16x16 / 32x8 tile instead of once per 8x8 block, and the backward's window is 64
// entries instead of 128.  Both sides, per block / shared in us, forward; backward, of 26,800
// blocks at 1600x1060: mean 154 (150k Gaussians) 75 / 79; 155 / 150, 256 (250k) 89 / 91; 209 / 178,
// 513 (500k) 125 / 112; 279 / 238, 1,025 (1M) 177 / 141; 342 / 298.  Up to 20,480 blocks the
// per-block side is the mixed form (below) and the two meet later: 17,172 blocks at 1296x840, mean
// 207 78 / 104; 176 / 188, 260 82 / 100; 161 / 173, 413 112 / 121; 205 / 209, 823 149 / 151; 259 /
// 258: there the shared form is taken from 256 on although it is the slower one up to about 800.
constexpr double kSharedBatchMeanLen = 256.0;
// The blend's slotted form (four wavefronts an 8x8 block instead of one, see blend.hip): up
// to kSlotBlocks blocks, ten plain wavefronts a SIMD, below which the plain walks of the
// longest lists end on an idle chip; and, beyond 2,048 blocks, where lists are not so
// short that starting four wavefronts a block costs more than their walks (from two
// records a block).  Both sides, 16x16 tiles, plain -> slotted, forward / backward in us: 9,600
// blocks, 200k Gaussians 127 -> 91 / 236 -> 156, 1M 252 -> 247 / 377 -> 329; 17,172 blocks, 200k
// 90 -> 131 / 172 -> 224 (plain); 6,600 blocks, 5k (0.8 records a block) 12 -> 22 / 17 -> 27
// (plain); 2,688 blocks, 5k 14 -> 13 / 25 -> 15 (plain, with the mixed forward 10: 1.9 records a
// block).  It depends on sizes alone, so that every mode takes the same form for the same frame.
constexpr uint32_t kSlotBlocks = 10240;
constexpr uint32_t kSlotFewBlocks = 2048;
inline bool slotted_blend(uint32_t n_blocks, uint32_t records)
{
    return n_blocks <= kSlotFewBlocks || (n_blocks <= kSlotBlocks && records / 2u >= n_blocks);
}
// The backward takes it only up to 2^20 records.  Its sums over pixels are in another order
// than the plain form's, and single scale and rotation gradients that cancel show the order: by
// 3e-4 of their size at most at 500k and 1M records (6 scenes each), by up to 2.4e-3 at 2M.
// Against 64 bits both forms are as far off: over 14 scenes of 2k to 2M Gaussians within kSlotBlocks
// the relative L2 errors (2e-6 to 3.5e-4 by scene and attribute) and the median, 99 % point and
// maximum of the Gaussians' own errors are the same to a few per cent, the forms 1e-7 to 3.4e-6
// apart.  So the line is no bound on an error: it keeps frames of more records at the values of
// the plain form.
constexpr uint32_t kSlotBackward = 1u << 20;
inline bool slotted_backward(uint32_t n_blocks, uint32_t records)
{
    return records <= kSlotBackward && slotted_blend(n_blocks, records);
}
// The mixed forward (blend.hip): the kMixedTiles longest tiles slotted, the others plain, for
// lists short enough that tiles do not share batches.  Up to 20 plain wavefronts a SIMD,
// where the longest walks outlast the rest, and with half a record a block or more.  Both
// sides, plain -> mixed in us: 17,172 blocks, 200k Gaussians 90 -> 78, 30k 30 -> 26, 3k 12 -> 15
// (plain); 6,600 blocks, 5k 12 -> 11; 17,010 blocks of 8x8 tiles, 300k 124 -> 114, of 32x8, 100k
// 51 -> 34; 26,800 blocks, 200k 95 -> 89, of 8x8 tiles 74 -> 82 (plain); 39,400 blocks, 250k 109 ->
// 127 (plain).  The number of tiles rests on the first alone: 64 took 80 us, 192 74, 256 79.
constexpr uint32_t kMixedTiles = 128;
constexpr uint32_t kMixedBlocks = 20480;
inline bool mixed_blend(uint32_t n_blocks, uint32_t records)
{
    return n_blocks > kSlotFewBlocks && n_blocks <= kMixedBlocks && records >= n_blocks / 2u;
}
static_assert(4u * kMixedTiles <= kSlotFewBlocks, "there are tiles left for the plain form");
// persistent blend kernels: one work queue per XCD, heads 128 bytes apart
constexpr uint32_t kQueues = 8;
constexpr uint32_t kQueueStride = 32;
// 2D gradient accumulator per (view, Gaussian): 9 floats
//   dmean x, dmean y, dA, dB, dC, dopacity, dred, dgreen, dblue
constexpr int kG2 = 9;
// per-pair gradient row: the 9 components and a stamp (uint32 bits) naming the
// frame whose backward wrote it; rows with another stamp count as zero (every
// backward of one frame writes the same rows: the entries some pixel blended)
constexpr int kRowF = 10;

struct ProjectFwdArgs {
    const float* means;
    const float* scales;
    const float* quats;
    const float* opac;
    const void* sh;
    uint32_t n;
    int32_t n_views;
    uint32_t flags;
    int32_t tile_shift_x, tile_shift_y;   // log2 of the tile shape
    const CamDev* cams;
    float4* rec;                          // [V*n][3]
    uint2* trect;                         // [V*n] (x0 | x1 << 16, y0 | y1 << 16), inclusive tile bounds
                                          //   (empty: x1 < x0); rect8: x0, x1, y0, y1 of 8 bits in one
                                          //   32-bit word [V*n] (carry_rects)
    bool rect8;
    int32_t* radius;                      // [V*n]
    float* depth;                         // [V*n] camera z: the sort's keys, by their bits (positive wherever
                                          //   the record has pairs; the others' place has no effect)
    // pair counting (count null: none): the sum of tiles touched of view v -> count_total[v], by
    // way of project_count_words(n, n_views) words at count; only views from store_from on are
    // stored, at the records of views 0, 1, ...
    uint64_t* count;
    uint64_t* count_total;
    int32_t store_from;
};

struct ProjectBwdArgs {
    const float* means;
    const float* scales;
    const float* quats;
    const float* opac;
    const void* sh;
    uint32_t n;
    int32_t n_views;
    uint32_t flags;
    const CamDev* cams;
    const float* grad2d;                  // [V*n][9], valid where rec_stamp == *stamp (else zero)
    const uint32_t* rec_stamp;            // [V*n]
    const uint32_t* stamp;                // the frame's stamp (device)
    float* g_means;
    float* g_scales;
    float* g_quats;
    float* g_opac;
    void* g_sh;
    // opacity regulariser fused into the projection backward (0 / null: none): g_opac also
    // gets dL_O/dsigma of L_O = reg_w / n sum exp(-(sigma - 0.5)^2 / 0.05), and, if reg_partial
    // is set, every wavefront writes the sum of its Gaussians' exp terms (FP64) to
    // reg_partial[4 * block + wavefront]
    float reg_w;
    double* reg_partial;
};

struct BlendFwdArgs {
    const float4* rec;
    const uint32_t* pair_vals;            // sorted pairs: emission index e of each (tile, Gaussian) pair
    const uint32_t* emit_vg;              // [P] record (view*n + Gaussian index) of emission index e
    const uint2* ranges;
    const CamDev* cams;
    int32_t n_views;
    int32_t tile_shift_x, tile_shift_y;
    int32_t spt;                          // 8x8 blocks per tile: 1 or 4
    uint32_t n_blocks;                    // 8x8 wave blocks over all views
    float* out_rgb;
    float* out_H;                         // out_H, out_T, out_nc, block_H: unused by the render-only variant
    float* out_T;
    int32_t* out_nc;
    float* block_H;                       // [n_blocks] sum of H over the block
    uint4* block_cnt;                     // [n_blocks][2]: (list positions visited, sum of n_contrib, blended, 0),
                                          //   (alpha tests made, 0: the backward writes its alpha tests, 0, 0)
    uint32_t* queues;                     // persistent mode: kQueues heads kQueueStride words apart, zeroed; or null
    int32_t render_only;                  // 1: colour only (no entropy, no saved state)
    const uint32_t* tile_order;           // [n_tiles] tiles, longest list first (hardware dispatch); or null
    int32_t shared_batches;               // 16x16 / 32x8 tiles: stage each batch once for the 4 blocks
    int32_t slotted;                      // the slotted form (no queues: a workgroup an 8x8 block)
    int32_t mixed;                        // the mixed form may be taken (mixed_blend)
};

struct BlendBwdArgs {
    const float4* rec;
    const uint32_t* pair_vals;            // sorted pairs: emission index e (the pair's gradient row)
    const uint32_t* emit_vg;              // [P] record of emission index e
    const uint2* ranges;
    const CamDev* cams;
    int32_t n_views;
    int32_t tile_shift_x, tile_shift_y;
    int32_t spt;
    uint32_t n_blocks;
    const float* T_final;
    const int32_t* n_contrib;
    const float* grad_rgb;
    const float* grad_H;                  // may be null
    const float* grad_LE;                 // [V] may be null
    float* pair_grad;                     // [P][10] per-pair gradient rows (9 values), emission order
    uint32_t* pair_stamp;                 // [P] stamp of the frame whose backward wrote each row
    const uint32_t* stamp;                // this frame's row stamp
    uint32_t* queues;                     // persistent mode: kQueues heads kQueueStride words apart, zeroed; or null
    const uint32_t* tile_order;           // [n_tiles] tiles, longest list first (hardware dispatch); or null
    uint4* block_cnt;                     // the forward's block counts: word 1 of [2 wb + 1] gets the
                                          //   backward's alpha tests of block wb
    int32_t slotted;                      // the slotted form (no queues: a workgroup a tile)
};

// Debug check of Eq. 9 after a forward (GSR_DEBUG_INVARIANTS): per pixel, the sum of
// the blending weights plus the final transmittance equals one.
struct InvArgs {
    const float4* rec;
    const uint32_t* pair_vals;
    const uint32_t* emit_vg;
    const uint2* ranges;
    const CamDev* cams;
    int32_t n_views;
    int32_t tile_shift_x, tile_shift_y;
    int64_t n_pix;
    const float* T_final;
    const int32_t* n_contrib;
    uint32_t* counters;                   // [6] max |sum w + T - 1| (float bits), [7] pixels past the bound
};

// ---- launchers (return hipError_t of the launch) ----
hipError_t launch_project_fwd(const ProjectFwdArgs& a, int sh_degree, bool sh_bf16, hipStream_t s);
inline size_t project_count_words(uint32_t n, int n_views) { return 4 * (size_t)((n + 255u) / 256u) * (size_t)n_views; }
hipError_t launch_project_bwd(const ProjectBwdArgs& a, int sh_degree, bool sh_bf16, hipStream_t s);

// The tile rectangles of large depth sorts travel with the sort as 32-bit words, from
// `records` on, where the large passes begin, if every view has at most 256 x 256 tiles: the four
// downsweeps and the scan of 24M records take 0.52 ms so (0.88 with the rectangles gathered at the
// end), with histograms and spines 0.65; of 3.3M 114 us (136); the small passes are bound by latency, and 1M records gather in 15 us.
constexpr uint32_t kCarryFrom = 1u << 21;
inline bool carry_rects(uint32_t records, int gx, int gy) { return records >= kCarryFrom && gx <= 256 && gy <= 256; }

// first[b] = pairs of the records before workgroup b of launch_duplicate, in depth order;
// their total -> *total (uint32), *overflow |= 1 if it does not fit in 32 bits.  carried:
// rect_s holds the 32-bit rectangles in depth order; else rect_s[i] = trect[order[i]].  first
// holds scan_tmp_words(n) words.
size_t scan_tmp_words(uint32_t n);
hipError_t launch_scan(const uint2* trect, const uint32_t* order, uint32_t n, uint2* rect_s, bool carried, uint32_t* first,
                       uint32_t* total, uint32_t* overflow, hipStream_t s);

// at most kSmallBin records: the depth order of all records (keys) and launch_scan's outputs
// for it, in one launch
constexpr uint32_t kSmallBin = 6144;
hipError_t launch_small_bin(const uint32_t* keys, const uint2* trect, uint32_t n, uint32_t* order, uint32_t* first,
                            uint2* rect_s, uint32_t* total, uint32_t* overflow, hipStream_t s);

// words of scratch of every radix pass over at most n_max items
size_t radix_tmp_words(uint32_t n_max);
// the depth order of n records (depth: their keys): stable LSD passes -> order[0]; keys and
// order[1] are scratch.  rect non-null (carry_rects): rect_s[0][i] = rect[order[0][i]], rect_s[1]
// scratch
hipError_t launch_depth_sort(const uint32_t* depth, uint32_t* const (&keys)[2], uint32_t* const (&order)[2], uint32_t n,
                             uint32_t* tmp, const uint32_t* rect, uint32_t* const (&rect_s)[2], hipStream_t s);
// passes of 8 bits that the tile ids take
int tile_sort_passes(uint32_t n_tiles);
// stable sort of the pairs (keys[0]: launch_duplicate's tile ids) by tile: the sorted
// emission indices -> vals[passes & 1]; the item count is min(*total, cap), read on the
// device.  The last pass writes no keys: it folds each tile's [start, end) into ranges[tile] by
// atomic min / max (initialised to (0xffffffff, 0) by launch_frame_begin; tiles without
// pairs keep that until launch_tile_order / launch_ranges_finish).
hipError_t launch_tile_sort(uint32_t* const (&keys)[2], uint32_t* const (&vals)[2], uint32_t n_tiles,
                            const uint32_t* total, uint32_t cap, uint2* ranges, uint32_t* tmp, hipStream_t s);

// write the tile id of every (tile, Gaussian) pair, Gaussians in depth order, at
// its emission index (keys[e]: 16-bit words up to 65,536 tiles, else 32-bit), and
// emit_vg[e] = view*n + Gaussian index; the pairs' sort values are their emission indices
// (the tile sort's first pass takes them as the items' indices)
hipError_t launch_duplicate(const uint32_t* order, const uint2* rect_s, bool carried, const uint32_t* first,
                            const CamDev* cams, uint32_t n, uint32_t vn, uint32_t n_tiles, const uint32_t* total, uint32_t cap,
                            uint32_t* keys, uint32_t* emit_vg, uint32_t* overflow, hipStream_t s);
// grad2d[vg] = sum of the per-pair rows pair_grad[10 e .. 10 e + 8] with pair_stamp[e] == *stamp over the Gaussian's
// emission range, written, with rec_stamp[vg] = *stamp, for every (view, Gaussian) with at least one such
// row; every other grad2d row is zero by definition and left untouched, with its old stamp;
// carry holds seg_carry_bytes(cap) bytes
size_t seg_carry_bytes(uint32_t cap);
hipError_t launch_grad_reduce(const float* pair_grad, const uint32_t* pair_stamp, const uint32_t* stamp,
                              const uint32_t* emit_vg, uint32_t vn,
                              const uint32_t* total, uint32_t cap, float* grad2d, uint32_t* rec_stamp, void* carry,
                              hipStream_t s);

// a forward's counters: pair total and overflow flag cleared, row stamp (counters[4]) advanced;
// the n_tiles tile bounds in ranges set to (0xffffffff, 0), the words after them up to
// ranges[n_words) cleared; n_cams cameras stored to `cams` from kernel arguments (a further
// launch for every kCamPack past the first)
hipError_t launch_frame_begin(uint32_t* counters, uint32_t* ranges, uint32_t n_tiles, uint32_t n_words,
                              const CamDev* host_cams, int n_cams, CamDev* cams, hipStream_t s);
hipError_t launch_fill_u32(uint32_t* p, uint32_t value, size_t count, hipStream_t s);
// tiles without pairs set to [0, 0), then order[n_tiles]: the tiles by decreasing list length
// (16 classes per octave);
// hist: 512 words, zeroed (bucket counts, then bucket fill counters)
constexpr uint32_t kTileHistWords = 512;
hipError_t launch_tile_order(uint2* ranges, uint32_t n_tiles, uint32_t* hist, uint32_t* order, hipStream_t s);
// tiles that the last tile-sort pass gave no bounds (no pairs): [0, 0) (persistent scheduling, which takes no order)
hipError_t launch_ranges_finish(uint2* ranges, uint32_t n_tiles, hipStream_t s);


hipError_t launch_blend_fwd(const BlendFwdArgs& a, int lds_batch, hipStream_t s);
hipError_t launch_blend_bwd(const BlendBwdArgs& a, int lds_batch, hipStream_t s);
hipError_t launch_invariants(const InvArgs& a, hipStream_t s);
// n_l1_blocks = sum over views of ceil(W H / kL1Block); tmp holds n_l1_blocks doubles
// L_O = w / n * sum exp(-(sigma - 0.5)^2 / 0.05); grad[i] += dL_O/dsigma_i (grad may be null);
// *loss (device, may be null); tmp holds opacity_reg_tmp_words(n) doubles
size_t opacity_reg_tmp_words(int64_t n);
hipError_t launch_opacity_reg(const float* opac, int64_t n, float w, float* grad, float* loss, double* tmp,
                              hipStream_t s);
// L_O = w / n * sum of the n_partial FP64 partial sums, in a fixed order -> *loss
hipError_t launch_opacity_reg_reduce(const double* partial, uint32_t n_partial, int64_t n, float w, float* loss,
                                     hipStream_t s);
// D-SSIM of packed views: loss[v] (device, may be null) = weight (1 - SSIM(x, y)); grad
// (may be null) += dloss/dx; x, y, grad [pixels][3]; tmp holds ssim_tmp_bytes bytes
struct SsimSizes {
    const int32_t* w0;                    // view v's width and height: w0[v * stride], h0[v * stride]
    const int32_t* h0;
    size_t stride;
    int n;
    int32_t w(int v) const { return w0[(size_t)v * stride]; }
    int32_t h(int v) const { return h0[(size_t)v * stride]; }
};
size_t ssim_tmp_bytes(const SsimSizes& z, bool with_grad);
hipError_t launch_dssim(const float* x, const float* y, const SsimSizes& z, float weight, float* grad, float* loss,
                        void* tmp, hipStream_t s);
// one bias-corrected Adam step on raw parameters (kind 0 identity, 1 exp, 2 sigmoid activation)
hipError_t launch_adam(float* raw, float* m, float* v, float* act, const float* grad_act, int64_t n, int kind,
                       float lr, float b1, float b2, float eps, int64_t step, hipStream_t s);
// s <- zeta * s in place over count floats; log_s (may be null) += log(zeta)
hipError_t launch_scale_reset(float* scales, float* log_scales, int64_t count, float zeta, hipStream_t s);
hipError_t launch_l1(const float* rgb, const float* target, const CamDev* cams, int n_views, uint32_t n_l1_blocks,
                     float weight, float* grad, float* loss, double* tmp, hipStream_t s);
// n_chunks = sum over views of ceil(blocks_v / kRedChunk); tmp holds n_chunks doubles
// max_blocks: the most blocks of one view
hipError_t launch_entropy_mean(const float* block_H, const CamDev* cams, int n_views, uint32_t n_chunks,
                               uint32_t max_blocks, double* tmp, float* out_mean, hipStream_t s);

}  // namespace gsr
