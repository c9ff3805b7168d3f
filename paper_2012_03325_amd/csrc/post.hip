// Bloom (paper Sec. 5.3) and final compositing with ACES tone mapping and
// gamma correction (Sec. 5.4).
//
// gfx950 mapping:
//  * bloom_down: one workgroup per 32x32-pixel tile reads the HDR planes
//    once (one level-1 texel per thread, its twelve loads in flight together),
//    forms the bright map and its 2x2 means, and builds pyramid levels 1..5 of
//    that tile in LDS (16x16 level-1 texels halve down to one at level 5),
//    writing every level once.
//  * bloom_blur: all levels in one launch; a wavefront holds its tile's columns
//    in registers and applies the separable [1 4 6 4 1] / 16 binomial (clamp to
//    edge) horizontally across lanes, then vertically.
//  * composite: a wavefront covers 64 columns x 8 rows, a thread one column
//    of 8 pixels; every blurred level is interpolated at the column (rows
//    first, then between two rows per pixel) in registers; each thread adds
//    the upsampled levels to its pixels, applies exposure, the ACES fit,
//    gamma and 8-bit rounding, and writes one 32-bit RGBA word per pixel
//    (small images: half a strip per wavefront, see kCompositeHalfStrips).
//  * pyramid texels are float4 (three floats before the blur), or four halves in the FP16 form.
//  * every stage has a single-view kernel and a batched kernel that walks the
//    work items of many views.
#include "device_common.hpp"
#include "launch.hpp"
#include "post_tiles.hpp"

namespace epb {

// ---------------------------------------------------------------------------
// kernels: single view (XCD-aware tile order) and batched (persistent range)
// ---------------------------------------------------------------------------
template <typename TH, typename TP>
__global__ void __launch_bounds__(256) k_bloom_down(const PostDesc c, int tiles) {
    __shared__ DownLds sm;
    bloom_down_tile<TH, TP>(c, xcd_tile(blockIdx.x, tiles), sm);
}

template <typename TP>
__global__ void __launch_bounds__(256) k_bloom_down_from1(const PostDesc c, int tiles) {
    __shared__ DownLds sm;
    bloom_down_from1_tile<TP>(c, xcd_tile(blockIdx.x, tiles), sm);
}

template <typename TP>
__global__ void __launch_bounds__(256) k_bloom_blur(const PostDesc c) {
    bloom_blur_item<kBloomSingle.cols, kBloomSingle.rows, TP>(c, blockIdx.x);
}

template <typename TH, typename TP>
__global__ void __launch_bounds__(kPostTx) __attribute__((amdgpu_waves_per_eu(4))) k_composite(const PostDesc c, int tiles) {
    composite_tile<sizeof(TP) == 8, WholeStrip, TH, TP>(c, xcd_tile(blockIdx.x, tiles), (int)threadIdx.x);
}

// Without a pyramid: the HDR image's own strips, in few registers and so with many wavefronts
// (3840x2160 in float32 21.4 us, 22.4 with the registers of the levels; 4096^2 in half storage 30.2 / 32.6).
template <typename TH>
__global__ void __launch_bounds__(kPostTx) k_composite_plain(const PostDesc c, int tiles) {
    PostDesc d = c;
    d.nl = 0;  // known to the compiler
    composite_tile<true, WholeStrip, TH, Half4>(d, xcd_tile(blockIdx.x, tiles), (int)threadIdx.x);
}

// Half a strip per wavefront (see kCompositeHalfStrips).
template <typename TH, typename TP>
__global__ void __launch_bounds__(kPostTx) k_composite_halves(const PostDesc c, int halves) {
    constexpr int kHalf = kPostTy / 2;
    int b = xcd_tile(blockIdx.x, halves), lane = (int)threadIdx.x;
    if (b & 1) composite_tile<true, StripRows<kHalf, kHalf>, TH, TP>(c, b >> 1, lane);
    else composite_tile<true, StripRows<0, kHalf>, TH, TP>(c, b >> 1, lane);
}

template <typename TH, typename TP>
__global__ void __launch_bounds__(256) k_bloom_down_batch(const void *__restrict__ table) {
    __shared__ DownLds sm;
    const BatchHeader *h = (const BatchHeader *)table;
    const int *start = batch_start(table, kStDown);
    const ViewDesc *views = batch_views(table);
    XcdRange w = xcd_range(h->total[kStDown]);
    for (int it = w.lb; it < w.count; it += w.stride) {
        int g = w.first + it;
        int v = find_view(start, h->n_views, g);
        bloom_down_tile<TH, TP>(views[v].post, g - start[v], sm);
    }
}

template <typename TP>
__global__ void __launch_bounds__(256) k_bloom_down_from1_batch(const void *__restrict__ table) {
    __shared__ DownLds sm;
    const BatchHeader *h = (const BatchHeader *)table;
    const int *start = batch_start(table, kStDown);
    const ViewDesc *views = batch_views(table);
    XcdRange w = xcd_range(h->total[kStDown]);
    for (int it = w.lb; it < w.count; it += w.stride) {
        int g = w.first + it;
        int v = find_view(start, h->n_views, g);
        bloom_down_from1_tile<TP>(views[v].post, g - start[v], sm);
    }
}

template <typename TP>
__global__ void __launch_bounds__(256) k_bloom_blur_batch(const void *__restrict__ table) {
    const BatchHeader *h = (const BatchHeader *)table;
    const int *start = batch_columns(table, kColBloom);
    const ViewDesc *views = batch_views(table);
    XcdRange w = xcd_range(h->columns[kColBloom]);
    for (int it = w.lb; it < w.count; it += w.stride) {
        int g = w.first + it;
        int v = find_view(start, h->n_views, g);
        bloom_blur_item<kBloomBatch.cols, kBloomBatch.rows, TP>(views[v].post, g - start[v]);
    }
}

template <typename TH, typename TP>
__global__ void __launch_bounds__(kPostTx) __attribute__((amdgpu_waves_per_eu(4))) k_composite_batch(const void *__restrict__ table) {
    const BatchHeader *h = (const BatchHeader *)table;
    const int *start = batch_start(table, kStComposite);
    const ViewDesc *views = batch_views(table);
    XcdRange w = xcd_range(h->total[kStComposite]);
    for (int it = w.lb; it < w.count; it += w.stride) {
        int g = w.first + it;
        int v = find_view(start, h->n_views, g);
        composite_tile<sizeof(TP) == 8, WholeStrip, TH, TP>(views[v].post, g - start[v], (int)threadIdx.x);
    }
}

// ---------------------------------------------------------------------------
// host side
// ---------------------------------------------------------------------------
PostPlan post_plan(int W, int H, int levels, epb_dtype pyr_dtype) {
    PostPlan q{};
    q.W = W;
    q.H = H;
    q.levels = levels;
    q.texel_bytes = pyr_dtype == EPB_F16 ? 8 : 16;
    q.lw[0] = W;
    q.lh[0] = H;
    for (int l = 1; l < levels; ++l) {
        q.lw[l] = (q.lw[l - 1] + 1) / 2;
        q.lh[l] = (q.lh[l - 1] + 1) / 2;
    }
    size_t off = 0;
    for (int l = 1; l < levels; ++l) {  // blurred levels first (documented scratch layout)
        q.off_blur[l] = off;
        off += (size_t)q.lw[l] * q.lh[l] * q.texel_bytes;
    }
    off = (off + 255) & ~size_t(255);
    for (int l = 1; l < levels; ++l) {
        q.off_raw[l] = off;
        off += (size_t)q.lw[l] * q.lh[l] * q.texel_bytes;
    }
    q.bytes = (off + 255) & ~size_t(255);
    if (q.bytes == 0) q.bytes = 256;
    return q;
}

PostDesc post_desc(const PostPlan &q, const void *hdr, float threshold, float strength, float exposure,
                   float gamma, int tonemap, uint8_t *ldr, void *scratch, BlurShape blur) {
    PostDesc c{};
    c.W = q.W;
    c.H = q.H;
    c.nl = q.levels - 1;
    c.texel_half = q.texel_bytes == 8;
    char *sc = (char *)scratch;
    for (int l = 0; l < q.levels; ++l) {
        c.lw[l] = q.lw[l];
        c.lh[l] = q.lh[l];
        if (l >= 1) {
            c.raw[l] = sc + q.off_raw[l];
            c.blur[l] = sc + q.off_blur[l];
        }
    }
    int nb = 0;
    for (int l = 1; l <= c.nl; ++l) {
        c.blk_start[l] = nb;
        nb += ceil_div(c.lw[l], blur.cols) * ceil_div(c.lh[l], 4 * blur.rows);
    }
    c.blk_start[c.nl + 1] = nb;
    c.threshold = threshold;
    c.strength = strength;
    c.exposure = exposure;
    c.inv_gamma = 1.0f / gamma;
    c.tonemap = tonemap;
    c.hdr = hdr;
    c.ldr = (uint32_t *)ldr;
    return c;
}

// Tiles of 32 x 16 texels of all levels, the blur stage's work items in a batch table.
int bloom_blur_tiles(const PostDesc &c) {
    int n = 0;
    for (int l = 1; l <= c.nl; ++l) n += ceil_div(c.lw[l], kBloomTile.cols) * ceil_div(c.lh[l], 4 * kBloomTile.rows);
    return n;
}

int post_items(const PostDesc &c, int stage) {
    if (stage == kStDown) return c.nl >= 1 ? ceil_div(c.lw[1], kDownTile) * ceil_div(c.lh[1], kDownTile) : 0;
    if (stage == kStBloomBlur) return c.nl >= 1 ? c.blk_start[c.nl + 1] : 0;
    return ceil_div(c.W, kPostTx) * ceil_div(c.H, kPostTy);
}

// Up to this many 64 x 8 strips (one and a half wavefronts per SIMD) a wavefront takes half a
// strip: the chip is not full and a wavefront's own instructions are the time.  A half strip
// interpolates three quarters of a strip's level rows (13 of 17), so that larger images take whole ones.  Composite
// of 256x256 in float32 5.0 us by strips, 3.6 by halves, quarters gain nothing more (launches
// bound bloom and tone mapping, 12.9 / 12.1 us); 1003x667 (1344 strips) 5.9 / 5.1; bloom and tone
// mapping of 1280x720 (1800) 17.3 / 17.6 in half storage, 1920x1080 22.6 / 23.5.
constexpr int kCompositeHalfStrips = 1536;

template <typename TH, typename TP>
static void launch_post(const PostDesc &c, bool level1_given, hipStream_t s) {
    if (c.nl >= 1) {
        int tiles = post_items(c, kStDown);
        if (!level1_given)
            hipLaunchKernelGGL((k_bloom_down<TH, TP>), dim3(tiles), dim3(256), 0, s, c, tiles);
        else if (c.nl >= 2)
            hipLaunchKernelGGL(k_bloom_down_from1<TP>, dim3(tiles), dim3(256), 0, s, c, tiles);
        hipLaunchKernelGGL(k_bloom_blur<TP>, dim3(post_items(c, kStBloomBlur)), dim3(256), 0, s, c);
    }
    int tiles = post_items(c, kStComposite);
    if (tiles <= kCompositeHalfStrips) {
        hipLaunchKernelGGL((k_composite_halves<TH, TP>), dim3(2 * tiles), dim3(kPostTx), 0, s, c, 2 * tiles);
        return;
    }
    if (c.nl == 0) hipLaunchKernelGGL(k_composite_plain<TH>, dim3(tiles), dim3(kPostTx), 0, s, c, tiles);
    else hipLaunchKernelGGL((k_composite<TH, TP>), dim3(tiles), dim3(kPostTx), 0, s, c, tiles);
}

template <typename TH, typename TP>
static void launch_post_batch_t(const BatchHeader &h, const void *table, hipStream_t s) {
    if (h.total[kStDown] > 0 && h.fuse_bloom)  // level 1 came from the shading stage
        hipLaunchKernelGGL(k_bloom_down_from1_batch<TP>, dim3(batch_grid(h.total[kStDown], h.blocks_per_cu)),
                           dim3(256), 0, s, table);
    else if (h.total[kStDown] > 0)
        hipLaunchKernelGGL((k_bloom_down_batch<TH, TP>), dim3(batch_grid(h.total[kStDown], h.blocks_per_cu)),
                           dim3(256), 0, s, table);
    if (h.columns[kColBloom] > 0)
        hipLaunchKernelGGL(k_bloom_blur_batch<TP>, dim3(batch_grid(h.columns[kColBloom], h.blocks_per_cu)),
                           dim3(256), 0, s, table);
    hipLaunchKernelGGL((k_composite_batch<TH, TP>), dim3(batch_grid(h.total[kStComposite], h.blocks_per_cu)),
                       dim3(kPostTx), 0, s, table);
}

hipError_t launch_bloom_tonemap(const PostDesc &c, epb_dtype hdr_dtype, epb_dtype pyr_dtype, hipStream_t s,
                                bool level1_given) {
    bool h16 = hdr_dtype == EPB_F16, p16 = pyr_dtype == EPB_F16;
    if (!h16 && !p16) launch_post<float, float4>(c, level1_given, s);
    else if (!h16 && p16) launch_post<float, Half4>(c, level1_given, s);
    else if (h16 && !p16) launch_post<__half, float4>(c, level1_given, s);
    else launch_post<__half, Half4>(c, level1_given, s);
    return hipGetLastError();
}

hipError_t launch_post_batch(const BatchHeader &h, const void *table, hipStream_t s) {
    bool h16 = h.hdr_dtype == EPB_F16, p16 = h.pyr_dtype == EPB_F16;
    if (!h16 && !p16) launch_post_batch_t<float, float4>(h, table, s);
    else if (!h16 && p16) launch_post_batch_t<float, Half4>(h, table, s);
    else if (h16 && !p16) launch_post_batch_t<__half, float4>(h, table, s);
    else launch_post_batch_t<__half, Half4>(h, table, s);
    return hipGetLastError();
}

}  // namespace epb
