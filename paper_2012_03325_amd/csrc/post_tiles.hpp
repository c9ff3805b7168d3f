// Per-tile device functions of bloom and compositing (paper Sec. 5.3, 5.4);
// shared by the single-view, batched and persistent kernels.
#pragma once

#include "device_common.hpp"

namespace epb {

__device__ __forceinline__ float4 add4(float4 a, float4 b) {
    return make_float4(a.x + b.x, a.y + b.y, a.z + b.z, 0.0f);
}
__device__ __forceinline__ float4 scale4(float4 a, float s) { return make_float4(a.x * s, a.y * s, a.z * s, 0.0f); }

__device__ __forceinline__ unsigned level_texel(const PostDesc &c, int L, int X, int Y) {
    return __umul24((unsigned)Y, (unsigned)c.lw[L]) + (unsigned)X;
}

// ---------------------------------------------------------------------------
// bloom_down: one 16x16 level-1 tile (32x32 pixels) -> levels 1..5 of that tile
// ---------------------------------------------------------------------------
struct DownLds {
    float4 s1[16][17];
    float4 s2[8][9];
    float4 s3[4][5];
    float4 s4[2][3];
};

// Level L texel (lx, ly) of tile (bx, by) as the mean of its in-range
// children in `src`; kept in `dst` for the next level when that is non-null.
template <int L, int N, typename TP, typename SRC, typename DST>
__device__ __forceinline__ void down_level(const PostDesc &c, int bx, int by, SRC src, DST dst) {
    typedef typename RawTexel<TP>::type TR;
    int t = threadIdx.x;
    if (t >= N * N) return;
    int lx = t % N, ly = t / N;
    int X = bx * N + lx, Y = by * N + ly;
    float4 v = make_float4(0, 0, 0, 0);
    if (X < c.lw[L] && Y < c.lh[L]) {
        // child (2X, 2Y) is always in range (each level is the previous one halved,
        // rounded up); 1 / n for n = 1, 2 or 4 children is a product of halves, exact
        bool x1 = 2 * X + 1 < c.lw[L - 1], y1 = 2 * Y + 1 < c.lh[L - 1];
        v = add4(v, src[2 * ly][2 * lx]);
        if (x1) v = add4(v, src[2 * ly][2 * lx + 1]);
        if (y1) v = add4(v, src[2 * ly + 1][2 * lx]);
        if (x1 && y1) v = add4(v, src[2 * ly + 1][2 * lx + 1]);
        v = scale4(v, (x1 ? 0.5f : 1.0f) * (y1 ? 0.5f : 1.0f));
        sto((TR *)c.raw[L], level_texel(c, L, X, Y) * (unsigned)sizeof(TR), pack<TR>(v));
    }
    if (dst) dst[ly][lx] = v;
}

// Levels 2..5 of tile (bx, by) from its level-1 texels in sm.s1 (the level
// count is uniform: barriers are safe).
template <typename TP>
__device__ __forceinline__ void down_levels_2_to_5(const PostDesc &c, int bx, int by, DownLds &sm) {
    __syncthreads();
    if (c.nl >= 2) {
        down_level<2, 8, TP>(c, bx, by, sm.s1, sm.s2);
        __syncthreads();
    }
    if (c.nl >= 3) {
        down_level<3, 4, TP>(c, bx, by, sm.s2, sm.s3);
        __syncthreads();
    }
    if (c.nl >= 4) {
        down_level<4, 2, TP>(c, bx, by, sm.s3, sm.s4);
        __syncthreads();
    }
    if (c.nl >= 5) down_level<5, 1, TP>(c, bx, by, sm.s4, (float4(*)[3]) nullptr);
    __syncthreads();  // the next item of a batched launch refills the LDS
}

// Two horizontally adjacent pixels of a plane (index p even, so the pair is
// 8-byte aligned in float32 and 4-byte aligned in half): one load.
__device__ __forceinline__ void ld_pair(const float *b, unsigned p, float &u, float &v) {
    float2 q = ldo((const float2 *)b, p * 4u);
    u = q.x;
    v = q.y;
}
struct alignas(4) HalfPair {
    __half a, b;
};
__device__ __forceinline__ void ld_pair(const __half *b, unsigned p, float &u, float &v) {
    HalfPair q = ldo((const HalfPair *)b, p * 2u);
    u = __half2float(q.a);
    v = __half2float(q.b);
}

template <typename TH, typename TP>
__device__ __forceinline__ void bloom_down_tile(const PostDesc &c, int tile, DownLds &sm) {
    typedef typename RawTexel<TP>::type TR;
    int tiles_x = (c.lw[1] + kDownTile - 1) / kDownTile;
    int by = tile / tiles_x, bx = tile - by * tiles_x;
    int t = threadIdx.x;
    const TH *hdr = (const TH *)c.hdr;
    unsigned plane = (unsigned)c.W * (unsigned)c.H;
    // level 1, one texel per thread: the bright map averaged over its in-range 2x2
    // children, summed as horizontal pairs and then the two rows (the order the
    // fused shading epilogue uses)
    int lx = t % kDownTile, ly = t / kDownTile;
    int X = bx * kDownTile + lx, Y = by * kDownTile + ly;
    float4 v = make_float4(0, 0, 0, 0);
    if (X < c.lw[1] && Y < c.lh[1]) {
        float R[4], G[4], B[4];
        bool in[4];
        if (!(c.W & 1)) {  // even width: a row's two children are one pair (six loads in flight)
#pragma unroll
            for (int r = 0; r < 2; ++r) {
                int py = 2 * Y + r;
                in[2 * r] = in[2 * r + 1] = py < c.H;
                unsigned p = in[2 * r] ? __umul24((unsigned)py, (unsigned)c.W) + (unsigned)(2 * X) : 0u;
                ld_pair(hdr, p, R[2 * r], R[2 * r + 1]);
                ld_pair(hdr, plane + p, G[2 * r], G[2 * r + 1]);
                ld_pair(hdr, 2 * plane + p, B[2 * r], B[2 * r + 1]);
            }
        } else {
#pragma unroll
            for (int k = 0; k < 4; ++k) {  // all twelve loads in flight together
                int px = 2 * X + (k & 1), py = 2 * Y + (k >> 1);
                in[k] = px < c.W && py < c.H;
                unsigned p = in[k] ? __umul24((unsigned)py, (unsigned)c.W) + (unsigned)px : 0u;
                R[k] = ldf(hdr, p);
                G[k] = ldf(hdr, plane + p);
                B[k] = ldf(hdr, 2 * plane + p);
            }
        }
        float cr[4], cg[4], cb[4];
#pragma unroll
        for (int k = 0; k < 4; ++k) {  // an out-of-image child adds an exact zero
            float sc = bright_scale(R[k], G[k], B[k], c.threshold);
            cr[k] = in[k] ? R[k] * sc : 0.0f;
            cg[k] = in[k] ? G[k] * sc : 0.0f;
            cb[k] = in[k] ? B[k] * sc : 0.0f;
        }
        float inv_n = (in[1] ? 0.5f : 1.0f) * (in[2] ? 0.5f : 1.0f);
        v = make_float4(((cr[0] + cr[1]) + (cr[2] + cr[3])) * inv_n, ((cg[0] + cg[1]) + (cg[2] + cg[3])) * inv_n,
                        ((cb[0] + cb[1]) + (cb[2] + cb[3])) * inv_n, 0.0f);
        TR st = pack<TR>(v);
        sto((TR *)c.raw[1], level_texel(c, 1, X, Y) * (unsigned)sizeof(TR), st);
        v = unpack(st);  // the next levels average what level 1 holds
    }
    sm.s1[ly][lx] = v;
    down_levels_2_to_5<TP>(c, bx, by, sm);
}

// Levels 2..5 when the shading pass has written level 1 (the fused form).
template <typename TP>
__device__ __forceinline__ void bloom_down_from1_tile(const PostDesc &c, int tile, DownLds &sm) {
    int tiles_x = (c.lw[1] + kDownTile - 1) / kDownTile;
    int by = tile / tiles_x, bx = tile - by * tiles_x;
    int t = threadIdx.x;
    int lx = t % kDownTile, ly = t / kDownTile;
    int X = bx * kDownTile + lx, Y = by * kDownTile + ly;
    float4 v = make_float4(0, 0, 0, 0);
    typedef typename RawTexel<TP>::type TR;
    if (X < c.lw[1] && Y < c.lh[1]) v = unpack(ldo((const TR *)c.raw[1], level_texel(c, 1, X, Y) * (unsigned)sizeof(TR)));
    sm.s1[ly][lx] = v;
    down_levels_2_to_5<TP>(c, bx, by, sm);
}

// ---------------------------------------------------------------------------
// bloom_blur: columns of one level by four wavefronts
// ---------------------------------------------------------------------------
__device__ __forceinline__ PackedRgb binomial5(PackedRgb a, PackedRgb b, PackedRgb m, PackedRgb d, PackedRgb e) {
    return PackedRgb{(a.x + e.x + 4.0f * (b.x + d.x) + 6.0f * m.x) * 0.0625f,
               (a.y + e.y + 4.0f * (b.y + d.y) + 6.0f * m.y) * 0.0625f,
               (a.z + e.z + 4.0f * (b.z + d.z) + 6.0f * m.z) * 0.0625f};
}

__device__ __forceinline__ PackedRgb lane_before(PackedRgb v) {
    return PackedRgb{lane_before(v.x), lane_before(v.y), lane_before(v.z)};
}
__device__ __forceinline__ PackedRgb lane_after(PackedRgb v) {
    return PackedRgb{lane_after(v.x), lane_after(v.y), lane_after(v.z)};
}

// An item is four wavefronts' tiles below each other, each of kRows rows.  A wavefront's lanes
// are kCols columns and two on each side for the halo: a lane holds its column of the footprint
// in registers, the horizontal sums take their neighbours from other lanes.  No LDS and no
// barriers, and all rows are in flight together.  Four rows in a single view (latency: 1920x1080
// in float32 6.4 us, with eight rows 6.6, 256x256 3.6 and 4.6), eight in a batch (a quarter instead
// of half of the rows read twice: 16 views of 13.2 Mpx in half storage 17.3 us against 19.4).  Tiles
// of 32 x 16 staged through LDS with both sums there: 7.8, 3.8 and 24.3 us.
template <int kCols, int kRows, typename TP>
__device__ __forceinline__ void bloom_blur_item(const PostDesc &c, int item) {
    static_assert(kCols <= 60, "and a halo of two on each side");
    typedef typename RawTexel<TP>::type TR;
    int L = 1;
    while (L < c.nl && item >= c.blk_start[L + 1]) ++L;
    int local = item - c.blk_start[L];
    int w = c.lw[L], h = c.lh[L];
    int tx = (w + kCols - 1) / kCols;
    int ty = local / tx;
    int lane = (int)threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
    int X = (local - ty * tx) * kCols - 2 + lane, Y0 = (ty * 4 + wave) * kRows;
    if (Y0 >= h) return;
    const TR *src = (const TR *)c.raw[L];
    unsigned col = (unsigned)min(max(X, 0), w - 1) * (unsigned)sizeof(TR);
    TR v[kRows + 4];
#pragma unroll
    for (int r = 0; r < kRows + 4; ++r)
        v[r] = ldo(src + (unsigned)min(max(Y0 + r - 2, 0), h - 1) * (unsigned)w, col);
    __builtin_amdgcn_sched_barrier(0);
    bool store = lane >= 2 && lane < 2 + kCols && X < w;
    PackedRgb s[kRows + 4];
#pragma unroll
    for (int r = 0; r < kRows + 4; ++r) {
        float4 f = unpack(v[r]);
        PackedRgb m{f.x, f.y, f.z}, b = lane_before(m), d = lane_after(m);
        s[r] = binomial5(lane_before(b), b, m, d, lane_after(d));
        if (r >= 4) {
            int j = r - 4;
            PackedRgb o = binomial5(s[j], s[j + 1], s[j + 2], s[j + 3], s[j + 4]);
            if (store && Y0 + j < h)
                sto((TP *)c.blur[L] + (unsigned)(Y0 + j) * (unsigned)w, (unsigned)X * (unsigned)sizeof(TP),
                    pack<TP>(make_float4(o.x, o.y, o.z, 0.0f)));
        }
        __builtin_amdgcn_sched_barrier(0);  // (a row at a time: few live registers)
    }
}

// ---------------------------------------------------------------------------
// composite + tone mapping: one 32x8 pixel tile
// ---------------------------------------------------------------------------
__device__ __forceinline__ float aces(float x) {
    return x * fmaf(2.51f, x, 0.03f) * rcp(fmaf(x, fmaf(2.43f, x, 0.59f), 0.14f));
}
// Reinhard's global operator on each channel (the paper's alternative curve).
__device__ __forceinline__ float reinhard(float x) { return x * rcp(1.0f + x); }
// x after exposure, tone curve, gamma and 8-bit rounding, as byte kByte of `word`.
// (y is in [0, 1], so g is, up to rounding; the conversion saturates, NaN gives 0, and
// its own rounding sees a whole number)
template <bool kReinhard, int kByte>
__device__ __forceinline__ uint32_t encode8(float x, float exposure, float inv_gamma, uint32_t word) {
    float e = exposure * x;
    float y = clamp01(kReinhard ? reinhard(e) : aces(e));
    float g = __builtin_amdgcn_exp2f(__builtin_amdgcn_logf(y) * inv_gamma);
    return __builtin_amdgcn_cvt_pk_u8_f32(floorf(fmaf(255.0f, g, 0.5f)), kByte, word);
}

// Level L samples pixel x at (x + 1/2) 2^-L - 1/2 = v / 2^(L+1) with v = 2x + 1 - 2^L:
// the texel is v >> (L+1) (an arithmetic shift floors) and the weight is the
// remainder (v & (2^(L+1) - 1)) / 2^(L+1), exact in float -- the same numbers as
// the float form, without floor or conversions.
//
// A thread owns one pixel column of an 8-row strip (the strip starts at a
// multiple of 8).  For each blurred level it first interpolates, at its column,
// the level rows under the strip (6, 4, 3, 2, 2 rows for levels 1..5: two texel
// loads per row, neighbouring lanes share cache lines), then every pixel of
// the column interpolates between two of those rows.  Because the strip starts
// at a multiple of 8, which rows a pixel uses is fixed at compile time (levels
// 1..3), or is the first pair for all eight pixels (levels 4 and 5, where the
// strip lies inside one texel row pair and the remainder grows by 2 per pixel
// without wrapping); the weights of levels 1..3 are compile-time constants as
// well.  Everything stays in registers: no LDS, no barriers, and the strip's
// 24 HDR loads are in flight with the pyramid's.  Rows are scalar addresses
// and bytes are packed by their conversion, since vector issue bounds the batched
// composite (81 % busy, half storage): 16 views of 13.2 Mpx 57 -> 52.5 us, and
// bloom and tone mapping of 3840x2160 in half storage 63.8 -> 61.8 us, against
// per-lane addresses, clamps of the 8-bit value and halves unpacked before the
// difference.  1920x1080 in float32 (11.2 us, 45 MB) is bound by memory latency.
// (SR: the rows of the strip that a wavefront takes, all or a half.)
template <int J0, int NJ>
struct StripRows {
    static constexpr int j0 = J0, n = NJ;
};
typedef StripRows<0, kPostTy> WholeStrip;
template <int L, typename SR = WholeStrip>
struct LevelRows {
    static constexpr int sh = L + 1, o = 1 - (1 << L), m = (1 << sh) - 1;
    static constexpr float inv = 1.0f / (float)(1 << sh);
    // first row (relative to the strip's first footprint row) of pixel j
    static constexpr int rel(int j) { return L <= 3 ? ((2 * j + o) >> sh) - (o >> sh) : 0; }
    static constexpr int first = rel(SR::j0), n = rel(SR::j0 + SR::n - 1) + 2 - first;
    // weight of pixel j (levels 1..3)
    static constexpr float wy(int j) { return (float)((2 * j + o) & m) * inv; }
};

// b - a of two pyramid texels.  From half storage a mixed-precision FMA takes the
// halves as they are: b * 1 - a, rounded once like the float32 difference.
__device__ __forceinline__ float4 texel_difference(float4 b, float4 a) {
    return make_float4(b.x - a.x, b.y - a.y, b.z - a.z, 0.0f);
}
__device__ __forceinline__ float4 texel_difference(Half4 b, Half4 a) {
    uint2 u, v;
    __builtin_memcpy(&u, &b, 8);
    __builtin_memcpy(&v, &a, 8);
    float4 d = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
    asm("v_fma_mix_f32 %0, %1, 1.0, -%2 op_sel_hi:[1,0,1]" : "=v"(d.x) : "v"(u.x), "v"(v.x));
    asm("v_fma_mix_f32 %0, %1, 1.0, -%2 op_sel:[1,0,1] op_sel_hi:[1,0,1]" : "=v"(d.y) : "v"(u.x), "v"(v.x));
    asm("v_fma_mix_f32 %0, %1, 1.0, -%2 op_sel_hi:[1,0,1]" : "=v"(d.z) : "v"(u.y), "v"(v.y));
    return d;
}

// The level-L texels beside the thread's column on the rows under the strip, and
// the column's weight.
template <int L, typename SR, typename TP>
struct LevelTexels {
    TP a[LevelRows<L, SR>::n], b[LevelRows<L, SR>::n];
    float wx;
};
template <int L, typename SR, typename TP>
__device__ __forceinline__ void load_level(const PostDesc &c, int x, int Y0, LevelTexels<L, SR, TP> &t) {
    using LR = LevelRows<L, SR>;
    const int w = c.lw[L], h = c.lh[L];
    const TP *lvl = (const TP *)c.blur[L];
    int vx = 2 * x + LR::o;
    t.wx = (float)(vx & LR::m) * LR::inv;
    int cx = vx >> LR::sh;
    unsigned c0 = (unsigned)min(max(cx, 0), w - 1), c1 = (unsigned)min(max(cx + 1, 0), w - 1);
    unsigned o0 = c0 * (unsigned)sizeof(TP), o1 = c1 * (unsigned)sizeof(TP);
    int ay = ((2 * Y0 + LR::o) >> LR::sh) + LR::first;
#pragma unroll
    for (int r = 0; r < LR::n; ++r) {
        const TP *row = lvl + (unsigned)min(max(ay + r, 0), h - 1) * (unsigned)w;  // uniform: scalar arithmetic
        t.a[r] = ldo(row, o0);
        t.b[r] = ldo(row, o1);
    }
}

// Their values interpolated at the thread's column.
template <int L, typename SR, typename TP>
__device__ __forceinline__ void level_rows(const LevelTexels<L, SR, TP> &t, float (&rows)[LevelRows<L, SR>::n][3]) {
#pragma unroll
    for (int r = 0; r < LevelRows<L, SR>::n; ++r) {
        float4 a = unpack(t.a[r]), d = texel_difference(t.b[r], t.a[r]);
        rows[r][0] = fmaf(t.wx, d.x, a.x);
        rows[r][1] = fmaf(t.wx, d.y, a.y);
        rows[r][2] = fmaf(t.wx, d.z, a.z);
    }
}

// Levels 4 and 5, which start the strip's sums: each pixel of the strip adds
// a_L + w_L(j) (b_L - a_L) for the one row pair (a_L, b_L) under the strip, with
// w_L(j) = w_L(0) + 2 j / 2^(L+1); the two a_L are summed once per thread and
// enter as the first addend, so a pixel spends one FMA per level and channel.
// Absent levels contribute nothing (their difference and weight are 0).
template <typename SR, typename TP>
__device__ __forceinline__ void init_coarse(const PostDesc &c, int Y0, const LevelTexels<4, SR, TP> &t4,
                                            const LevelTexels<5, SR, TP> &t5, float (&acc)[SR::n][3]) {
    float base[3] = {0.0f, 0.0f, 0.0f}, d4[3] = {0.0f, 0.0f, 0.0f}, d5[3] = {0.0f, 0.0f, 0.0f};
    float w4 = 0.0f, w5 = 0.0f;
    if (c.nl >= 4) {
        float rows[2][3];
        level_rows<4, SR, TP>(t4, rows);
#pragma unroll
        for (int ch = 0; ch < 3; ++ch) {
            base[ch] = rows[0][ch];
            d4[ch] = rows[1][ch] - rows[0][ch];
        }
        w4 = (float)((2 * Y0 + LevelRows<4>::o) & LevelRows<4>::m) * LevelRows<4>::inv;
    }
    if (c.nl >= 5) {
        float rows[2][3];
        level_rows<5, SR, TP>(t5, rows);
#pragma unroll
        for (int ch = 0; ch < 3; ++ch) {
            base[ch] += rows[0][ch];
            d5[ch] = rows[1][ch] - rows[0][ch];
        }
        w5 = (float)((2 * Y0 + LevelRows<5>::o) & LevelRows<5>::m) * LevelRows<5>::inv;
    }
#pragma unroll
    for (int j = 0; j < SR::n; ++j) {
        float wj4 = w4 + (float)(2 * (SR::j0 + j)) * LevelRows<4>::inv, wj5 = w5 + (float)(2 * (SR::j0 + j)) * LevelRows<5>::inv;
#pragma unroll
        for (int ch = 0; ch < 3; ++ch) acc[j][ch] = fmaf(wj5, d5[ch], fmaf(wj4, d4[ch], base[ch]));
    }
}

// Levels 1..3: (1 - w) a + w b for the pixel's row pair, two FMAs per channel.
template <int L, typename SR, typename TP>
__device__ __forceinline__ void add_fine(const LevelTexels<L, SR, TP> &t, float (&acc)[SR::n][3]) {
    using LR = LevelRows<L, SR>;
    float rows[LR::n][3];
    level_rows<L, SR, TP>(t, rows);
#pragma unroll
    for (int j = 0; j < SR::n; ++j) {
        const int r0 = LR::rel(SR::j0 + j) - LR::first;
        const float w = LR::wy(SR::j0 + j);
#pragma unroll
        for (int ch = 0; ch < 3; ++ch) acc[j][ch] = fmaf(w, rows[r0 + 1][ch], fmaf(1.0f - w, rows[r0][ch], acc[j][ch]));
    }
}

// Bloom added to the strip's HDR, tone mapped and stored as RGBA8.
template <bool kReinhard, int NJ>
__device__ __forceinline__ void store_strip(const PostDesc &c, int x, int Y0, const float (&px)[NJ][3],
                                            const float (&acc)[NJ][3]) {
#pragma unroll
    for (int j = 0; j < NJ; ++j) {
        if (Y0 + j >= c.H) break;
        float R = fmaf(c.strength, acc[j][0], px[j][0]);
        float G = fmaf(c.strength, acc[j][1], px[j][1]);
        float Bc = fmaf(c.strength, acc[j][2], px[j][2]);
        uint32_t word = encode8<kReinhard, 0>(R, c.exposure, c.inv_gamma, 255u << 24);
        word = encode8<kReinhard, 1>(G, c.exposure, c.inv_gamma, word);
        word = encode8<kReinhard, 2>(Bc, c.exposure, c.inv_gamma, word);
        sto(c.ldr + (unsigned)(Y0 + j) * (unsigned)c.W, (unsigned)x * 4u, word);
    }
}

// The rows SR of one 64 x 8 tile by one wavefront; `lane` is the thread's lane (its column).
template <bool kOneTrip, typename SR, typename TH, typename TP>
__device__ __forceinline__ void composite_tile(const PostDesc &c, int tile, int lane) {
    tile = __builtin_amdgcn_readfirstlane(tile);  // one per wavefront: rows are scalar addresses
    int tiles_x = (c.W + kPostTx - 1) / kPostTx;
    int ty = tile / tiles_x;
    int x = (tile - ty * tiles_x) * kPostTx + lane, Y0 = ty * kPostTy;
    const int Y1 = Y0 + SR::j0;  // the first row of the part
    if (x >= c.W || Y1 >= c.H) return;
    unsigned plane = (unsigned)c.W * (unsigned)c.H;
    const TH *hdr = (const TH *)c.hdr;
    // the strip's HDR first (in flight while the pyramid is read); rows below the image are
    // clamped to the last row and not stored
    float px[SR::n][3];
#pragma unroll
    for (int j = 0; j < SR::n; ++j) {
        const TH *row = hdr + (unsigned)min(Y1 + j, c.H - 1) * (unsigned)c.W;
        px[j][0] = ldf(row, (unsigned)x);
        px[j][1] = ldf(row + plane, (unsigned)x);
        px[j][2] = ldf(row + 2 * (size_t)plane, (unsigned)x);
    }
    // the bloom sum of levels 5, 4 (one row pair for the whole strip), then 1 .. 3
    // (nl is uniform).  The texels come in as few round trips as the registers hold:
    // half texels all with the HDR (111 registers), float texels as {5, 4, 1} with it and
    // {2, 3} (107; the scheduler would otherwise interleave loads and uses).  Four waves
    // per SIMD are about what 1920x1080 has to give.  One trip per level: bloom and tone
    // mapping of 1920x1080 float 26.8 us against 26.3, of 3840x2160 half 61.8 against
    // 58.9; float texels in one trip need 140 registers (26.7);
    // float figures with unblurred levels of four floats.
    float acc[SR::n][3];
    LevelTexels<4, SR, TP> t4;
    LevelTexels<5, SR, TP> t5;
    LevelTexels<1, SR, TP> t1;
    LevelTexels<2, SR, TP> t2;
    LevelTexels<3, SR, TP> t3;
    if (c.nl >= 5) load_level<5, SR, TP>(c, x, Y0, t5);
    if (c.nl >= 4) load_level<4, SR, TP>(c, x, Y0, t4);
    if (c.nl >= 1) load_level<1, SR, TP>(c, x, Y0, t1);
    if (kOneTrip) {
        if (c.nl >= 2) load_level<2, SR, TP>(c, x, Y0, t2);
        if (c.nl >= 3) load_level<3, SR, TP>(c, x, Y0, t3);
    }
    __builtin_amdgcn_sched_barrier(0);
    init_coarse<SR, TP>(c, Y0, t4, t5, acc);
    if (c.nl >= 1) add_fine<1, SR, TP>(t1, acc);
    if (!kOneTrip) {
        if (c.nl >= 2) load_level<2, SR, TP>(c, x, Y0, t2);
        if (c.nl >= 3) load_level<3, SR, TP>(c, x, Y0, t3);
        __builtin_amdgcn_sched_barrier(0);
    }
    if (c.nl >= 2) add_fine<2, SR, TP>(t2, acc);
    if (c.nl >= 3) add_fine<3, SR, TP>(t3, acc);
    if (c.tonemap == EPB_TONEMAP_REINHARD) store_strip<true, SR::n>(c, x, Y1, px, acc);
    else store_strip<false, SR::n>(c, x, Y1, px, acc);
}

}  // namespace epb
