// Image-based-lighting precompute (paper Sec. 3.1): a solid-angle-weighted
// average of the environment, the diffuse irradiance map, the split-sum
// prefiltered specular chain and the environment BRDF table.
//
// gfx950 mapping:
//  * irradiance: 6*32^2 outputs x 6*64^2 source texels.  One thread per
//    output, source texels by scalar loads, those behind a wavefront's horizon
//    left out; the source range is split across workgroups so that the
//    grid gives every CU about four, and the per-split Kahan partials are combined in
//    a fixed order by a second kernel (deterministic, no atomics).
//  * a GGX sample's tangent-frame half vector depends on the sample and the
//    roughness only, and its square roots, reciprocal and sine/cosine are most
//    of a sample's instructions, so it is made once per level (prefilter) or
//    per table row (BRDF table) and only turned into each texel's frame.
//  * prefilter from the full-resolution environment: one wavefront per output
//    texel, the 64 lanes split the samples, whose taps then stay within the
//    texel's GGX lobe (a few cache lines at the rough levels' narrow lobes);
//    per-lane Kahan sums, compensated wave reduction through cross-lane
//    shuffles; a lane takes two samples at a time (both lookups' taps in
//    flight), their half vectors from the level's table one iteration ahead,
//    the taps, where lookups are many, from a copy of the environment that holds
//    vertical pairs of RGB texels (the texture data path bounds this kernel: fewer
//    loads and lines per lookup).
//  * prefilter with filtered importance sampling (taps on the mip level that
//    matches each sample's footprint): one wavefront per 8x8 tile of output
//    texels and chunk of the samples; all lanes take the same sample at once,
//    so its half vector is a uniform (scalar) table load and neighbouring
//    texels' taps share cache lines; per-lane Kahan sums per chunk, the chunks
//    added in a fixed order by a second kernel (deterministic, no atomics).
//  * BRDF table: one wavefront per entry, the 64 lanes split the Hammersley
//    samples (per-lane Kahan sums, compensated wave reduction through
//    cross-lane shuffles); a block makes its row's half vectors into LDS, and
//    a lane Kahan-adds its (non-negative) terms four at a time.
//  * roughness-0 prefilter level: every GGX half vector equals the normal, so
//    the N.L-weighted mean is the environment along the texel direction; one
//    bilinear lookup per texel.
#include <cmath>

#include "device_common.hpp"
#include "launch.hpp"

namespace epb {

// Solid angle of texel (i, j) of a face of size S.  The texel is a planar
// quadrilateral at unit distance whose edges project to great circles; split
// along its diagonal into two spherical triangles, each is evaluated with the
// Van Oosterom-Strackee formula tan(W / 2) = |a.(b x c)| / (|a||b||c| +
// (a.b)|c| + (a.c)|b| + (b.c)|a|).  For corners (x0,y0,1), (x1,y0,1),
// (x1,y1,1), (x0,y1,1) the triple products are exactly dx dy and the
// denominators are sums of positive terms, so no cancellation occurs even for
// texels of 1e-5 sr.
__device__ float texel_solid_angle(int i, int j, int S) {
    float inv = 1.0f / (float)S;
    float x0 = (float)(2 * i - S) * inv, x1 = (float)(2 * i + 2 - S) * inv;
    float y0 = (float)(2 * j - S) * inv, y1 = (float)(2 * j + 2 - S) * inv;
    float num = (x1 - x0) * (y1 - y0);
    v3 a = mk3(x0, y0, 1.0f), b = mk3(x1, y0, 1.0f), c = mk3(x1, y1, 1.0f), d = mk3(x0, y1, 1.0f);
    float la = sqrtf(dot(a, a)), lb = sqrtf(dot(b, b)), lc = sqrtf(dot(c, c)), ld_ = sqrtf(dot(d, d));
    float den1 = la * lb * lc + dot(a, b) * lc + dot(a, c) * lb + dot(b, c) * la;
    float den2 = la * lc * ld_ + dot(a, c) * ld_ + dot(a, d) * lc + dot(c, d) * la;
    return 2.0f * (atan2f(num, den1) + atan2f(num, den2));
}

// Compensated sum over aligned segments of `width` lanes (a power of two <= 64):
// Knuth two-sums down a butterfly, the rounding errors carried beside.
__device__ __forceinline__ float segment_sum_compensated(float v, int width) {
    float comp = 0.0f;
    for (int off = width >> 1; off >= 1; off >>= 1) {
        float o = __shfl_xor(v, off, 64);
        float oc = __shfl_xor(comp, off, 64);
        float s, e;
        two_sum(v, o, s, e);
        v = s;
        comp = comp + oc + e;
    }
    return v + comp;
}

// Irradiance source: texel (f, i, j) of size Ss is the solid-angle-weighted mean
// of the k x k environment texels it covers (k = S / Ss).  Because solid angles
// add, this equals repeated 2x2 weighted halving.  Also writes the source
// table entry (unit direction, solid angle at size Ss).
// A segment of lpt lanes (the k x k block rounded up to a power of two, at most
// 64) per texel (i, j), for all six faces or for one (see kSourceThreads).  Each lane
// sums its share of the block with Kahan, the segment adds the lanes' sums
// compensated.  lpt is uniform.
// All six faces share their solid angles, most of the work (6x512^2 to 64^2: 31 us with a
// segment per face); but up to this many threads a face (a wavefront on a quarter of the SIMDs) the segments are few
// and long, and those of one face are shorter (whole precompute with six faces / one: 6x512^2 to
// 4^2 200 / 147 us, to 16^2 41.9 / 34.7; 6x256^2 to 2^2 198 / 144; 6x128^2 to 8^2 28.6 / 20.5).
constexpr int kSourceThreads = 16384;
template <int kFaces>
__device__ __forceinline__ void ibl_source_block(int block, const float4 *__restrict__ env, int S, int Ss, int lpt,
                                                 float4 *__restrict__ src, float4 *__restrict__ tab) {
    int nface = Ss * Ss, per = (nface * lpt + 255) / 256;  // blocks of one group of faces
    int f0 = kFaces < 6 ? block / per * kFaces : 0;
    int t = (kFaces < 6 ? block % per : block) * 256 + (int)threadIdx.x;
    int o = t / lpt, sub = t - o * lpt;
    // (the segment stays together: nface * lpt threads fill whole segments)
    bool live = o < nface;
    int oc = live ? o : nface - 1;
    int j = oc / Ss, i = oc - j * Ss;
    int k = S / Ss;
    Kahan w{0, 0};
    Kahan c[kFaces][3] = {};
    for (int q = sub; q < k * k; q += lpt) {
        int bj = q / k, bi = q - bj * k;
        int ci = i * k + bi, cj = j * k + bj;
        float4 L[kFaces];
#pragma unroll
        for (int f = 0; f < kFaces; ++f) L[f] = env[(size_t)(f0 + f) * S * S + (size_t)cj * S + ci];
        float dw = k == 1 ? 1.0f : texel_solid_angle(ci, cj, S);
#pragma unroll
        for (int f = 0; f < kFaces; ++f) {
            kahan_add(c[f][0], L[f].x * dw);
            kahan_add(c[f][1], L[f].y * dw);
            kahan_add(c[f][2], L[f].z * dw);
        }
        kahan_add(w, dw);
    }
    float iw = 1.0f / segment_sum_compensated(kahan_value(w), lpt);
    float dw = texel_solid_angle(i, j, Ss);
#pragma unroll
    for (int f = 0; f < kFaces; ++f) {
        float R = segment_sum_compensated(kahan_value(c[f][0]), lpt);
        float G = segment_sum_compensated(kahan_value(c[f][1]), lpt);
        float Bv = segment_sum_compensated(kahan_value(c[f][2]), lpt);
        if (live && sub == 0) {
            src[(f0 + f) * nface + o] = make_float4(R * iw, G * iw, Bv * iw, 0.0f);
            v3 d = normalize(cube_texel_dir(f0 + f, i, j, Ss));
            tab[(f0 + f) * nface + o] = make_float4(d.x, d.y, d.z, dw);
        }
    }
}

// The value that lane k holds, in every lane.
__device__ __forceinline__ float lane_value(float v, int k) {
    return __builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, v), k));
}

// Four texels by one scalar load.
typedef float Float16 __attribute__((ext_vector_type(16), aligned(16)));
typedef __attribute__((address_space(4))) const Float16 ConstFloat16;
constexpr int kWaitScalar = 0xC07F;  // s_waitcnt: scalar loads and LDS only

// Output o of the irradiance map for thread t of its launch: a wavefront takes an 8 x 8 tile of
// a face where those fit (a narrow cone of normals, see below), 64 outputs in a row otherwise.
__device__ __forceinline__ int irradiance_output(int t, int irr) {
    if (irr & 7) return t;
    int across = irr >> 3, lane = t & 63, tile = t >> 6;
    int f = tile / (across * across), r = tile - f * across * across;
    int ty = r / across, tx = r - ty * across;
    return (f * irr + ty * 8 + (lane >> 3)) * irr + tx * 8 + (lane & 7);
}

// Partial irradiance sums over source chunk `chunk` for 256 outputs.  A group of four
// source texels behind the horizon of every output of a wavefront adds exact zeros (to a
// Kahan sum too) and is left out: each lane tests one group of 64 against the cone around
// the wavefront's normals.  That is about a quarter of the groups for 16 x 16 outputs a
// face and a third for 32 x 32.  The groups are the same for every lane and come by scalar
// loads, the next one's in flight while one is added; vector issue bounds the sums.  With
// every group, staged through LDS: whole precompute of 6x512^2 with 256 filtered samples
// 130 us against 110, of 6x64^2 39.6 against 38.5 (16 x 16 outputs).
// part layout: [chunk][output][8] = Kahan (s, c) of R, G, B, weight.
__device__ __forceinline__ void irradiance_partial_block(int block, int chunk, const float4 *__restrict__ src,
                                                         const float4 *__restrict__ tab, int nsrc, int chunk_len,
                                                         int irr, float *__restrict__ part) {
    int nout = 6 * irr * irr;
    int t = block * 256 + (int)threadIdx.x, lane = threadIdx.x & 63;
    int o = irradiance_output(min(t, nout - 1), irr);
    int f = o / (irr * irr), j = (o / irr) % irr, i = o % irr;
    v3 n = normalize(cube_texel_dir(f, i, j, irr));
    // The cone around a tile's normals: the axis through the tile's centre, the half angle h
    // that of its farthest corner.  A direction d with axis . d below -sin h has n . d < 0 for all
    // of them (by far more than rounding, with 1e-4 to spare).
    float horizon = -2.0f;
    v3 axis = n;
    if (!(irr & 7)) {
        auto corner = [&](int k) { return mk3(lane_value(n.x, k), lane_value(n.y, k), lane_value(n.z, k)); };
        v3 c0 = corner(0), c1 = corner(7), c2 = corner(56), c3 = corner(63);
        axis = normalize((c0 + c1) + (c2 + c3));
        float ch = fminf(fminf(dot(c0, axis), dot(c1, axis)), fminf(dot(c2, axis), dot(c3, axis)));
        if (ch > 0.1f) horizon = -sqrtf(fmaxf(0.0f, 1.0f - ch * ch)) - 1e-4f;
    }
    Kahan r{0, 0}, g{0, 0}, b{0, 0}, w{0, 0};
    int beg = min(chunk * chunk_len, nsrc), cnt = min(chunk_len, nsrc - beg), whole = cnt & ~3;  // (0: past the end)
    src += beg;
    tab += beg;
    const ConstFloat16 *gs = (const ConstFloat16 *)as_constant((const float *)src);
    const ConstFloat16 *gt = (const ConstFloat16 *)as_constant((const float *)tab);
    // Every term is >= 0, so a group of four summed in plain float and then
    // Kahan-added keeps the whole sum within about 3 units of rounding of
    // its value (each group's error is bounded by its own terms), as with
    // a Kahan add per term, at a quarter of the compensation work.
    auto add = [&](const Float16 &l, const Float16 &T) {
        float c[4];
#pragma unroll
        for (int u = 0; u < 4; ++u)
            c[u] = fmaxf(0.0f, fmaf(n.x, T[4 * u], fmaf(n.y, T[4 * u + 1], n.z * T[4 * u + 2]))) * T[4 * u + 3];
        kahan_add(r, fmaf(l[12], c[3], fmaf(l[8], c[2], fmaf(l[4], c[1], l[0] * c[0]))));
        kahan_add(g, fmaf(l[13], c[3], fmaf(l[9], c[2], fmaf(l[5], c[1], l[1] * c[0]))));
        kahan_add(b, fmaf(l[14], c[3], fmaf(l[10], c[2], fmaf(l[6], c[1], l[2] * c[0]))));
        kahan_add(w, ((c[0] + c[1]) + c[2]) + c[3]);
    };
    for (int base = 0; base < whole; base += 256) {
        int first = base + 4 * lane;
        bool need = false;
        if (first < whole) {
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                float4 T = tab[first + u], L = src[first + u];
                // (a texel that is no finite number reaches every output)
                need |= !(dot(axis, mk3(T.x, T.y, T.z)) < horizon) || !(fabsf(L.x + L.y + L.z) < __builtin_inff());
            }
        }
        unsigned long long todo = __ballot(need);
        if (!todo) continue;
        // the next group's scalar loads are in flight while one is added (at the end the last
        // group's again)
        int q = 0;
        auto next = [&] {
            if (todo) q = (base >> 2) + __builtin_ctzll(todo);
            todo &= todo - 1;
        };
        int count = __builtin_popcountll(todo);
        next();
        Float16 l0 = gs[q], t0 = gt[q], l1, t1;
        __builtin_amdgcn_s_waitcnt(kWaitScalar);
        for (int pairs = count >> 1; pairs; --pairs) {
            next();
            l1 = gs[q];
            t1 = gt[q];
            __builtin_amdgcn_sched_barrier(0);
            add(l0, t0);
            __builtin_amdgcn_sched_barrier(0);
            __builtin_amdgcn_s_waitcnt(kWaitScalar);
            next();
            l0 = gs[q];
            t0 = gt[q];
            __builtin_amdgcn_sched_barrier(0);
            add(l1, t1);
            __builtin_amdgcn_sched_barrier(0);
            __builtin_amdgcn_s_waitcnt(kWaitScalar);
        }
        if (count & 1) add(l0, t0);
    }
    for (int q = whole; q < cnt; ++q) {
        float4 T = tab[q], L = src[q];
        float c = fmaxf(0.0f, fmaf(n.x, T.x, fmaf(n.y, T.y, n.z * T.z))) * T.w;
        kahan_add(r, L.x * c);
        kahan_add(g, L.y * c);
        kahan_add(b, L.z * c);
        kahan_add(w, c);
    }
    if (t < nout) {
        float *p = part + ((size_t)chunk * nout + o) * 8;
        p[0] = r.s; p[1] = g.s; p[2] = b.s; p[3] = w.s;
        p[4] = r.c; p[5] = g.c; p[6] = b.c; p[7] = w.c;
    }
}

// Sums of the chunks' partials, one lane per component of an output (four lanes
// side by side: their serial compensated adds run beside each other).
__device__ __forceinline__ void irradiance_final_block(int block, const float *__restrict__ part, int chunks, int nout,
                                                       float4 *__restrict__ out) {
    int t = block * 256 + (int)threadIdx.x;
    int o = t >> 2, q = t & 3;
    bool live = o < nout;
    Kahan acc{0, 0};
    const float *p = part + (size_t)(live ? o : 0) * 8 + q;
    // (unrolled: several chunks' loads in flight ahead of the serial adds)
#pragma unroll 8
    for (int c = 0; c < chunks; ++c) {
        float v = p[(size_t)c * nout * 8], e = p[(size_t)c * nout * 8 + 4];
        kahan_add(acc, v);
        kahan_add(acc, -e);
    }
    float v = kahan_value(acc);
    float iw = 1.0f / __shfl(v, (int)(threadIdx.x & 63) | 3, 64);  // the weight's lane
    if (live) ((float *)out)[(size_t)o * 4 + q] = q < 3 ? v * iw : 0.0f;
}

// Roughness-0 level: the environment along each texel direction.
__device__ __forceinline__ void prefilter_mirror_block(int block, const float4 *__restrict__ env, int S, int sm,
                                                       float4 *__restrict__ out) {
    int o = block * 256 + (int)threadIdx.x;
    if (o >= 6 * sm * sm) return;
    int f = o / (sm * sm), j = (o / sm) % sm, i = o % sm;
    v3 n = normalize(cube_texel_dir(f, i, j, sm));
    out[o] = cube_bilinear(env, face_dims(S), n);
}

// Environment mip chain for filtered importance sampling: levels 1 .. last of one
// buffer (level 0 is the environment itself), level k (faces S >> k, S a power of
// two) at texel 2 S^2 - 8 (S >> k)^2 = 6 ((S/2)^2 + ... + (S >> (k-1))^2).
__host__ __device__ inline unsigned chain_offset_pow2(int S, int k) {
    unsigned s = (unsigned)S, sk = (unsigned)(S >> k);
    return 2u * s * s - 8u * sk * sk;
}

// The solid-angle-weighted mean of the 2x2 children L of texel (i, j) of a level
// whose parent level has faces of size Sp, as the irradiance source is built.
__device__ __forceinline__ float4 mean_of_children(const float4 (&L)[4], const float (&dw)[4]) {
    float r = 0.0f, g = 0.0f, b = 0.0f, w = 0.0f;
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        r = fmaf(L[q].x, dw[q], r);
        g = fmaf(L[q].y, dw[q], g);
        b = fmaf(L[q].z, dw[q], b);
        w += dw[q];
    }
    float iw = 1.0f / w;
    return make_float4(r * iw, g * iw, b * iw, 0.0f);
}

// Up to five chain levels in one launch: a block takes the 32 x 32 texels (or the
// whole face) at its place of level `first` of `faces` faces (all six, or one, see
// chain_faces) and writes what it covers of the levels below it, each from the one
// before in LDS.  The solid angles of all its levels, which do not depend on the
// face, are made first, side by side (level after level they are a serial chain: 17 us
// for the preparing launch of a 6x64^2 cube).
constexpr int kChainStep = 5;
// Faces a block takes where the chain starts from faces of size S (the later steps start from
// 128 at most, and take one): one while that gives few blocks, which the six faces' loads and
// the solid angles then bound (preparing launch of a 6x64^2 cube 11.9 us with six, 8.5 with one;
// 6x256^2 12.2 / 11.7); six where the solid angles are much of the work (6x512^2 26 / 34 us).
__host__ __device__ inline int chain_faces(int S) { return S > 256 ? 6 : 1; }
struct ChainLds {
    float4 a[6 * 16 * 16], b[6 * 8 * 8];
    float dw[32 * 32 + 16 * 16 + 8 * 8 + 4 * 4 + 2 * 2];
};
__device__ __forceinline__ void env_chain_block(int block, const float4 *__restrict__ env, float4 *__restrict__ chain,
                                                int S, int first, int last, int faces, ChainLds &sm) {
    int Sp = S >> first;
    const float4 *src = first == 0 ? env : chain + chain_offset_pow2(S, first);
    int side = min(Sp, 32);  // a power of two
    int across = Sp / side;
    int group = block / (across * across), place = block - group * across * across;
    int by = place / across, bx = place - by * across;
    int f0 = group * faces;
    int t = (int)threadIdx.x;
    int levels = min(kChainStep, last - first);
    int n = side >> 1;  // the first level's texels, at most one per thread
    int ly = t / n, lx = t - ly * n;
    bool live = t < n * n;
    float *dws = sm.dw;  // of the level that the children are on
    for (int r = 0, at = 0; r < levels; ++r) {
        int w = side >> r;
        for (int q = t; q < w * w; q += 256) {
            int y = q / w;
            dws[at + q] = texel_solid_angle(bx * w + (q - y * w), by * w + y, Sp >> r);
        }
        at += w * w;
    }
    __syncthreads();
    if (live) {
        int i = bx * n + lx, j = by * n + ly;
        float4 *out = chain + chain_offset_pow2(S, first + 1);
        float dw[4];
#pragma unroll
        for (int c = 0; c < 4; ++c) dw[c] = dws[(2 * ly + (c >> 1)) * 2 * n + 2 * lx + (c & 1)];
        for (int e = 0; e < faces; ++e) {
            int f = f0 + e;
            float4 L[4];
#pragma unroll
            for (int c = 0; c < 4; ++c) L[c] = src[((size_t)f * Sp + 2 * j + (c >> 1)) * Sp + 2 * i + (c & 1)];
            float4 v = mean_of_children(L, dw);
            out[((size_t)f * (Sp >> 1) + j) * (Sp >> 1) + i] = v;
            sm.a[(e * n + ly) * n + lx] = v;
        }
    }
    __syncthreads();
    float4 *from = sm.a, *to = sm.b;
    for (int k = first + 2; k <= first + levels; ++k) {
        dws += 4 * n * n;
        n >>= 1;  // this block's n x n texels of level k
        int Sd = S >> k;
        float4 *out = chain + chain_offset_pow2(S, k);
        for (int q = t; q < n * n * faces; q += 256) {
            int e = q / (n * n), r = q - e * n * n;
            int y = r / n, x = r - y * n;
            float dw[4];
            float4 L[4];
#pragma unroll
            for (int c = 0; c < 4; ++c) {
                dw[c] = dws[(2 * y + (c >> 1)) * 2 * n + 2 * x + (c & 1)];
                L[c] = from[(e * 2 * n + 2 * y + (c >> 1)) * 2 * n + 2 * x + (c & 1)];
            }
            float4 v = mean_of_children(L, dw);
            out[((size_t)(f0 + e) * Sd + by * n + y) * Sd + bx * n + x] = v;
            to[(e * n + y) * n + x] = v;
        }
        __syncthreads();
        // (the next level's texels fit the other array: a quarter of them; it is read no more)
        float4 *swap = from;
        from = to;
        to = swap;
    }
}

// Level 0 of the environment for the prefilter, whose taps use only the colour: each
// texel holds its own RGB and that of the texel below it (24 bytes; the last row
// repeats itself and is never a lookup's upper row), so that the 2x2 texels of a
// lookup are 48 bytes in one piece: three loads and mostly one cache line, where
// rows of packed RGB took four loads and two lines (6x512^2 precompute: 407 us).
// Not where lookups are few: with up to half a lookup a texel of the environment the copy costs
// more than it saves, and with up to 32 samples a wavefront's lanes are half idle and wait for
// no unit (whole precompute, with pairs / without: 6x4096^2, 128^2 in five levels, 1024 samples
// 1825 / 1496 us, 0.33 lookups; 512^2 in five, 128 samples 2633 / 2809, 0.66; 32^2 in three, 16
// samples 1067 / 301; 6x1024^2, 512^2 in five, 16 samples 414 / 374, 48 samples 452 / 498).
struct Rgb {
    float r, g, b;
};
struct RgbPair {
    Rgb top, bottom;
};
__device__ __forceinline__ void env_rgb_block(int block, const float4 *__restrict__ env, int S,
                                              RgbPair *__restrict__ dst) {
    int o = block * 256 + (int)threadIdx.x;
    if (o >= 6 * S * S) return;
    float4 t = env[o], u = env[o / S % S + 1 < S ? o + S : o];
    sto(dst, (unsigned)o * 24u, RgbPair{Rgb{t.x, t.y, t.z}, Rgb{u.x, u.y, u.z}});
}

// face_bilinear over the environment's texels or these pairs, split into its loads and its
// interpolation (so that several lookups' loads can be in flight): the same coordinates, taps
// and interpolation, so the same values.
struct TapPlace {
    unsigned idx;  // upper left texel
    float wx, wy;
};
__device__ __forceinline__ TapPlace tap_place(const FaceDims &g, FaceST f) {
    float x = clamp_to(fmaf(f.s, g.half, g.off), g.hi);
    float y = clamp_to(fmaf(f.t, g.half, g.off), g.hi);
    float x0f = clamp_to(floorf(x), g.hi1), y0f = clamp_to(floorf(y), g.hi1);
    return TapPlace{__umul24((unsigned)fmaf(f.face, (float)g.S, y0f), (unsigned)g.S) + (unsigned)x0f, x - x0f, y - y0f};
}
struct TexelTaps {
    float4 a, b, c, d;
    float wx, wy;
};
__device__ __forceinline__ TexelTaps env_taps(const float4 *__restrict__ lvl, const FaceDims &g, FaceST f) {
    TapPlace t = tap_place(g, f);
    unsigned o0 = t.idx * 16u, o1 = o0 + (unsigned)g.S * 16u;
    return TexelTaps{ldo(lvl, o0), ldo(lvl + 1, o0), ldo(lvl, o1), ldo(lvl + 1, o1), t.wx, t.wy};
}
__device__ __forceinline__ float4 env_value(const TexelTaps &q) {
    return lerp4(lerp4(q.a, q.b, q.wx), lerp4(q.c, q.d, q.wx), q.wy);
}
struct PairTaps {
    float4 v[3];  // a.rgb c.r | c.gb b.rg | b.b d.rgb
    float wx, wy;
};
__device__ __forceinline__ PairTaps env_taps(const RgbPair *__restrict__ lvl, const FaceDims &g, FaceST f) {
    TapPlace t = tap_place(g, f);
    PairTaps q;
    q.wx = t.wx;
    q.wy = t.wy;
    const float4 *p = reinterpret_cast<const float4 *>(lvl);
#pragma unroll
    for (int k = 0; k < 3; ++k) q.v[k] = ldo(p + k, t.idx * 24u);
    return q;
}
__device__ __forceinline__ float4 env_value(const PairTaps &q) {
    float4 A = make_float4(q.v[0].x, q.v[0].y, q.v[0].z, 0.0f), C = make_float4(q.v[0].w, q.v[1].x, q.v[1].y, 0.0f);
    float4 B = make_float4(q.v[1].z, q.v[1].w, q.v[2].x, 0.0f), D = make_float4(q.v[2].y, q.v[2].z, q.v[2].w, 0.0f);
    return lerp4(lerp4(A, B, q.wx), lerp4(C, D, q.wx), q.wy);
}

// The GGX samples of the prefiltered levels: entry k of level m is the tangent-frame half vector of Hammersley sample k for
// roughness^2 = alpha_m and, for filtered importance sampling, the environment
// chain level that sample reads (w; 0 otherwise).  That level is lod0 - log2(den)
// clamped to [0, last], where den = (1 - u2) + alpha^2 u2 is the GGX sampling
// denominator: for V = N the pdf of l is D / 4 = den^2 / (4 pi alpha^2), so
// 1/2 log2(omega_s / omega_p) + 1 = 1/2 log2(6 S^2 alpha^2 / N) + 1 - log2(den)
// (lod0 is that constant part, computed on the host in double precision).
// Levels with alpha = 0 (the mirror level) have no table.
struct GgxLevels {
    float alpha[8], lod0[8];
};
__device__ __forceinline__ void ggx_table_block(int block, int m, const GgxLevels &lv, int samples, int fis, int last,
                                                float4 *__restrict__ tables) {
    int k = block * 256 + (int)threadIdx.x;
    float alpha = lv.alpha[m];
    if (k >= samples || alpha == 0.0f) return;
    float a2 = alpha * alpha;
    float inv_n = 1.0f / (float)samples;
    float u2 = radical_inverse2((uint32_t)k);
    float4 t = ggx_tangent((float)k * inv_n, u2, a2);
    if (fis) {
        float den = fmaf(a2, u2, 1.0f - u2);
        t.w = fminf(fmaxf(lv.lod0[m] - __log2f(den), 0.0f), (float)last);
    }
    tables[(size_t)m * samples + k] = t;
}

// One wavefront per prefiltered texel of a level (roughness > 0), from level 0
// of the environment (or its RGB pairs): sample k's half vector from the table, its direction l
// the half vector reflected about the texel normal n; with N.L > 0 it adds
// L(l) N.L and N.L.  A lane takes its samples k and k + 64 together: both
// lookups' taps are in flight before either is added (the adds keep the order
// k, k + 64, k + 128, ...), and the next pair's table entries load one
// iteration ahead, with the current pair's taps.
template <typename TE>
__device__ __forceinline__ void prefilter_block(int block, int blocks, const TE *__restrict__ env, int S, int sm,
                                                const float4 *__restrict__ table, int samples,
                                                float4 *__restrict__ out) {
    int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
    // XCD-aware: each XCD's blocks take a contiguous run of texels, whose lobes
    // cover a fraction of the environment that its own L2 can hold
    int o = xcd_tile(block, blocks) * 4 + wave;
    if (o >= 6 * sm * sm) return;  // whole wavefront leaves together
    int f = o / (sm * sm), j = (o / sm) % sm, i = o % sm;
    v3 n = normalize(cube_texel_dir(f, i, j, sm));
    v3 T, B;
    tangent_frame(n, T, B);
    FaceDims dims = face_dims(S);
    Kahan r{0, 0}, g{0, 0}, b{0, 0}, w{0, 0};
    int last = samples - 1;
    float4 na = table[min(lane, last)], nb = table[min(lane + 64, last)];
    for (int k = lane; k < samples; k += 128) {
        float4 ta = na, tb = nb;
        if (k + 128 < samples) {
            na = table[k + 128];
            nb = table[min(k + 192, last)];
        }
        v3 ha = ggx_to_world(ta, n, T, B), hb = ggx_to_world(tb, n, T, B);
        float vha = dot(n, ha), vhb = dot(n, hb);
        v3 la = ha * (2.0f * vha) - n, lb = hb * (2.0f * vhb) - n;
        float nla = dot(n, la), nlb = dot(n, lb);
        bool ua = nla > 0.0f, ub = k + 64 < samples && nlb > 0.0f;
        decltype(env_taps(env, dims, FaceST{})) qa{}, qb{};
        if (ua) qa = env_taps(env, dims, cube_face(la));
        if (ub) qb = env_taps(env, dims, cube_face(lb));
        float4 La = env_value(qa), Lb = env_value(qb);
        if (ua) {
            kahan_add(r, La.x * nla);
            kahan_add(g, La.y * nla);
            kahan_add(b, La.z * nla);
            kahan_add(w, nla);
        }
        if (ub) {
            kahan_add(r, Lb.x * nlb);
            kahan_add(g, Lb.y * nlb);
            kahan_add(b, Lb.z * nlb);
            kahan_add(w, nlb);
        }
    }
    float R = wave_sum_compensated(kahan_value(r));
    float G = wave_sum_compensated(kahan_value(g));
    float Bv = wave_sum_compensated(kahan_value(b));
    float W = wave_sum_compensated(kahan_value(w));
    if (lane == 0) {
        float iw = 1.0f / W;
        out[o] = make_float4(R * iw, G * iw, Bv * iw, 0.0f);
    }
}

// Partial sums of a prefiltered level (roughness > 0) with filtered importance
// sampling.  Wavefront w of the grid takes tile w / chunks (8x8 texels of one
// face) and chunk w % chunks of the samples; its lanes are the tile's texels (a
// lane past the face edge computes a clamped texel and writes nothing).  Sample
// k's direction l is its half vector reflected about the texel normal n; with
// N.L > 0 it adds L(l) N.L and N.L, L read trilinearly from the environment
// chain at the sample's level.  part: [chunk][texel][8] = Kahan (s, c) of R,
// G, B and the weight, as irradiance_final_block sums them.
__device__ __forceinline__ void prefilter_fis_block(int block, const float4 *__restrict__ env,
                                                    const float4 *__restrict__ chain, int S, int last, int sm,
                                                    const float4 *__restrict__ table, int samples, int chunks,
                                                    float *__restrict__ part) {
    // wave-uniform by construction; readfirstlane tells the compiler, so the
    // sample loop and its table loads are scalar
    // (not XCD-aware: the matched mip levels are small enough for every L2,
    // and the XCD-contiguous order measured slower here)
    int w = __builtin_amdgcn_readfirstlane(block * 4 + (int)(threadIdx.x >> 6));
    int lane = threadIdx.x & 63;
    int tpf = (sm + 7) >> 3;
    if (w >= 6 * tpf * tpf * chunks) return;  // whole wavefront leaves together
    int tile = w / chunks, chunk = w - tile * chunks;
    int f = tile / (tpf * tpf), t = tile - f * (tpf * tpf);
    int i = (t % tpf) * 8 + (lane & 7), j = (t / tpf) * 8 + (lane >> 3);
    v3 n = normalize(cube_texel_dir(f, min(i, sm - 1), min(j, sm - 1), sm));
    v3 T, B;
    tangent_frame(n, T, B);
    Kahan r{0, 0}, g{0, 0}, b{0, 0}, wt{0, 0};
    // (samples <= 2^20 and chunks <= 16: the products fit in 32 bits)
    int k0 = chunk * samples / chunks, k1 = (chunk + 1) * samples / chunks;
    // two samples at a time, so that their taps are in flight together (the adds keep the
    // samples' order): the whole precompute of a 6x512^2 cube with 1024 samples takes 254 us,
    // with one at a time 275, with four (148 registers) 268
    constexpr int kFisRun = 2;
    const ConstFloat *tab = as_constant((const float *)table);
    for (int k = k0; k < k1; k += kFisRun) {
        TexelTaps t0[kFisRun], t1[kFisRun];
        float nl[kFisRun], fl[kFisRun];
#pragma unroll
        for (int u = 0; u < kFisRun; ++u) {
            const ConstFloat *e = tab + 4 * min(k + u, k1 - 1);
            float lod = e[3];  // the sample's, so wave-uniform
            v3 h = ggx_to_world(make_float4(e[0], e[1], e[2], 0.0f), n, T, B);
            float vh = dot(n, h);
            v3 l = h * (2.0f * vh) - n;
            nl[u] = k + u < k1 ? dot(n, l) : 0.0f;
            int l0 = __builtin_amdgcn_readfirstlane((int)lod);
            int l1 = min(l0 + 1, last);
            fl[u] = lod - (float)l0;
            if (nl[u] > 0.0f) {
                FaceST fs = cube_face(l);
                t0[u] = env_taps(l0 ? chain + chain_offset_pow2(S, l0) : env, face_dims(S >> l0), fs);
                t1[u] = env_taps(l1 ? chain + chain_offset_pow2(S, l1) : env, face_dims(S >> l1), fs);
            }
        }
#pragma unroll
        for (int u = 0; u < kFisRun; ++u) {
            if (nl[u] > 0.0f) {
                float4 L = lerp4(env_value(t0[u]), env_value(t1[u]), fl[u]);
                kahan_add(r, L.x * nl[u]);
                kahan_add(g, L.y * nl[u]);
                kahan_add(b, L.z * nl[u]);
                kahan_add(wt, nl[u]);
            }
        }
    }
    if (i < sm && j < sm) {
        int nout = 6 * sm * sm;
        int o = f * sm * sm + j * sm + i;
        float *p = part + ((size_t)chunk * nout + o) * 8;
        p[0] = r.s; p[1] = g.s; p[2] = b.s; p[3] = wt.s;
        p[4] = r.c; p[5] = g.c; p[6] = b.c; p[7] = wt.c;
    }
}

// One wavefront per BRDF table entry: N = +z, V = (sqrt(1 - NoV^2), 0, NoV).
// G_vis = G VoH / (NoH NoV) with G = G1(NoL) G1(NoV), G1(x) = x / (x(1-k)+k),
// written without the division by NoV: NoL VoH / (NoH (NoL(1-k)+k)(NoV(1-k)+k)).
__global__ void __launch_bounds__(256) k_brdf_lut(int size, int samples, float2 *__restrict__ out) {
    int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
    int o = blockIdx.x * 4 + wave;
    if (o >= size * size) return;
    int j = o / size, i = o % size;
    float NoV = ((float)i + 0.5f) / (float)size;
    float rough = ((float)j + 0.5f) / (float)size;
    float alpha = rough * rough, a2 = alpha * alpha, k = 0.5f * alpha;
    v3 V = mk3(sqrtf(fmaxf(0.0f, 1.0f - NoV * NoV)), 0.0f, NoV);
    v3 n = mk3(0.0f, 0.0f, 1.0f), T, B;
    tangent_frame(n, T, B);
    float gv = fmaf(NoV, 1.0f - k, k);
    float inv_n = 1.0f / (float)samples;
    Kahan A{0, 0}, Bs{0, 0};
    for (int s = lane; s < samples; s += 64) {
        v3 h = ggx_half((float)s * inv_n, radical_inverse2((uint32_t)s), a2, n, T, B);
        float vh = dot(V, h);
        float nl = fmaf(2.0f * vh, h.z, -V.z);
        if (nl > 0.0f) {
            float gvis = nl * vh / (h.z * fmaf(nl, 1.0f - k, k) * gv);
            float fc = pow5(1.0f - vh);
            kahan_add(A, (1.0f - fc) * gvis);
            kahan_add(Bs, fc * gvis);
        }
    }
    float a = wave_sum_compensated(kahan_value(A));
    float b = wave_sum_compensated(kahan_value(Bs));
    if (lane == 0) out[o] = make_float2(a * inv_n, b * inv_n);
}

// The same entries with the row's GGX half vectors made once into LDS (for up
// to kLutLdsSamples samples): block b takes kLutRowSlice entries of one row (one
// roughness), each wavefront a quarter of them in turn, its lanes splitting
// the samples as in k_brdf_lut (the same order); G_vis from a reciprocal, the
// compensated sums over groups of four samples.  The tangent frame of n = +z is
// T = -y, B = +x, so a half vector (x, y, z) of the sample table is (y, -x, z) in
// the frame of V, which has no y component: the table keeps (y, z), 8 bytes a
// sample, and V.h is two products (the table alone: 67 us with the frame's nine).
constexpr int kLutLdsSamples = 2048, kLutRowSlice = 32;
__device__ __forceinline__ void brdf_lut_rows_block(int block, int size, int samples, float2 *__restrict__ out,
                                                    float2 *tab) {  // tab: samples entries in LDS
    int slices = (size + kLutRowSlice - 1) / kLutRowSlice;
    int j = block / slices, i0 = (block - j * slices) * kLutRowSlice;
    float rough = ((float)j + 0.5f) / (float)size;
    float alpha = rough * rough, a2 = alpha * alpha, k = 0.5f * alpha;
    float inv_n = 1.0f / (float)samples;
    for (int s = (int)threadIdx.x; s < samples; s += 256) {
        float4 t = ggx_tangent((float)s * inv_n, radical_inverse2((uint32_t)s), a2);
        tab[s] = make_float2(t.y, t.z);
    }
    __syncthreads();
    int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
    for (int q = wave; q < kLutRowSlice; q += 4) {
        int i = i0 + q;
        if (i >= size) break;  // wave-uniform
        float NoV = ((float)i + 0.5f) / (float)size;
        float Vx = sqrtf(fmaxf(0.0f, 1.0f - NoV * NoV));
        float gv = fmaf(NoV, 1.0f - k, k);
        // Sample s's two terms, both >= 0: with N.L clamped at 0, a sample
        // below the horizon gets G_vis = 0 (N.L is a factor, the denominator
        // stays positive: h.z > 0, k > 0) and adds nothing, as if skipped.
        auto terms = [&](int s, float &ta, float &tb) {
            float2 h = tab[s];
            float vh = fmaf(Vx, h.x, NoV * h.y);
            float nl = fmaxf(fmaf(2.0f * vh, h.y, -NoV), 0.0f);
            float gvis = nl * vh * rcp(h.y * fmaf(nl, 1.0f - k, k) * gv);
            float fc = pow5(1.0f - vh);
            ta = (1.0f - fc) * gvis;
            tb = fc * gvis;
        };
        // a lane's samples in groups of four summed in plain float, each group
        // Kahan-added (the whole sum stays within a few units of rounding, as
        // for the irradiance), then the ones left over one by one
        Kahan A{0, 0}, Bs{0, 0};
        int s = lane;
        for (; s + 192 < samples; s += 256) {
            float a0, b0, a1, b1, a2, b2, a3, b3;
            terms(s, a0, b0);
            terms(s + 64, a1, b1);
            terms(s + 128, a2, b2);
            terms(s + 192, a3, b3);
            kahan_add(A, ((a0 + a1) + a2) + a3);
            kahan_add(Bs, ((b0 + b1) + b2) + b3);
        }
        for (; s < samples; s += 64) {
            float ta, tb;
            terms(s, ta, tb);
            kahan_add(A, ta);
            kahan_add(Bs, tb);
        }
        float a = wave_sum_compensated(kahan_value(A));
        float b = wave_sum_compensated(kahan_value(Bs));
        if (lane == 0) out[j * size + i] = make_float2(a * inv_n, b * inv_n);
    }
}

// ---------------------------------------------------------------------------
// launches
// ---------------------------------------------------------------------------
// Independent steps share a launch, each workgroup taking one step's block by its
// index: (1) irradiance source, RGB copy or the first chain levels, GGX tables and
// mirror levels; (chain levels beyond five: one launch per five more); (2) the
// integrals (rough prefiltered levels, irradiance partials, BRDF table); (3) the
// sums of partials.  Besides the launches this saves the tails of small levels,
// and it runs the prefilter, which the texture data path bounds, beside the
// irradiance and the BRDF table, which vector issue bounds.  One launch per step and
// level (ten, with filtered sampling sixteen or more) took 544 us at 6x512^2 and
// 108 us for the small filtered tables of a 6x64^2 cube, this takes 348 and 38.  At
// 6x512^2 the preparing launch is 27 us (25 MB read, 38 MB written), the integrals 330
// under the profiler (its steps one by one, with row-wise packed texels: 511), bound by the
// texture data path (90 % busy; vector issue 71 %), the sums 5 to 6.
struct IblLevel {
    int sm, chunks;         // face size; sample chunks (filtered sampling)
    int blocks;             // blocks in the integral launch (padded to whole rounds of XCDs)
    int final_blocks;       // blocks of the sum of partials
    float *part;
    const float4 *table;
    float4 *out;
};
struct IblArgs {
    const float4 *env;
    int S, src, irr, lpt, chunks, chunk_len;
    int fis, chain_last, levels, pref_samples, lut, lut_samples;
    float4 *src_tex, *src_tab, *chain;
    RgbPair *rgb;
    float *part;
    float4 *ggx, *irr_out;
    float2 *lut_out;
    GgxLevels lv;
    IblLevel level[8];
    int source_faces, source_blocks, env_blocks, ggx_blocks;  // launch 1 (then the mirror levels' blocks)
    int heavy, light, heavy_run, light_run;      // launch 2: blocks of each kind, and of each in a round / 8
    int partial_blocks, lut_blocks, out_blocks;  // (light = partial_blocks + lut_blocks)
};

template <bool kFis>
__global__ void __launch_bounds__(256) k_ibl_prepare(const IblArgs a) {
    int b = (int)blockIdx.x;
    if (b < a.source_blocks) {
        if (a.source_faces == 6) return ibl_source_block<6>(b, a.env, a.S, a.src, a.lpt, a.src_tex, a.src_tab);
        return ibl_source_block<1>(b, a.env, a.S, a.src, a.lpt, a.src_tex, a.src_tab);
    }
    b -= a.source_blocks;
    if (b < a.env_blocks) {
        if constexpr (kFis) {
            __shared__ ChainLds sm;
            env_chain_block(b, a.env, a.chain, a.S, 0, a.chain_last, chain_faces(a.S), sm);
        } else {
            env_rgb_block(b, a.env, a.S, a.rgb);
        }
        return;
    }
    b -= a.env_blocks;
    if (b < a.ggx_blocks) {
        int per = (a.pref_samples + 255) / 256, m = b / per;
        return ggx_table_block(b - m * per, m, a.lv, a.pref_samples, a.fis, a.chain_last, a.ggx);
    }
    b -= a.ggx_blocks;
    for (int m = 0; m < a.levels; ++m) {
        if (a.lv.alpha[m] != 0.0f) continue;
        int n = (6 * a.level[m].sm * a.level[m].sm + 255) / 256;
        if (b < n) return prefilter_mirror_block(b, a.env, a.S, a.level[m].sm, a.level[m].out);
        b -= n;
    }
}

__global__ void __launch_bounds__(256) k_env_chain(const IblArgs a, int first) {
    __shared__ ChainLds sm;
    env_chain_block((int)blockIdx.x, a.env, a.chain, a.S, first, a.chain_last, 1, sm);
}

// Rounds of 8 heavy_run prefilter blocks and 8 light_run others: the two kinds are
// spread over the launch, and every index keeps its XCD (blockIdx % 8).  The kind that
// would hold up the other issues first: the plain prefilter waits for the texture data
// path, so that the others, which only compute, go ahead of it (348 us for 6x512^2, 351
// without); the filtered prefilter's wavefronts are chains of dependent lookups, and go
// ahead in longer runs (6x512^2, 1024 samples: 217 us; in runs of 8 without, 238).
template <bool kFis, bool kPairs>
__global__ void __launch_bounds__(256) k_ibl_integrate(const IblArgs a) {
    extern __shared__ float4 lds[];
    int run = kNumXcd * (a.heavy_run + a.light_run);
    int round = (int)blockIdx.x / run, at = (int)blockIdx.x - round * run;
    if (at < kNumXcd * a.heavy_run) {
        int b = round * kNumXcd * a.heavy_run + at;
        for (int m = 0; m < a.levels; ++m) {
            const IblLevel &v = a.level[m];
            if (b < v.blocks) {
                if constexpr (kFis) {
                    __builtin_amdgcn_s_setprio(1);
                    prefilter_fis_block(b, a.env, a.chain, a.S, a.chain_last, v.sm, v.table, a.pref_samples, v.chunks,
                                        v.part);
                } else if constexpr (kPairs) {
                    prefilter_block(b, v.blocks, a.rgb, a.S, v.sm, v.table, a.pref_samples, v.out);
                } else {
                    prefilter_block(b, v.blocks, a.env, a.S, v.sm, v.table, a.pref_samples, v.out);
                }
                return;
            }
            b -= v.blocks;
        }
        return;
    }
    int b = round * kNumXcd * a.light_run + at - kNumXcd * a.heavy_run;
    if constexpr (!kFis) __builtin_amdgcn_s_setprio(1);
    if (b < a.partial_blocks) {
        int c = b / a.out_blocks;
        return irradiance_partial_block(b - c * a.out_blocks, c, a.src_tex, a.src_tab, 6 * a.src * a.src, a.chunk_len,
                                        a.irr, a.part);
    }
    b -= a.partial_blocks;
    if (b < a.lut_blocks) brdf_lut_rows_block(b, a.lut, a.lut_samples, a.lut_out, (float2 *)lds);
}

__global__ void __launch_bounds__(256) k_ibl_final(const IblArgs a) {
    int b = (int)blockIdx.x, nout = 6 * a.irr * a.irr, n = (4 * nout + 255) / 256;
    if (b < n) return irradiance_final_block(b, a.part, a.chunks, nout, a.irr_out);
    b -= n;
    for (int m = 0; m < a.levels; ++m) {
        const IblLevel &v = a.level[m];
        if (b < v.final_blocks) return irradiance_final_block(b, v.part, v.chunks, 6 * v.sm * v.sm, v.out);
        b -= v.final_blocks;
    }
}

// Sample chunks of a prefiltered level of face size sm: enough wavefronts to
// fill the chip (about 8192, 32 per CU) without splitting a tile's samples
// more than 16 ways.
static int prefilter_chunks(int sm) {
    int tpf = (sm + 7) / 8;
    int tiles = 6 * tpf * tpf;
    int c = (8192 + tiles - 1) / tiles;
    return c < 1 ? 1 : (c > 16 ? 16 : c);
}

IblPlan ibl_plan(int S, const epb_ibl_params &p) {
    IblPlan q{};
    q.S = S;
    q.src = S < p.irr_src_size ? S : p.irr_src_size;
    q.irr = p.irr_size;
    q.pref_base = S < p.pref_size ? S : p.pref_size;
    q.pref_levels = p.pref_levels;
    q.pref_samples = p.pref_samples;
    q.lut = p.lut_size;
    q.lut_samples = p.lut_samples;
    q.fis = p.pref_fis;
    q.chain_last = 0;
    while ((S >> (q.chain_last + 1)) >= 2) ++q.chain_last;
    int nsrc = 6 * q.src * q.src;
    int nout = 6 * q.irr * q.irr;
    int out_blocks = (nout + 255) / 256;
    // about four workgroups per CU (one per SIMD is too few to hide the serial
    // Kahan chains; eight gain nothing more), chunks of >= 256 sources
    int chunks = (1024 + out_blocks - 1) / out_blocks;
    int max_chunks = (nsrc + 255) / 256;
    if (chunks > max_chunks) chunks = max_chunks;
    if (chunks < 1) chunks = 1;
    q.chunks = chunks;
    size_t off = 0;
    auto take = [&](size_t bytes) {
        size_t o = off;
        off += (bytes + 255) & ~size_t(255);
        return o;
    };
    q.off_src = take((size_t)nsrc * 16);
    q.off_tab = take((size_t)nsrc * 16);
    q.off_part = take((size_t)chunks * nout * 8 * 4);
    // What the prefilter reads beside the environment itself: RGB pairs for plain sampling where
    // they pay (see RgbPair; 24 bytes a texel, 36 MiB at 6x512^2; rows of packed RGB took half),
    // levels 1 .. last of the mip chain for filtered sampling (16 bytes, a third as many texels).
    // The room never shrinks with a larger environment, more samples or levels, and is the same
    // for both, so that filtered sampling, which adds the partial sums, never asks for less than plain
    // sampling of the same sizes.
    size_t texels = (size_t)6 * S * S, lookups = 0;
    for (int m = 1; m < q.pref_levels; ++m) {
        size_t sm = (size_t)(q.pref_base >> m);
        lookups += 6 * sm * sm * q.pref_samples;
    }
    size_t most = q.pref_samples > 32 ? 2 * lookups : 0;  // texels of which a copy pays
    q.pairs = !q.fis && texels <= most;
    size_t pairs = (texels < most ? texels : most) * sizeof(RgbPair);
    size_t chain = q.fis ? (size_t)chain_offset_pow2(S, q.chain_last + 1) * sizeof(float4) : 0;
    q.off_env = take(pairs > chain ? pairs : chain);
    // the prefilter's GGX sample tables and partial sums of every level
    size_t part = 0;
    for (int m = 1; q.fis && m < q.pref_levels; ++m) {  // (level 0 has roughness 0: no samples)
        int sm = q.pref_base >> m;
        part += (size_t)prefilter_chunks(sm) * 6 * sm * sm * 8 * 4;
    }
    q.off_ggx = take(q.pref_levels > 1 ? (size_t)q.pref_levels * q.pref_samples * 16 : 0);  // a table per level
    q.off_ppart = take(part);
    q.bytes = off;
    return q;
}

hipError_t launch_precompute_ibl(const IblPlan &q, const float *env, float *irr, float *pref, float *lut,
                                 void *scratch, hipStream_t s) {
    char *sc = (char *)scratch;
    IblArgs a{};
    a.env = (const float4 *)env;
    a.S = q.S; a.src = q.src; a.irr = q.irr; a.chunks = q.chunks;
    a.fis = q.fis; a.chain_last = q.chain_last; a.levels = q.pref_levels; a.pref_samples = q.pref_samples;
    a.lut = q.lut; a.lut_samples = q.lut_samples;
    a.src_tex = (float4 *)(sc + q.off_src);
    a.src_tab = (float4 *)(sc + q.off_tab);
    a.part = (float *)(sc + q.off_part);
    a.chain = (float4 *)(sc + q.off_env);
    a.rgb = (RgbPair *)(sc + q.off_env);
    a.ggx = (float4 *)(sc + q.off_ggx);
    a.irr_out = (float4 *)irr;
    a.lut_out = (float2 *)lut;
    int nsrc = 6 * q.src * q.src, nout = 6 * q.irr * q.irr, n0 = 6 * q.S * q.S;
    int kk = (q.S / q.src) * (q.S / q.src);
    a.lpt = 1;
    while (a.lpt < kk && a.lpt < 64) a.lpt *= 2;
    a.chunk_len = (nsrc + q.chunks - 1) / q.chunks;
    // the levels, and the blocks of every step
    float *ppart = (float *)(sc + q.off_ppart);
    float4 *out = (float4 *)pref;
    int mirror_blocks = 0, final_blocks = ceil_div(4 * nout, 256);
    for (int m = 0; m < q.pref_levels; ++m) {
        IblLevel &v = a.level[m];
        v.sm = q.pref_base >> m;
        int n = 6 * v.sm * v.sm;
        v.out = out;
        out += n;
        v.table = a.ggx + (size_t)m * q.pref_samples;
        float rough = q.pref_levels > 1 ? (float)m / (float)(q.pref_levels - 1) : 0.0f;
        float alpha = a.lv.alpha[m] = rough * rough;
        if (alpha == 0.0f) {
            mirror_blocks += ceil_div(n, 256);
            continue;
        }
        int blocks = ceil_div(n, 4);
        if (q.fis) {
            double a2 = (double)alpha * alpha;
            a.lv.lod0[m] = (float)(0.5 * std::log2(6.0 * q.S * q.S * a2 / q.pref_samples) + 1.0);
            int tpf = (v.sm + 7) / 8;
            v.chunks = prefilter_chunks(v.sm);
            v.part = ppart;
            ppart += (size_t)v.chunks * n * 8;
            v.final_blocks = ceil_div(4 * n, 256);
            final_blocks += v.final_blocks;
            blocks = ceil_div(6 * tpf * tpf * v.chunks, 4);
        }
        v.blocks = ceil_div(blocks, kNumXcd) * kNumXcd;
        a.heavy += v.blocks;
    }
    a.source_faces = q.src * q.src * a.lpt <= kSourceThreads ? 1 : 6;
    a.source_blocks = ceil_div(q.src * q.src * a.lpt, 256) * (6 / a.source_faces);
    int side = q.S < 32 ? q.S : 32;
    if (q.fis) a.env_blocks = q.chain_last > 0 ? (q.S / side) * (q.S / side) * (6 / chain_faces(q.S)) : 0;
    else a.env_blocks = q.pairs ? ceil_div(n0, 256) : 0;
    a.ggx_blocks = q.pref_levels > 1 ? ceil_div(q.pref_samples, 256) * q.pref_levels : 0;
    a.out_blocks = ceil_div(nout, 256);
    a.partial_blocks = a.out_blocks * q.chunks;
    bool lut_rows = q.lut_samples <= kLutLdsSamples;
    a.lut_blocks = lut_rows ? q.lut * ceil_div(q.lut, kLutRowSlice) : 0;
    a.light = a.partial_blocks + a.lut_blocks;
    // rounds of so many prefilter blocks per XCD, the others spread over them (k_ibl_integrate)
    a.heavy_run = a.heavy > 0 ? (q.fis ? 32 : 8) : 0;
    int rounds = a.heavy > 0 ? ceil_div(a.heavy, kNumXcd * a.heavy_run) : 1;
    a.light_run = ceil_div(a.light, kNumXcd * rounds);
    int grid = rounds * kNumXcd * (a.heavy_run + a.light_run);
    // (at most 16 KB: ten workgroups would fit a CU, more than the prefilter's registers allow)
    size_t lds = lut_rows ? (size_t)q.lut_samples * sizeof(float2) : 0;

    int first = a.source_blocks + a.env_blocks + a.ggx_blocks + mirror_blocks;
    if (q.fis) hipLaunchKernelGGL(k_ibl_prepare<true>, dim3(first), dim3(256), 0, s, a);
    else hipLaunchKernelGGL(k_ibl_prepare<false>, dim3(first), dim3(256), 0, s, a);
    for (int k = kChainStep; q.fis && k < q.chain_last; k += kChainStep) {
        int Sk = q.S >> k, w = Sk < 32 ? 1 : Sk / 32;
        hipLaunchKernelGGL(k_env_chain, dim3(w * w * 6), dim3(256), 0, s, a, k);
    }
    if (q.fis) hipLaunchKernelGGL((k_ibl_integrate<true, false>), dim3(grid), dim3(256), lds, s, a);
    else if (q.pairs) hipLaunchKernelGGL((k_ibl_integrate<false, true>), dim3(grid), dim3(256), lds, s, a);
    else hipLaunchKernelGGL((k_ibl_integrate<false, false>), dim3(grid), dim3(256), lds, s, a);
    hipLaunchKernelGGL(k_ibl_final, dim3(final_blocks), dim3(256), 0, s, a);
    if (!lut_rows)
        hipLaunchKernelGGL(k_brdf_lut, dim3(ceil_div(q.lut * q.lut, 4)), dim3(256), 0, s, q.lut, q.lut_samples,
                           a.lut_out);
    return hipGetLastError();
}

}  // namespace epb
