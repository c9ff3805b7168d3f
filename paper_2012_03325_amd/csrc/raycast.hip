// G-buffer and depth-map pass on sphere fields: the stand-in for the paper's
// rasterised geometry pass (Sec. 4) and its depth renders from each light
// (Sec. 5.1), on the device so that cameras and lights can change per frame.
//
// gfx950 mapping:
//  * k_sphere_records: one thread per sphere writes a conservative pixel box
//    (the projected corners of the sphere's bounding cube plus a texel of margin;
//    the cube lies wholly in front of the camera there, so the hull of its
//    corners contains the sphere's image; a sphere crossing the camera plane
//    covers the screen, one behind it nothing) and a lower bound of its hits'
//    depths.
//  * k_raycast: one workgroup per region of wavefront tiles.  The whole
//    workgroup tests every box against the region once and appends the
//    overlapping spheres to a list in LDS; then each wavefront goes through the
//    list by itself, 64 spheres at a time, one per lane: a lane forms its
//    sphere's ray-independent terms (centre offset and c = |oc|^2 - r^2) and
//    tests the sphere against the cone around the wavefront's rays, and the
//    survivors' terms go to the wavefront's LDS slots, from which the
//    intersection loop reads them as broadcasts.  A survivor whose depth bound
//    lies behind every lane's hit costs one compare.
//  * intersections are double precision with contraction off (IEEE sqrt and
//    division), the results rounded to the destination types on store.  A hit
//    replaces the current one if it is strictly nearer, or equally near with a
//    lower index, so the order of the list does not matter.
//
// Bound: double-precision issue and the latency of the candidate loop where
// spheres overlap, the G-buffer's stores elsewhere.  Measured per call (512
// spheres and the plane): 1920x1080 G-buffer 26 us (74.6 MB of stores, 2.9 TB/s),
// 2048^2 depth map of a light 23 us; 16384 spheres at 1280x720 41 us.  One workgroup per
// 16x16 pixels that took every box by itself, its list to every pixel and an
// XCD-contiguous order: 50, 57 and 163 us.
#include <type_traits>

#include "device_common.hpp"
#include "launch.hpp"

namespace epb {

// A sphere's pixel box [x0, x1) x [y0, y1) (inside the image) and a lower bound
// of the depth of its hits.  The box is kept as (x0, -x1) and (y0, -y1), so that
// adding (-X1, X0) and (-Y1, Y0) to it leaves four negative halves exactly when it
// meets the region [X0, X1) x [Y0, Y1): two packed additions, one and, one compare.
typedef short Short2 __attribute__((ext_vector_type(2)));
struct SphereRec {
    Short2 x, y;
    float zmin;
    unsigned pad;
};
static_assert(sizeof(SphereRec) == kSphereRecBytes, "the scratch holds one record per sphere");

__global__ void __launch_bounds__(256) k_sphere_records(const RayScene s, const RayCam c,
                                                        SphereRec *__restrict__ rec) {
#pragma clang fp contract(off)
    int k = blockIdx.x * blockDim.x + threadIdx.x;
    if (k >= s.n) return;
    double cc[3] = {s.center[3 * k], s.center[3 * k + 1], s.center[3 * k + 2]};
    double r = s.radius[k];
    double v[3];
    for (int i = 0; i < 3; ++i) v[i] = c.M[4 * i] * cc[0] + c.M[4 * i + 1] * cc[1] + c.M[4 * i + 2] * cc[2] + c.M[4 * i + 3];
    const double eps = 1e-3;
    int x0 = 0, x1 = 0, y0 = 0, y1 = 0;  // behind the camera
    if (-(v[2] + r) <= eps && -(v[2] - r) <= eps) {
    } else if (-(v[2] + r) <= eps) {  // crosses the camera plane
        x1 = c.W;
        y1 = c.H;
    } else {
        double lx = 1e300, hx = -1e300, ly = 1e300, hy = -1e300;
        for (int q = 0; q < 4; ++q) {  // near and far edges of the cube, per axis
            double e = (q & 1) ? r : -r, z = -(v[2] + ((q & 2) ? r : -r));
            double px = c.cx + c.fx * (v[0] + e) / z - 0.5, py = c.cy - c.fy * (v[1] + e) / z - 0.5;
            lx = fmin(lx, px); hx = fmax(hx, px);
            ly = fmin(ly, py); hy = fmax(hy, py);
        }
        // clamp in double before converting (far-off boxes would overflow int)
        x0 = (int)fmin(fmax(floor(lx) - 1.0, 0.0), (double)c.W);
        x1 = (int)fmax(fmin(ceil(hx) + 2.0, (double)c.W), 0.0);
        y0 = (int)fmin(fmax(floor(ly) - 1.0, 0.0), (double)c.H);
        y1 = (int)fmax(fmin(ceil(hy) + 2.0, (double)c.H), 0.0);
    }
    // depth of the nearest point, lowered by far more than a hit's rounding error: the hit of a
    // grazing ray is off by up to sqrt(2^-53) of the distances that enter it, about 1e-8 of them.
    // The ray parameter t is the depth only as far as R is a rotation: with E = R R^T - 1 the hit
    // o + t d has the depth t + (E T)_z - t (E v)_z, and t |v| is at most about the distances' sum, so
    // that t differs from it by less than 3 |E| of them up to |E| = 1/4; above that no bound is used.
    double mag = fabs(cc[0]) + fabs(cc[1]) + fabs(cc[2]) + fabs(c.M[3]) + fabs(c.M[7]) + fabs(c.M[11]) + fabs(r);
    SphereRec q;
    q.x = Short2{(short)x0, (short)-x1};
    q.y = Short2{(short)y0, (short)-y1};
    q.zmin = c.skew <= 0.25 ? (float)(-v[2] - fabs(r) - (4e-6 + 3.0 * c.skew) * mag) : -__builtin_inff();
    q.pad = 0;
    rec[k] = q;
}

// A wavefront's lanes cover LX x 64 / LX pixels, each lane PPT pixels of one column
// (64 / LX rows apart), and a workgroup NX x NY wavefronts; kLoads spheres per thread are
// tested against the workgroup's region between two barriers.

// Ray-independent terms of a sphere that a wavefront will intersect.
struct alignas(16) RayCand {
    double oc[3], c0;
};

__device__ __forceinline__ float3 to_float3(const double v[3]) { return make_float3((float)v[0], (float)v[1], (float)v[2]); }
__device__ __forceinline__ float from_lane(float v, int lane) {
    return __builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, v), lane));
}

template <typename TG, int LX, int PPT, int NX, int NY, int kLoads>
__global__ void __launch_bounds__(64 * NX *NY) k_raycast(const RayScene s, const RayCam c,
                                                         const SphereRec *__restrict__ rec, RayOut out) {
#pragma clang fp contract(off)
    constexpr int kWaves = NX * NY, kThreads = 64 * kWaves;
    constexpr int kRayLx = LX, kRayLy = 64 / LX, kRayTy = kRayLy * PPT, kRx = NX * kRayLx, kRy = NY * kRayTy;
    constexpr int kGroup = kThreads * kLoads;  // spheres tested between two barriers
    constexpr int kList = kGroup + 512;
    __shared__ unsigned short list[kList];
    __shared__ int list_n;
    __shared__ RayCand cand[kWaves][64];
    __shared__ float cand_z[kWaves][64];
    __shared__ unsigned short cand_k[kWaves][64];
    // Regions in launch order, so that the XCDs share the crowded rows of the image: with a
    // contiguous band of regions per XCD, most XCDs idle while those of the crowded bands work
    // (512 spheres at 1920x1080: 37 us against 27).
    int region = (int)blockIdx.x;
    int across = (c.W + kRx - 1) / kRx;
    int ry = region / across;
    int X0 = (region - ry * across) * kRx, Y0 = ry * kRy;
    int t = threadIdx.x, lane = t & 63;
    int wv = __builtin_amdgcn_readfirstlane(t >> 6);
    int x = X0 + (wv % NX) * kRayLx + lane % kRayLx, y = Y0 + (wv / NX) * kRayTy + lane / kRayLx;
    if (t == 0) list_n = 0;
    // (the region's far edges at most 16384 + a region: 16 bits hold every sum)
    Short2 at_x = {(short)-(X0 + kRx), (short)X0}, at_y = {(short)-(Y0 + kRy), (short)Y0};
    // The view-space rays' x of the region's columns and y of its rows: one division each where
    // a lane has several pixels (four 2048^2 depth maps and their tiling 144 us with the divisions
    // of every pixel, 139), every lane's own elsewhere (720p, 16384 spheres: 40.7 us against 41.1,
    // the additional barrier delays the region test).
    double v0, v1s[PPT];
    if constexpr (PPT > 1) {
        __shared__ double ray_v[kRx + kRy];
        static_assert(kRx + kRy <= kThreads, "a thread per column and row");
        if (t < kRx + kRy) {
            bool col = t < kRx;
            double at = col ? (double)(X0 + t) + 0.5 - c.cx : (double)(Y0 + t - kRx) + 0.5 - c.cy;
            double v = at / (col ? c.fx : c.fy);
            ray_v[t] = col ? v : -v;
        }
        __syncthreads();
        v0 = ray_v[x - X0];
        for (int j = 0; j < PPT; ++j) v1s[j] = ray_v[kRx + y - Y0 + j * kRayLy];
    } else {
        v0 = ((double)x + 0.5 - c.cx) / c.fx;
        v1s[0] = -(((double)y + 0.5 - c.cy) / c.fy);
    }
    double d[PPT][3], aa[PPT];
#pragma unroll
    for (int j = 0; j < PPT; ++j) {
        double v1 = v1s[j], v2 = -1.0;
        for (int k = 0; k < 3; ++k) d[j][k] = c.M[k] * v0 + c.M[4 + k] * v1 + c.M[8 + k] * v2;
        aa[j] = d[j][0] * d[j][0] + d[j][1] * d[j][1] + d[j][2] * d[j][2];
    }
    // The cone around the wavefront's rays, made when there is a sphere to test: axis = the mean of
    // its corner rays (its centre ray), sin_a = the largest sine of an angle to the axis, which a
    // corner has (the directions within an angle below 90 degrees form a convex cone).  cos_a =
    // sin_a = 0 keeps every sphere.
    float3 ax = make_float3(0.0f, 0.0f, 0.0f);
    float sin_a = 0.0f, cos_a = 0.0f;
    bool have_cone = false;
    auto make_cone = [&]() {
        constexpr int kC1 = kRayLx - 1, kC2 = 64 - kRayLx, kC3 = 63;
        float3 f0 = to_float3(d[0]), f1 = to_float3(d[PPT - 1]);
        ax.x = from_lane(f0.x, 0) + from_lane(f0.x, kC1) + from_lane(f1.x, kC2) + from_lane(f1.x, kC3);
        ax.y = from_lane(f0.y, 0) + from_lane(f0.y, kC1) + from_lane(f1.y, kC2) + from_lane(f1.y, kC3);
        ax.z = from_lane(f0.z, 0) + from_lane(f0.z, kC1) + from_lane(f1.z, kC2) + from_lane(f1.z, kC3);
        float inv = rsq(ax.x * ax.x + ax.y * ax.y + ax.z * ax.z);
        ax.x *= inv; ax.y *= inv; ax.z *= inv;
        // (the lanes of the upper half hold the last row's rays, those of the lower half the first row's)
        float3 f = lane < 32 ? f0 : f1;
        float il = rsq(f.x * f.x + f.y * f.y + f.z * f.z);
        float cx = f.y * ax.z - f.z * ax.y, cy = f.z * ax.x - f.x * ax.z, cz = f.x * ax.y - f.y * ax.x;
        float sn = sqrtf(cx * cx + cy * cy + cz * cz) * il;
        float cs = (f.x * ax.x + f.y * ax.y + f.z * ax.z) * il;
        sin_a = fmaxf(fmaxf(from_lane(sn, 0), from_lane(sn, kC1)), fmaxf(from_lane(sn, kC2), from_lane(sn, kC3)));
        float cmin = fminf(fminf(from_lane(cs, 0), from_lane(cs, kC1)), fminf(from_lane(cs, kC2), from_lane(cs, kC3)));
        cos_a = sqrtf(fmaxf(1.0f - sin_a * sin_a, 0.0f));
        if (!(cmin > 0.1f)) sin_a = cos_a = 0.0f;  // (also for overflowing or undefined rays)
        have_cone = true;
    };
    double best[PPT], far_num[PPT];  // far_num / aa is past best
    int who[PPT];
#pragma unroll
    for (int j = 0; j < PPT; ++j) {
        best[j] = far_num[j] = __builtin_inf();
        who[j] = -1;
    }
    if (PPT == 1) __syncthreads();  // list_n (with several pixels the barrier above)
    for (int base = 0; base < s.n; base += kGroup) {
        // the spheres of this group whose boxes meet the region, appended in any order
        Short2 bx[kLoads], by[kLoads];
#pragma unroll
        for (int g = 0; g < kLoads; ++g) {
            const SphereRec &q = rec[min(base + g * kThreads + t, s.n - 1)];
            bx[g] = q.x;
            by[g] = q.y;
        }
#pragma unroll
        for (int g = 0; g < kLoads; ++g) {
            int k = base + g * kThreads + t;
            Short2 ox = bx[g] + at_x, oy = by[g] + at_y;
            unsigned both = __builtin_bit_cast(unsigned, ox) & __builtin_bit_cast(unsigned, oy);
            bool in = k < s.n && (both & 0x80008000u) == 0x80008000u;
            unsigned long long m = __ballot(in);
            if (m) {
                int at = 0;
                if (lane == 0) at = atomicAdd(&list_n, __popcll(m));
                at = __builtin_amdgcn_readfirstlane(at) + __popcll(m & ((1ull << lane) - 1ull));
                if (in) list[at] = (unsigned short)k;
            }
        }
        __syncthreads();
        int n = __builtin_amdgcn_readfirstlane(list_n);
        bool last = base + kGroup >= s.n;
        if (!last) {
            __syncthreads();  // every wavefront has read the count
            if (n <= kList - kGroup) continue;  // another group fits behind it: the list keeps growing
            if (t == 0) list_n = 0;
        }
        if (n > 0 && !have_cone) make_cone();
        for (int e = 0; e < n; e += 64) {
            bool keep = false;
            RayCand q{};
            int k = 0;
            float z = 0.0f;
            if (e + lane < n) {
                k = list[e + lane];
                z = rec[k].zmin;
                double r = s.radius[k];
                for (int i = 0; i < 3; ++i) q.oc[i] = c.o[i] - s.center[3 * k + i];
                q.c0 = (q.oc[0] * q.oc[0] + q.oc[1] * q.oc[1] + q.oc[2] * q.oc[2]) - r * r;
                // distance of the centre from the cone (a lower bound): over it by more than the
                // radius and the rounding of these lines means that no ray meets the sphere
                float3 o = to_float3(q.oc);
                float cx = o.y * ax.z - o.z * ax.y, cy = o.z * ax.x - o.x * ax.z, cz = o.x * ax.y - o.y * ax.x;
                float off = sqrtf(cx * cx + cy * cy + cz * cz) * cos_a + (o.x * ax.x + o.y * ax.y + o.z * ax.z) * sin_a;
                float mag = fabsf(o.x) + fabsf(o.y) + fabsf(o.z) + fabsf((float)r);
                keep = !(off > fabsf((float)r) + 1e-5f * mag) || !(mag < 1e15f);
            }
            unsigned long long m = __ballot(keep);
            int at = __popcll(m & ((1ull << lane) - 1ull)), cnt = __popcll(m);
            if (keep) {
                cand[wv][at] = q;
                cand_z[wv][at] = z;
                cand_k[wv][at] = (unsigned short)k;
            }
            __builtin_amdgcn_wave_barrier();  // the wavefront's own slots: written before they are read
            // The survivors, kWidth at a time: those whose depth bound lies behind every lane's hit are
            // skipped, the discriminants of the others formed side by side, and the roots taken only
            // where some lane has a hit.
            auto meet = [&](auto width) {
                constexpr int kWidth = decltype(width)::value;
                for (int i = 0; i < cnt; i += kWidth) {
                    int at[kWidth];
                    double zi[kWidth], b[kWidth][PPT], disc[kWidth][PPT];
                    bool near[kWidth][PPT], open = false, any = false;
#pragma unroll
                    for (int u = 0; u < kWidth; ++u) {
                        at[u] = kWidth == 1 ? i : min(i + u, cnt - 1);  // (the last one again: no nearer than itself)
                        zi[u] = (double)cand_z[wv][at[u]];
#pragma unroll
                        for (int j = 0; j < PPT; ++j) open |= best[j] > zi[u];
                    }
                    if (!__ballot(open)) continue;
#pragma unroll
                    for (int u = 0; u < kWidth; ++u) {
                        const RayCand &a = cand[wv][at[u]];
#pragma unroll
                        for (int j = 0; j < PPT; ++j) {
                            b[u][j] = d[j][0] * a.oc[0] + d[j][1] * a.oc[1] + d[j][2] * a.oc[2];
                            disc[u][j] = b[u][j] * b[u][j] - aa[j] * a.c0;
                            near[u][j] = !(disc[u][j] < 0.0) && best[j] > zi[u];
                            any |= near[u][j];
                        }
                    }
                    if (kWidth * PPT > 1 && !__ballot(any)) continue;
#pragma unroll
                    for (int u = 0; u < kWidth; ++u)
#pragma unroll
                        for (int j = 0; j < PPT; ++j) {
                            if (!near[u][j]) continue;
                            double num = -b[u][j] - sqrt(disc[u][j]);
                            // the quotient is monotone in its numerator: no division for a hit that lies behind
                            if (!(num > 0.0) || num > far_num[j]) continue;
                            double tt = num / aa[j];
                            int kk = cand_k[wv][at[u]];
                            if (tt > 0.0 && (tt < best[j] || (tt == best[j] && kk < who[j]))) {
                                best[j] = tt;
                                far_num[j] = num * (1.0 + 0x1p-50);
                                who[j] = kk;
                            }
                        }
                }
            };
            // Two at a time where most of 64 spheres have survived: a wavefront there is a serial chain of
            // discriminants (512 spheres within some pixels of 1920x1080: 106 us with one at a time and the
            // root before the vote, 80 one at a time, 71 so); with fewer survivors each is worth its own
            // skip (64 large spheres over 1920x1080, depth: 35.1 us, 36.6 two at a time throughout).
            if (PPT > 1 && cnt > 32) meet(std::integral_constant<int, 2>());
            else meet(std::integral_constant<int, 1>());
            __builtin_amdgcn_wave_barrier();
        }
        if (!last) __syncthreads();  // the next group refills the list
    }
    unsigned plane = (unsigned)c.W * (unsigned)c.H;
#pragma unroll
    for (int j = 0; j < PPT; ++j) {
        int yj = y + j * kRayLy;
        if (s.plane && d[j][1] < 0.0) {
            double tt = -c.o[1] / d[j][1];
            if (tt > 0.0 && tt < best[j]) {
                best[j] = tt;
                who[j] = s.n;
            }
        }
        if (x >= c.W || yj >= c.H) continue;
        unsigned p = __umul24((unsigned)yj, (unsigned)c.W) + (unsigned)x;
        stf(out.depth, p, (float)best[j]);
        if (!out.normal) continue;
        float nr[3] = {0.0f, 0.0f, 0.0f}, al[3] = {0.0f, 0.0f, 0.0f}, rg = 0.0f, mt = 0.0f;
        int w = who[j];
        if (w >= 0 && w < s.n) {
            double r = s.radius[w];
            double n3[3];
            for (int k = 0; k < 3; ++k) n3[k] = (c.o[k] + best[j] * d[j][k] - s.center[3 * w + k]) / r;
            double len = sqrt(n3[0] * n3[0] + n3[1] * n3[1] + n3[2] * n3[2]);
            for (int k = 0; k < 3; ++k) nr[k] = (float)(n3[k] / len);
            for (int k = 0; k < 3; ++k) al[k] = s.albedo[3 * w + k];
            rg = s.rough[w];
            mt = s.metal[w];
        } else if (w == s.n) {
            nr[1] = 1.0f;
            for (int k = 0; k < 3; ++k) al[k] = s.plane_albedo[k];
            rg = s.plane_rough;
            mt = s.plane_metal;
        }
        TG *nrm = (TG *)out.normal, *alb = (TG *)out.albedo;
        for (int k = 0; k < 3; ++k) {
            stf(nrm, k * plane + p, nr[k]);
            stf(alb, k * plane + p, al[k]);
        }
        stf((TG *)out.rough, p, rg);
        stf((TG *)out.metal, p, mt);
    }
}

template <typename TG, int LX, int PPT, int NX, int NY, int kLoads>
static void go_raycast(const RayScene &s, const RayCam &c, const RayOut &out, const SphereRec *rec, hipStream_t st) {
    int regions = ceil_div(c.W, NX * LX) * ceil_div(c.H, NY * (64 / LX) * PPT);
    hipLaunchKernelGGL((k_raycast<TG, LX, PPT, NX, NY, kLoads>), dim3(regions), dim3(64 * NX * NY), 0, st, s, c, rec, out);
}

hipError_t launch_raycast(const RayScene &s, const RayCam &c, const RayOut &out, epb_dtype dtype, void *scratch,
                          hipStream_t st) {
    SphereRec *rec = (SphereRec *)scratch;
    if (s.n > 0) hipLaunchKernelGGL(k_sphere_records, dim3(ceil_div(s.n, 256)), dim3(256), 0, st, s, c, rec);
    // Two pixels per lane share the ray set-up, the region test and the cone test: the better split
    // while there are few spheres per wavefront and enough wavefronts for the chip (512 spheres:
    // 1920x1080 29 us against 32, 640x480 17 against 14).  With more spheres the narrower cone of an
    // 8 x 8 tile and the workgroup's eight wavefronts sharing one region test win (1920x1080, 16384
    // spheres: 89 us against 99; 2048 spheres equal).
    if (s.n <= 1024 && (size_t)c.W * c.H >= (size_t)1 << 20) {
        // Regions of 32 x 16 pixels where attributes are written, so that a workgroup fills whole
        // 128-byte lines of every plane: neighbouring regions belong to different XCDs, which write
        // parts of a line one by one (3840x2160 G-buffer of the plane alone 57 us with regions of 16 x
        // 32, 46 so, with 512 spheres 75 and 66).  A depth map keeps the narrower cone of 8 x 16 pixels
        // (2048^2, 512 spheres: 30.5 us, 33.9 with 16 x 8).
        if (!out.normal) go_raycast<float, 8, 2, 2, 2, 2>(s, c, out, rec, st);
        else if (dtype == EPB_F32) go_raycast<float, 16, 2, 2, 2, 2>(s, c, out, rec, st);
        else go_raycast<__half, 16, 2, 2, 2, 2>(s, c, out, rec, st);
    } else {
        if (dtype == EPB_F32) go_raycast<float, 8, 1, 2, 4, 4>(s, c, out, rec, st);
        else go_raycast<__half, 8, 1, 2, 4, 4>(s, c, out, rec, st);
    }
    return hipGetLastError();
}

}  // namespace epb
