// Batch LiDAR: ray casting of the resident, rigidly posed Gaussians for grids
// of rays (rotating or solid-state sensors) and for listed rays
// (non-repetitive scan patterns, ordered on the host into compact tiles), through
// the same sort and tile binning as the cameras.
//
// Projection (one thread per Gaussian, a group of scans per thread):
//   * pose into the sensor frame with the binary32 specification of the
//     camera path (t = A mu + a);
//   * key = bits of the centre distance |t| (binary32, sqrt correctly
//     rounded), so the compositing order is (distance, index);
//   * tile rectangle: rows and columns of rays whose direction lies in the
//     cone of the sphere of radius sqrt(Qmax) * max scale around t (Qmax the
//     opacity bucket bound of the camera path), its sine widened by a relative
//     2e-4 and 4e-6, its angles by kAngleSlack against the errors of their
//     polynomials; a cone across the seam of a full turn takes the hull of its
//     two column ranges, a sensor inside the sphere takes the whole grid;
//   * record: whitening W = S^-1 R^T (R, S the Gaussian's rotation in the
//     sensor frame and its scales), the centre t, log2 o, the cosine of the
//     cone's half-angle for culling, and W t as far as it fits: 64 bytes, one
//     aligned sector, since the projection is bound by these stores and the
//     rasteriser gathers them at 2.5 TB/s.  What else a ray needs (the last of
//     W t, the centre direction) is made when a record is staged.
// Raster (one workgroup per tile of rays, one ray per thread): for each
// listed Gaussian, d' = W d, t* = (d' . W t) / |d'|^2 (the peak of the
// Gaussian along the ray), q = |W (t - t* d)|^2 (the offset taken in metres
// first, so that no large whitened terms cancel), log2 alpha = log2 o - q/2
// log2 e; then the compositing rules of the camera path with the range t* in
// place of the depth.
#include "gsr_device.h"
#include "gsr_wave.h"

#include <algorithm>
#include <type_traits>

namespace gsr {
namespace {

constexpr float kLidarLogAlphaMin = -7.99435343685886f;   // log2(1/255)
constexpr float kHalfPi = 1.5707963267948966f;
constexpr float kTwoPi = 6.283185307179586f;
constexpr int kLdsBeams = 256;      // angular scans with at most this many beams search their elevations in LDS
constexpr int kLdsTileAz = 1024;     // listed rays: tile azimuth tables up to this many floats are read from LDS
constexpr int kLidarRec = 4;        // float4s per record: whitening rows + centre, (log2 o, cone, first two of W t)
constexpr int kLidarStage = 5;      // float4s per staged record: whitening rows + centre, log2 o + W t, cone

// First index r in [0, H) with v[r] >= x (strict = false) or v[r] > x
// (strict = true), v ascending; H if none.
__device__ __forceinline__ int first_at_least(const float* v, int H, float x, bool strict)
{
    int lo = 0, hi = H;
    while (lo < hi) {
        const int mid = (lo + hi) >> 1;
        const bool below = strict ? v[mid] <= x : v[mid] < x;
        if (below) lo = mid + 1; else hi = mid;
    }
    return lo;
}

// Rows [r0, r1) with lo[r] >= a (r0) and hi[r] > b (r1): both binary searches
// over H ascending values step for step, so each waits for one pair of reads
// per halving.
__device__ __forceinline__ void rows_between(const float* lo, const float* hi, int H, float a, float b, int* r0, int* r1)
{
    int p = 0, q = 0;
    for (int step = 1 << (31 - __builtin_clz((unsigned)H)); step > 0; step >>= 1) {     // H is the same in every lane
        const int pn = p + step, qn = q + step;
        const float x = lo[min(pn, H) - 1], y = hi[min(qn, H) - 1];
        if (pn <= H && x < a) p = pn;
        if (qn <= H && y <= b) q = qn;
    }
    *r0 = p;
    *r1 = q;
}

// Rectangles, cones and the azimuth window are bounds (any ray tile too many
// costs time only), so their angles come from polynomials, with kAngleSlack
// added against their errors: asin x = pi/2 - sqrt(1 - x) P3(x) (Abramowitz and
// Stegun 4.4.45, 6.8e-5) and an odd fit of atan on [0, 1] (1.2e-5).
constexpr float kAngleSlack = 1.5e-4f;
__device__ __forceinline__ float asin_poly(float x)       // x in [0, 1]
{
    const float p = fmaf(x, fmaf(x, fmaf(x, -0.0187293f, 0.0742610f), -0.2121144f), 1.5707288f);
    return fmaf(-__builtin_amdgcn_sqrtf(fmaxf(0.0f, 1.0f - x)), p, kHalfPi);
}
__device__ __forceinline__ float atan2_poly(float y, float x)
{
    const float ax = fabsf(x), ay = fabsf(y);
    const float t = fminf(ax, ay) * __builtin_amdgcn_rcpf(fmaxf(fmaxf(ax, ay), 1e-30f)), t2 = t * t;
    float r = t * fmaf(t2, fmaf(t2, fmaf(t2, fmaf(t2, 0.02084509f, -0.0851563f), 0.18015926f), -0.33030478f), 0.99986633f);
    r = ay > ax ? kHalfPi - r : r;
    r = x < 0.0f ? 2.0f * kHalfPi - r : r;
    return y < 0.0f ? -r : r;
}

// Columns c in [0, n) with c0 + (c + 0.5) step in [a, b], both given in columns
// (less c0 and divided by the step); an empty range when none.  The products
// with an approximate 1 / step are off by less than 0.01 of a column (8192 of
// them, twice over); 0.02 is allowed for.
__device__ __forceinline__ void columns_between(float a, float b, int n, int* k0, int* k1)
{
    const int x0 = (int)ceilf(fmaxf(a - 0.52f, -1.0f)), x1 = (int)floorf(fminf(b - 0.48f, (float)n)) + 1;
    *k0 = max(x0, 0);
    *k1 = min(x1, n);
}

// Records leave through LDS as in the camera projection: a wave's 64 records
// (64 bytes each) are written to LDS and stored back lane-contiguously, so
// each store instruction writes 1 KB of consecutive records.  The image
// descriptions come in as a restrict argument (uniform reads become scalar
// loads).  Six waves per SIMD (80 registers; left alone the compiler takes 84,
// which makes five): 512 heightmaps 6.00 -> 5.92 ms, 64 rosette scans 1.61 ->
// 1.56, 512 scans of 32 x 1024 16.69 -> 16.56.  (The camera projection, at 125
// registers and four waves, spills at five: 256 image pairs 20.6 -> 22.2 ms.)
template <int ST>
__global__ __launch_bounds__(256, 6) void k_project_lidar(SceneDev s, ChunkDev c, const ImageInfo* __restrict__ imgs,
                                                          int ts, int ipt)
{
    __shared__ float4 stage[4][kLidarRec * 64];
    // the elevation table of the current angular image (up to kLdsBeams beams;
    // the row search reads it ten times per Gaussian), or a listed-ray image's
    // band tables, and its tiles' azimuth spans
    __shared__ float elev_s[kLdsBeams];
    __shared__ float taz_s[kLdsTileAz];
    float4* const st = stage[threadIdx.x >> 6];
    const uint32_t L = xcd_remap(blockIdx.x + blockIdx.y * gridDim.x, gridDim.x * gridDim.y);
    const uint32_t bx = L / gridDim.y, by = L - bx * gridDim.y;
    const int64_t g_lane = (int64_t)bx * 256 + threadIdx.x;
    // lanes past the last Gaussian stay (invisible) so that every record store slot of the wave has a lane
    const bool valid = g_lane < s.n;
    const int64_t g = valid ? g_lane : s.n - 1;
    const int lane = __lane_id();
    const int i_begin = (int)by * ipt;
    const int slot = body_slot(s, g);
    const float4 pm = s.pos[g];
    float q[4], sc[3];
    load_rot_scale<ST>(s, g, q, sc);
    float Rg[9];
    quat_rot(q[0], q[1], q[2], q[3], Rg);
    const float mu[3] = {pm.x, pm.y, pm.z};
    const float op = pm.w;
    const float log2o = log2f(op);
    const float rho = sqrtf(opacity_qmax(op)) * fmaxf(sc[0], fmaxf(sc[1], sc[2]));
    const float isc[3] = {1.0f / sc[0], 1.0f / sc[1], 1.0f / sc[2]};

    for (int ii = 0; ii < ipt; ++ii) {
        const int i = __builtin_amdgcn_readfirstlane(i_begin + ii);     // the same in every lane
        if (i >= c.n_img) break;
        const ImageInfo im = imgs[i];
        // block-uniform: every thread of the block projects into image i
        const int n_ev = im.kind == 3 ? 2 * im.height : im.height;
        const int n_taz = im.kind == 3 ? 2 * im.tiles_x * im.tiles_y : 0;
        const bool lds_elev = (im.kind == 1 || im.kind == 3) && n_ev <= kLdsBeams;
        const bool lds_taz = im.kind == 3 && n_taz <= kLdsTileAz;
        if (lds_elev || lds_taz) {
            __syncthreads();                    // the previous image's tables are no longer read
            if (lds_elev && (int)threadIdx.x < n_ev) elev_s[threadIdx.x] = im.elev[threadIdx.x];
            if (lds_taz)
                for (int k = (int)threadIdx.x; k < n_taz; k += 256) taz_s[k] = im.ray_tile_az[k];
            __syncthreads();
        }
        const float* ev = lds_elev ? elev_s : im.elev;
        const float* taz = lds_taz ? taz_s : im.ray_tile_az;
        const float* X = c.xform + ((size_t)i * (s.n_bodies + 1) + slot) * 16;
        float A[9];
#pragma unroll
        for (int k = 0; k < 9; ++k) A[k] = X[k];
        const float tx = ((A[0] * mu[0] + A[1] * mu[1]) + A[2] * mu[2]) + X[9];
        const float ty = ((A[3] * mu[0] + A[4] * mu[1]) + A[5] * mu[2]) + X[10];
        const float tz = ((A[6] * mu[0] + A[7] * mu[1]) + A[8] * mu[2]) + X[11];
        const bool grid = im.kind == 2;
        // key: centre distance (angular), depth of the centre below the sensor plane (grid)
        const float d2 = (tx * tx + ty * ty) + tz * tz;
        float D = grid ? (-tz > 0.0f ? -tz : 0.0f) : sqrt_rn(d2);
        if (!grid && __ballot(!(d2 > 0x1p-100f && d2 < 0x1p126f)) != 0ull) D = sqrtf(d2);
        const size_t o = (size_t)i * (size_t)s.n + (size_t)g;
        bool ok = valid && isfinite(tx) && isfinite(ty) && isfinite(tz) && op >= 1.0f / 255.0f && isfinite(D) &&
                  sc[0] > 0.0f && sc[1] > 0.0f && sc[2] > 0.0f;
        int r0 = 0, r1 = 0, c0 = 0, c1 = 0;
        float cone_c = -2.0f;                           // cosine of the cone half-angle; -2 = every direction
        float disc = 0.0f;                              // grid: footprint radius on the sensor plane
        if (grid) {
            // the alpha >= 1/255 ellipsoid lies in the sphere of radius rho: rays (which look
            // down from z = 0) can reach it only if it dips below the plane, and only inside
            // its footprint disc (widened against the rounding of the ray origins)
            ok = ok && tz < rho;
            disc = rho * 1.0001f + 1e-6f * ((((1.0f + fabsf(tx)) + fabsf(ty)) + fabsf(im.gx0)) + fabsf(im.gy0));
            if (ok) {
                const float ix = __builtin_amdgcn_rcpf(im.gdx), iy = __builtin_amdgcn_rcpf(im.gdy);
                columns_between(((tx - disc) - im.gx0) * ix, ((tx + disc) - im.gx0) * ix, im.width, &c0, &c1);
                columns_between(((ty - disc) - im.gy0) * iy, ((ty + disc) - im.gy0) * iy, im.height, &r0, &r1);
            }
        } else if ((ok = ok && D > 0.0f)) {
            if (D <= rho * 1.001f + 1e-6f) {            // the sensor may sit inside: every ray
                r0 = 0;
                r1 = im.height;
                c0 = 0;
                c1 = im.width;
            } else {
                // sine and cosine of the cone's half-angle (widened), of the centre's elevation and of their sum
                const float iD = rcp_rn(D);
                const float sa = fminf(1.0f, fmaf(rho * iD, 1.0002f, 4e-6f));
                const float ca = __builtin_amdgcn_sqrtf(fmaxf(0.0f, fmaf(-sa, sa, 1.0f)));
                const float se = fminf(1.0f, fabsf(tz) * iD);
                const float ce = __builtin_amdgcn_sqrtf(fmaxf(0.0f, fmaf(-se, se, 1.0f)));
                const float cs = fmaf(ce, ca, -se * sa);
                cone_c = ca;
                // towards the poles the elevation is as uncertain as se / ce
                const float ang = asin_poly(sa) + kAngleSlack + 5e-7f * __builtin_amdgcn_rcpf(fmaxf(ce, 5e-4f));
                const float el = copysignf(asin_poly(se), tz);
                // angular: rows with |elevation - el| <= ang; listed rays: bands whose [smallest, largest] meets that
                rows_between(im.kind == 3 ? ev + im.height : ev, ev, im.height, el - ang, el + ang, &r0, &r1);
                if (cs <= 0.02f) {                          // the cone reaches (almost) over the pole
                    c0 = 0;
                    c1 = im.width;
                } else {
                    const float daz = asin_poly(fminf(1.0f, fmaf(sa * 1.002f, __builtin_amdgcn_rcpf(cs), 1e-5f))) + 2.0f * kAngleSlack;
                    const float th = atan2_poly(ty, tx);
                    if (im.kind == 3) {
                        // per tile row of the bands, the ray tiles whose azimuth span
                        // [smallest, largest] meets the window, at each 2 pi shift that
                        // meets [-pi, pi]; the hull over the tile rows, in rays
                        const int TX = im.tiles_x, y0 = r0 / ts, y1 = (r1 + ts - 1) / ts;
                        const float* tmin = taz;
                        const float* tmax = taz + (size_t)TX * im.tiles_y;
                        int lo = TX, hi = 0;
                        for (int y = y0; y < y1; ++y) {
#pragma unroll
                            for (int k = -1; k <= 1; ++k) {
                                const float a0 = th - daz + (float)k * kTwoPi, a1 = th + daz + (float)k * kTwoPi;
                                if (a1 < -3.1416f || a0 > 3.1416f) continue;
                                const int a = first_at_least(tmax + (size_t)y * TX, TX, a0, false);   // largest >= a0
                                const int b = first_at_least(tmin + (size_t)y * TX, TX, a1, true);    // smallest <= a1
                                if (a < b) {
                                    lo = min(lo, a);
                                    hi = max(hi, b);
                                }
                            }
                        }
                        c0 = lo * ts;
                        c1 = min(im.width, hi * ts);
                    } else {
                        // the azimuth window, tested at its three 2 pi shifts; the hull of the hits
                        const float is = __builtin_amdgcn_rcpf(im.az_step), turn = kTwoPi * is;
                        const float wa = ((th - daz) - im.az0) * is, wb = ((th + daz) - im.az0) * is;
                        int lo = im.width, hi = 0;
#pragma unroll
                        for (int k = -1; k <= 1; ++k) {
                            int a, b;
                            columns_between(fmaf((float)k, turn, wa), fmaf((float)k, turn, wb), im.width, &a, &b);
                            if (a < b) {
                                lo = min(lo, a);
                                hi = max(hi, b);
                            }
                        }
                        c0 = lo;
                        c1 = hi;
                    }
                }
            }
        }
        const bool vis = ok && r1 > r0 && c1 > c0;
        if (valid) c.keyz[o] = vis ? __float_as_uint(D) : kInvalidKey;
        const uint64_t vmask = __ballot(vis);
        if (vmask == 0ull) continue;            // wave-uniform
        if (vis) {
            const int x0 = c0 / ts, x1 = (c1 + ts - 1) / ts, y0 = r0 / ts, y1 = (r1 + ts - 1) / ts;
            put_rect(c.rect, c.rect4, o, (uint32_t)x0, (uint32_t)x1, (uint32_t)y0, (uint32_t)y1);
            // whitening W = S^-1 (A Rg)^T: row k = (A Rg)[:, k] / s_k
            float Rs[9];
            mat3_mul(A, Rg, Rs);
            float W[9];
#pragma unroll
            for (int k = 0; k < 3; ++k)
#pragma unroll
                for (int j = 0; j < 3; ++j) W[3 * k + j] = Rs[3 * j + k] * isc[k];
            const float w0 = (W[0] * tx + W[1] * ty) + W[2] * tz;
            const float w1 = (W[3] * tx + W[4] * ty) + W[5] * tz;
            float4* r = st + kLidarRec * lane;
            r[0] = make_float4(W[0], W[1], W[2], tx);
            r[1] = make_float4(W[3], W[4], W[5], ty);
            r[2] = make_float4(W[6], W[7], W[8], tz);
            r[3] = make_float4(log2o, grid ? disc : cone_c, w0, w1);
        }
        wave_lds_sync();
        // float4 q of the wave's records belongs to lane q / kLidarRec
        float4* rec = c.rec + kLidarRec * ((size_t)i * (size_t)s.n + (size_t)(g_lane - lane));
#pragma unroll
        for (int k = 0; k < kLidarRec; ++k) {
            const int q = lane + 64 * k;
            if ((vmask >> (q / kLidarRec)) & 1ull) store_stream(rec + q, st[q]);
        }
        wave_lds_sync();
    }
}

// f(u, v) = f0 + 2 (b1 u + b2 v) + a11 u^2 + 2 a12 u v + a22 v^2.
struct Quad2 {
    float a11, a12, a22, b1, b2, f0;
};

// Whether f stays above `bound` on [u0, u1] x [v0, v1] (a sufficient test:
// false where f is not clearly convex).  A convex f has its minimum over the
// rectangle at its own minimum if that lies inside, else on an edge that faces
// it: one u edge and one v edge are evaluated, each at its clamped 1D minimum
// (where the minimum lies between u0 and u1 the u edge taken is just more of
// the rectangle).  An approximate reciprocal only moves the evaluated point
// along its edge, by a relative 1e-7: a second-order change of the value.
__device__ __forceinline__ bool above_on_rect(const Quad2& q, float u0, float u1, float v0, float v1, float bound)
{
    const float det = fmaf(q.a11, q.a22, -q.a12 * q.a12);
    const float id = __builtin_amdgcn_rcpf(det);
    const float uc = fmaf(q.b2, q.a12, -q.b1 * q.a22) * id, vc = fmaf(q.b1, q.a12, -q.b2 * q.a11) * id;
    const float ue = uc < u0 ? u0 : u1, ve = vc < v0 ? v0 : v1;
    const bool inside = uc >= u0 && uc <= u1 && vc >= v0 && vc <= v1;
    auto f = [&](float u, float v) {
        const float x = fmaf(q.a11, u, fmaf(2.0f * q.a12, v, 2.0f * q.b1));
        const float y = fmaf(q.a22, v, 2.0f * q.b2);
        return fmaf(u, x, fmaf(v, y, q.f0));
    };
    const float vu = fminf(fmaxf(-fmaf(q.a12, ue, q.b2) * __builtin_amdgcn_rcpf(q.a22), v0), v1);
    const float uv = fminf(fmaxf(-fmaf(q.a12, ve, q.b1) * __builtin_amdgcn_rcpf(q.a11), u0), u1);
    const float m = fminf(f(ue, vu), f(uv, ve));
    return q.a11 > 0.0f && q.a22 > 0.0f && det > 1e-5f * (q.a11 * q.a22) && !inside && m > bound;
}

__device__ __forceinline__ float dot3(const float a[3], const float b[3])
{
    return fmaf(a[2], b[2], fmaf(a[1], b[1], a[0] * b[0]));
}

__device__ __forceinline__ float lane_value(float x, int lane)
{
    return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(x), lane));
}

// Smallest and largest x over the lanes with `on` set (the same in every lane).
__device__ __forceinline__ void wave_range(float x, bool on, float* lo, float* hi)
{
    float a = on ? x : 3.0e38f, b = on ? x : -3.0e38f;
#pragma unroll
    for (int m = 1; m < 64; m <<= 1) {
        a = fminf(a, __shfl_xor(a, m, 64));
        b = fmaxf(b, __shfl_xor(b, m, 64));
    }
    *lo = a;
    *hi = b;
}

// One workgroup per TS x TS tile of rays; batches of kLBatch records in LDS.
// Culling in three steps.  First the bound stored in the record.
// Angular rays: the wave bounds its rays by a cone (axis = their normalised
// mean direction, half-angle beta = the widest ray), and a Gaussian stays when
// its own cone (half-angle alpha around its centre direction, as used for the
// tile rectangle) comes within alpha + beta of that axis.  Grid rays: the
// wave's ray origins span a rectangle of the sensor plane, and a Gaussian
// stays when its footprint disc reaches it.  Those bounds come from the sphere
// around the Gaussian; the batch's survivors are packed, 64 to a group, and
// each lane then tests one of them with its own ellipsoid: the rays are points
// (u, v) of a rectangle (the plane tangent to the axis; the sensor plane), and
// on it
//     angular: (|c|^2 - Q) |W d|^2 - (c . W d)^2,   d = w + u e1 + v e2, c = W t
//     grid:    (|r|^2 - Q) |a|^2 - (r . a)^2,       r = c - u W ex - v W ey, a = W d
// is a quadratic in (u, v) that is <= 0 exactly where q <= Q, Q the value at
// which alpha falls to 1/255.  A Gaussian whose quadratic stays above a bound
// for its rounding on the rectangle of the live rays is taken by none of them.
// Third, each ray evaluates the quadratics of the survivors at its own (u, v),
// five multiply-adds each, into a mask, 32 survivors to a word, and evaluates
// only those of its mask: the rays of a wave walk different survivors side by
// side, each reading its own from LDS.  What is evaluated in full costs 33
// vector instructions (48 with its blending) and four 16-byte LDS reads.
// A 16 x 4 ray wave of a 32 x 1024 scan over 300k Gaussians of 0.03 m walks
// 2900 candidates: the first step leaves 759, the second 346, the third 87 per
// ray, of which 64 are taken; the longest mask of each word adds up to 167, for
// which the lanes evaluate together.  (A heightmap's wave: 2252, 1224, 87, 62
// and 349; a rosette's: 336, 140, 83, 60 and 93.)  Before, each quarter of a
// wave walked the survivors of its own rectangle, about 300 in a scan.  Times of
// when each step came in: 512 scans 17.5 -> 17.1 ms with the third step, 512 heightmaps of 64 x 64 rays
// 7.5 -> 7.1 ms, 64 rosette scans of 24,576 rays 2.55 -> 2.20 ms; without any
// but the first 26.7, 16.2 and 10.3 ms.  Measured and no faster: waves without
// shared staging (17.1, 7.7, 2.18 ms: four times the reads miss L2, 18.7 GB
// instead of 8.8 a pass), survivors kept in two halves so that a ray may lag
// (18.1, 7.9, 2.4 ms), masks of 96 survivors (18.9, 7.8, 2.3 ms).
template <int TS>
struct LidarLds {
    float4 sr[kLidarStage][TS * TS];
    uint32_t live_w[2][TS * TS / 64];     // per wave: live rays left after a batch (by batch parity)
    uint8_t pick[TS * TS / 64][TS * TS];        // per wave: the batch's candidates that the first step keeps
    // those the second step keeps: their quadratics less the bound, a11, 2 a12,
    // a22, 2 b1, 2 b2, f0 - bound; the third step reads them 16 bytes at a time
    alignas(16) float quad[TS * TS / 64][64 * 6];
    uint8_t surv[TS * TS / 64][64];             // and their places in the batch
};

// Launches of short lists (kShortList) take the first step only, and a wave's rays
// walk its survivors together: what a tile costs there is what it sets up, and how
// many others its CU holds beside it (7 workgroups of 48 registers and 20 KB a
// tile, 5 of 93 and 28 KB with all three steps).
template <int TS>
struct LidarShortLds {
    float4 sr[kLidarStage][TS * TS];
    uint32_t live_w[2][TS * TS / 64];
};

// m = 2 m + (f > 0 ? 0 : 1) for f0, then for f1.  A vector instruction that
// reads a mask which a vector instruction has written must follow it by two wait
// states on this GPU, and the compiler inserts none inside inline assembly: the
// two compares and one s_nop stand between each compare and its add.
__device__ __forceinline__ void shift_in(uint32_t& m, float f0, float f1)
{
    uint64_t c1;
    asm("v_cmp_nlt_f32 vcc, 0, %2\n\t"
        "v_cmp_nlt_f32 %1, 0, %3\n\t"
        "s_nop 0\n\t"
        "v_addc_co_u32 %0, vcc, %0, %0, vcc\n\t"
        "v_addc_co_u32 %0, vcc, %0, %0, %1"
        : "+v"(m), "=&s"(c1)
        : "v"(f0), "v"(f1)
        : "vcc");
}

template <int TS, bool GRID, bool SHORT, class Lds>
__device__ __forceinline__ void lidar_tile(const SceneDev& s, const ChunkDev& c, int i, const ImageInfo& im, int tx,
                                           int ty, uint32_t t, Lds& L_)
{
    constexpr int NT = TS * TS;
    constexpr int kLBatch = NT;
    auto& sr = L_.sr;
    auto& live_w = L_.live_w;
    const int tid = threadIdx.x, lane = __lane_id();
    // a wave's rays: 16 x 4 of a 16 x 16 tile (8 x 8 of an 8 x 8 one), each quarter of the lanes 8 x 2 of them
    const int quarter = lane >> 4;
    const int col = tx * TS + (lane & 7) + (TS == 16 ? 8 * (quarter & 1) : 0);
    const int row = ty * TS + ((lane >> 3) & 1) + (TS == 16 ? 4 * (tid >> 6) + 2 * (quarter >> 1) : 2 * quarter);
    const bool inside = col < im.width && row < im.height;
    // ray: origin o (grid; the sensor origin otherwise) and direction d
    float d[3] = {0.0f, 0.0f, GRID ? -1.0f : 0.0f};
    float ox = 0.0f, oy = 0.0f;
    if (GRID) {
        ox = im.gx0 + ((float)col + 0.5f) * im.gdx;
        oy = im.gy0 + ((float)row + 0.5f) * im.gdy;
    } else if (inside) {
        float az, el;
        if (im.kind == 3) {
            az = im.ray_az[(size_t)row * im.width + col];
            el = im.ray_el[(size_t)row * im.width + col];
        } else {
            az = im.az0 + ((float)col + 0.5f) * im.az_step;
            el = im.elev[row];
        }
        float sa, ca, se, ce;
        sincosf(az, &sa, &ca);
        sincosf(el, &se, &ce);
        d[0] = ce * ca;
        d[1] = ce * sa;
        d[2] = se;
    }
    // the wave's bound: a cone (angular; culling off when wider than 90 degrees) or the
    // rectangle of its ray origins (grid)
    float w[3] = {d[0], d[1], d[2]};
    bool cull = true;
    float cb = 1.0f, sb = 0.0f;
    float bx0 = 0.0f, bx1 = 0.0f, by0 = 0.0f, by1 = 0.0f;
    // this ray's point (u, v) for the second step, and the basis of the tangent plane
    float ru = ox, rv = oy;
    float e1[3] = {1.0f, 0.0f, 0.0f}, e2[3] = {0.0f, 1.0f, 0.0f};
    if (GRID) {
        wave_range(ox, inside, &bx0, &bx1);
        wave_range(oy, inside, &by0, &by1);
    } else {
#pragma unroll
        for (int m = 1; m < 64; m <<= 1)
#pragma unroll
            for (int k = 0; k < 3; ++k) w[k] += __shfl_xor(w[k], m, 64);
        const float wn = sqrtf(w[0] * w[0] + w[1] * w[1] + w[2] * w[2]);
        cull = wn > 0.0f;
        if (cull)
#pragma unroll
            for (int k = 0; k < 3; ++k) w[k] /= wn;
        cb = inside ? d[0] * w[0] + d[1] * w[1] + d[2] * w[2] : 1.0f;
#pragma unroll
        for (int m = 1; m < 64; m <<= 1) cb = fminf(cb, __shfl_xor(cb, m, 64));
        cb = cb - 1e-5f;                              // rounding of the directions and of the axis
        cull = cull && cb > 0.0f;
        sb = sqrtf(fmaxf(0.0f, 1.0f - cb * cb));
        // e1 horizontal where the axis is not steep, e2 = w x e1
        const bool steep = fabsf(w[2]) > 0.9f;
        e1[0] = steep ? 0.0f : -w[1];
        e1[1] = steep ? -w[2] : w[0];
        e1[2] = steep ? w[1] : 0.0f;
        const float en = __builtin_amdgcn_rsqf(dot3(e1, e1));
#pragma unroll
        for (int k = 0; k < 3; ++k) e1[k] *= en;
        e2[0] = w[1] * e1[2] - w[2] * e1[1];
        e2[1] = w[2] * e1[0] - w[0] * e1[2];
        e2[2] = w[0] * e1[1] - w[1] * e1[0];
        const float dw = __builtin_amdgcn_rcpf(dot3(d, w));
        ru = dot3(d, e1) * dw;
        rv = dot3(d, e2) * dw;
    }
    // the rectangle of the live rays' points, taken again whenever a quarter of
    // them have stopped; the second step needs rays within about 45 degrees of
    // the axis.  Waves of wider rays (a 16 x 64 scan) skip it and the third, whose
    // masks would hold everything: 64 such scans over 100k Gaussians 2.14 ms, 2.71
    // with a mask of all survivors for every ray
    float u0, u1, v0, v1;
    const bool tight = !SHORT && (GRID || (cull && cb > 0.75f));
    auto live_rect = [&](bool on) {
        float r[4] = {on ? ru : 3.0e38f, on ? -ru : 3.0e38f, on ? rv : 3.0e38f, on ? -rv : 3.0e38f};
#pragma unroll
        for (int k = 0; k < 4; ++k) {
#pragma unroll
            for (int m = 1; m < 64; m <<= 1) r[k] = fminf(r[k], __shfl_xor(r[k], m, 64));
        }
        const float pu = 4e-6f * (1.0f + fmaxf(fabsf(r[0]), fabsf(r[1])));
        const float pv = 4e-6f * (1.0f + fmaxf(fabsf(r[2]), fabsf(r[3])));
        u0 = lane_value(r[0] - pu, 0);
        u1 = lane_value(pu - r[1], 0);
        v0 = lane_value(r[2] - pv, 0);
        v1 = lane_value(pv - r[3], 0);
    };
    const float uu = ru * ru, uv = ru * rv, vv = rv * rv;

    const float um = fmaxf(fabsf(bx0), fabsf(bx1)), vm = fmaxf(fabsf(by0), fabsf(by1));     // grid: largest |u|, |v|
    bool live = inside;
    uint32_t rect_rays = (uint32_t)__popcll(__ballot(live));
    uint8_t *pick = nullptr, *surv = nullptr;
    float* quad = nullptr;
    if constexpr (!SHORT) {
        live_rect(live);
        pick = L_.pick[tid >> 6];
        quad = L_.quad[tid >> 6];
        surv = L_.surv[tid >> 6];
        surv[lane] = 0;                 // every slot holds a place of the batch, also beyond the survivors so far
    }
    float T = 1.0f, Rg = 0.0f;
    // returns at t* <= reach are not taken: the sensor's near range, infinity once the ray has stopped
    float reach = inside ? im.near_plane : INFINITY;
    const uint32_t* R = c.tile_range + ((size_t)i * c.t_max + t) * 2;
    const uint32_t start = R[0], end = R[1];
    const uint32_t* list = c.pairs + c.pair_base[i];
    const float4* rec = c.rec + (size_t)i * (size_t)s.n * kLidarRec;
    const uint32_t n = (uint32_t)s.n;
    bool wave_live = __ballot(live) != 0ull;
    bool bad_entry = false;
    int par = 0;
    // ids are read one batch ahead, and a batch's records before the barrier
    // that frees the staged ones: both reads pass while other waves still work
    uint32_t gid = start + (uint32_t)tid < end ? list[start + (uint32_t)tid] : 0u;
    for (uint32_t b0 = start; b0 < end; b0 += kLBatch, par ^= 1) {
        float4 rr[kLidarRec];
        {
            uint32_t g = gid;
            if (b0 + (uint32_t)tid < end && g >= n) {       // impossible by construction: reported at the end, a
                bad_entry = true;                           // valid record read
                g = 0;
            }
#pragma unroll
            for (int k = 0; k < kLidarRec; ++k) rr[k] = rec[kLidarRec * (size_t)g + k];
            const uint32_t e = b0 + (uint32_t)(kLBatch + tid);
            gid = e < end ? list[e] : 0u;
        }
        __syncthreads();
        // every wave's flag from the previous batch is visible after the
        // barrier, so all waves take the same decision
        if (b0 != start) {
            uint32_t any = 0;
#pragma unroll
            for (int ww = 0; ww < NT / 64; ++ww) any |= live_w[par ^ 1][ww];
            if (!any) break;
        }
        {
            const float4 m0 = rr[0], m1 = rr[1], m2 = rr[2], m3 = rr[3];
            sr[0][tid] = m0;
            sr[1][tid] = m1;
            sr[2][tid] = m2;
            // the last of W t, rounded as the projection rounds the others
            sr[3][tid] = make_float4(m3.x, m3.z, m3.w, (m2.x * m0.w + m2.y * m1.w) + m2.z * m2.w);
            if (GRID) {
                // every ray's direction is (0, 0, -1): W d = -(third column of W), the same for all of them
                sr[4][tid] = make_float4(m0.w, m1.w, m3.y,
                                         __builtin_amdgcn_rcpf(fmaf(m2.z, m2.z, fmaf(m1.z, m1.z, m0.z * m0.z))));
            } else {
                const float iD = __builtin_amdgcn_rsqf(fmaf(m2.w, m2.w, fmaf(m1.w, m1.w, m0.w * m0.w)));
                sr[4][tid] = make_float4(m0.w * iD, m1.w * iD, m2.w * iD, m3.y);
            }
        }
        __syncthreads();
        const int cnt = (int)min((uint32_t)kLBatch, end - b0);
        auto eval = [&](int j, float* ts_out, float* la_out) {
            const float4 m0 = sr[0][j], m1 = sr[1][j], m2 = sr[2][j], m3 = sr[3][j];
            float tstar, px, py, pz;
            if (GRID) {
                // centre relative to the ray origin, and W times it
                px = m0.w - ox;
                py = m1.w - oy;
                const float wcx = m3.y - fmaf(m0.y, oy, m0.x * ox);
                const float wcy = m3.z - fmaf(m1.y, oy, m1.x * ox);
                const float wcz = m3.w - fmaf(m2.y, oy, m2.x * ox);
                tstar = fmaf(-m2.z, wcz, fmaf(-m1.z, wcy, -m0.z * wcx)) * sr[4][j].w;
                pz = m2.w + tstar;
            } else {
                // d' = W d
                const float dx = fmaf(m0.z, d[2], fmaf(m0.y, d[1], m0.x * d[0]));
                const float dy = fmaf(m1.z, d[2], fmaf(m1.y, d[1], m1.x * d[0]));
                const float dz = fmaf(m2.z, d[2], fmaf(m2.y, d[1], m2.x * d[0]));
                const float aa = fmaf(dz, dz, fmaf(dy, dy, dx * dx));
                const float bb = fmaf(dz, m3.w, fmaf(dy, m3.z, dx * m3.y));
                tstar = bb * __builtin_amdgcn_rcpf(aa);
                // offset of the centre from the ray's closest point, in metres
                px = fmaf(-tstar, d[0], m0.w);
                py = fmaf(-tstar, d[1], m1.w);
                pz = fmaf(-tstar, d[2], m2.w);
            }
            // the offset whitened
            const float wx = fmaf(m0.z, pz, fmaf(m0.y, py, m0.x * px));
            const float wy = fmaf(m1.z, pz, fmaf(m1.y, py, m1.x * px));
            const float wz = fmaf(m2.z, pz, fmaf(m2.y, py, m2.x * px));
            const float qq = fmaf(wz, wz, fmaf(wy, wy, wx * wx));
            *ts_out = tstar;
            *la_out = fmaf(-0.72134752044448170f, qq, m3.x);      // log2 o - q/2 log2 e
        };
        auto take = [&](float tstar, float la) {
            if (tstar > reach && la >= kLidarLogAlphaMin) {
                // only the rays that take the Gaussian run this (exec mask);
                // the empty asm keeps it a branch rather than selects
                asm volatile("");
                const float alpha = fminf(0.99f, __builtin_amdgcn_exp2f(la));
                const float Tn = fmaf(-T, alpha, T);
                const bool stop = Tn < 1e-4f;           // stops here, adds nothing
                Rg = stop ? Rg : fmaf(tstar, alpha * T, Rg);
                T = stop ? T : Tn;
                reach = stop ? INFINITY : reach;
            }
        };
        uint32_t n_pick = 0;
        for (int sub = 0; sub < cnt && wave_live; sub += 64) {
            const int jl = sub + lane;
            bool keep = false;
            if (jl < cnt) {
                const float4 cn = sr[4][jl];
                if (GRID) {
                    // distance from the footprint centre to the origin rectangle, against the disc radius
                    const float ex = fmaxf(0.0f, fmaxf(bx0 - cn.x, cn.x - bx1));
                    const float ey = fmaxf(0.0f, fmaxf(by0 - cn.y, cn.y - by1));
                    keep = ex * ex + ey * ey <= cn.z * cn.z * 1.0001f;
                } else if (!cull || cn.w < -1.5f) {
                    keep = true;
                } else {
                    const float sa = __builtin_amdgcn_sqrtf(fmaxf(0.0f, fmaf(-cn.w, cn.w, 1.0f)));
                    keep = fmaf(cn.z, w[2], fmaf(cn.y, w[1], cn.x * w[0])) >= fmaf(cn.w, cb, -sa * sb) - 2e-6f;
                }
            }
            const uint64_t kept = __ballot(keep);
            if (!tight) {               // the rays walk what the first step keeps together
                for (uint64_t m = kept; m != 0ull;) {
                    const int j0 = sub + __builtin_ctzll(m);
                    m &= m - 1;
                    const bool two = m != 0ull;
                    const int j1 = two ? sub + __builtin_ctzll(m) : j0;
                    m &= m - 1;         // (zero stays zero)
                    float t0, l0, t1, l1;
                    eval(j0, &t0, &l0);
                    eval(j1, &t1, &l1);
                    l1 = two ? l1 : -INFINITY;
                    asm volatile("" : "+v"(t0), "+v"(l0), "+v"(t1), "+v"(l1));      // two independent chains, as below
                    take(t0, l0);
                    take(t1, l1);
                }
                wave_live = __ballot(reach < INFINITY) != 0ull;
            } else if constexpr (!SHORT) {
                if (keep) pick[n_pick + lanes_below(kept)] = (uint8_t)jl;
                n_pick += (uint32_t)__popcll(kept);
            }
        }
        wave_lds_sync();
        const uint64_t live_m = __ballot(live);
        if (tight && 4u * (uint32_t)__popcll(live_m) <= 3u * rect_rays) {
            rect_rays = (uint32_t)__popcll(live_m);
            live_rect(live);
        }
        for (uint32_t p0 = 0; p0 < n_pick && wave_live; p0 += 64) {
            const bool have = p0 + (uint32_t)lane < n_pick;
            const int jp = have ? (int)pick[p0 + (uint32_t)lane] : 0;
            Quad2 qd;
            float bound;
            const float4 m0 = sr[0][jp], m1 = sr[1][jp], m2 = sr[2][jp], m3 = sr[3][jp];
            auto whiten = [&](const float x[3], float y[3]) {
                y[0] = fmaf(m0.z, x[2], fmaf(m0.y, x[1], m0.x * x[0]));
                y[1] = fmaf(m1.z, x[2], fmaf(m1.y, x[1], m1.x * x[0]));
                y[2] = fmaf(m2.z, x[2], fmaf(m2.y, x[1], m2.x * x[0]));
            };
            const float cw[3] = {m3.y, m3.z, m3.w};
            const float cc = dot3(cw, cw);
            // q at which log2 alpha = log2(1/255), with a margin for the rays' own rounding
            const float Q = fmaf(1.3862944f * 1.002f, m3.x - kLidarLogAlphaMin, 0.01f);
            float a0[3], a1[3], a2[3];
            if (GRID) {
#pragma unroll
                for (int k = 0; k < 3; ++k) {
                    a0[k] = k == 0 ? -m0.z : k == 1 ? -m1.z : -m2.z;      // W d, d = (0, 0, -1)
                    a1[k] = k == 0 ? m0.x : k == 1 ? m1.x : m2.x;
                    a2[k] = k == 0 ? m0.y : k == 1 ? m1.y : m2.y;
                }
                const float aa = dot3(a0, a0), g1 = dot3(a1, a0), g2 = dot3(a2, a0), gc = dot3(cw, a0);
                const float n1 = dot3(a1, a1), n2 = dot3(a2, a2);
                qd.a11 = fmaf(n1, aa, -g1 * g1);
                qd.a12 = fmaf(dot3(a1, a2), aa, -g1 * g2);
                qd.a22 = fmaf(n2, aa, -g2 * g2);
                qd.b1 = fmaf(gc, g1, -dot3(cw, a1) * aa);
                qd.b2 = fmaf(gc, g2, -dot3(cw, a2) * aa);
                qd.f0 = fmaf(cc - Q, aa, -gc * gc);
                bound = 2e-6f * aa * (cc + n1 * um * um + n2 * vm * vm);
            } else {
                whiten(w, a0);
                whiten(e1, a1);
                whiten(e2, a2);
                const float k = cc - Q, h0 = dot3(cw, a0), h1 = dot3(cw, a1), h2 = dot3(cw, a2);
                const float n0 = dot3(a0, a0), n1 = dot3(a1, a1), n2 = dot3(a2, a2);
                qd.a11 = fmaf(k, n1, -h1 * h1);
                qd.a12 = fmaf(k, dot3(a1, a2), -h1 * h2);
                qd.a22 = fmaf(k, n2, -h2 * h2);
                qd.b1 = fmaf(k, dot3(a0, a1), -h0 * h1);
                qd.b2 = fmaf(k, dot3(a0, a2), -h0 * h2);
                qd.f0 = fmaf(k, n0, -h0 * h0);
                // f's own rounding, below 2e-6, and that of the rays' (u, v), which moves a direction by
                // 1.3e-6 and f where it is near 0 by at most 3.5e-6 sqrt(Q / |c|^2) of the same product
                bound = cc > 2.0f * Q ? 5e-6f * cc * (n0 + n1 + n2) : INFINITY;      // the sensor well outside
            }
            const bool keep = have && !above_on_rect(qd, u0, u1, v0, v1, bound);
            const uint64_t kept = __ballot(keep);
            const uint32_t n_s = (uint32_t)__popcll(kept);
            if (keep) {
                const uint32_t r = lanes_below(kept);
                float2* qp = reinterpret_cast<float2*>(&quad[6u * r]);
                qp[0] = make_float2(qd.a11, 2.0f * qd.a12);
                qp[1] = make_float2(qd.a22, 2.0f * qd.b1);
                qp[2] = make_float2(2.0f * qd.b2, qd.f0 - bound);
                surv[r] = (uint8_t)jp;
            }
            wave_lds_sync();
            // third step: each ray evaluates the quadratics at its own point
            // and walks those that do not stay above the bound there
            for (uint32_t s0 = 0; s0 < n_s; s0 += 32u) {
                const uint32_t some = min(32u, n_s - s0);
                uint32_t mask = 0;
                for (uint32_t k = (some + 1u) & ~1u; k != 0u; k -= 2u) {
                    const float4* qp = reinterpret_cast<const float4*>(&quad[6u * (s0 + k - 2u)]);
                    const float4 q0 = qp[0], q1 = qp[1], q2 = qp[2];
                    const float fa = fmaf(q0.x, uu, fmaf(q0.y, uv, fmaf(q0.z, vv, fmaf(q0.w, ru, fmaf(q1.x, rv, q1.y)))));
                    const float fb = fmaf(q1.z, uu, fmaf(q1.w, uv, fmaf(q2.x, vv, fmaf(q2.y, ru, fmaf(q2.z, rv, q2.w)))));
                    shift_in(mask, fb, fa);
                }
                // (an odd count's last pair holds one of an earlier group)
                mask &= some == 32u ? 0xFFFFFFFFu : (1u << some) - 1u;
                if (!(reach < INFINITY)) mask = 0u;
                // two at a time: both are evaluated (independent dependency
                // chains the wave interleaves), then composited in list order
                auto next = [&]() {             // place of the lowest of the mask in the batch
                    // (an empty mask gives some place of the batch: it is read and not used)
                    const uint32_t j = s0 + lowest_bit(mask);
                    mask &= mask - 1u;
                    return (int)surv[j];
                };
                bool a_on = mask != 0u;
                int ja = next();
                bool b_on = mask != 0u;
                int jb = next();
                while (a_on) {
                    const int j0 = ja, j1 = jb;
                    const bool two = b_on;
                    a_on = mask != 0u;
                    ja = next();
                    b_on = mask != 0u;
                    jb = next();
                    float t0, l0, t1, l1;
                    eval(j0, &t0, &l0);
                    eval(j1, &t1, &l1);
                    l1 = two ? l1 : -INFINITY;
                    // both are complete before the first is taken: two independent chains
                    asm volatile("" : "+v"(t0), "+v"(l0), "+v"(t1), "+v"(l1));
                    take(t0, l0);
                    take(t1, l1);
                }
            }
            wave_lds_sync();
        }
        live = reach < INFINITY;
        if (__ballot(live) == 0ull) wave_live = false;
        if (lane == 0) live_w[par][tid >> 6] = wave_live ? 1u : 0u;
    }
    if (bad_entry) atomicOr(c.err, kErrListEntry);
    if (inside) {
        // listed rays leave in the caller's order
        const size_t pix = im.kind == 3 ? (size_t)im.ray_perm[(size_t)row * im.width + col]
                                        : (size_t)row * im.width + col;
        im.out_depth[pix] = T < 1.0f ? Rg / (1.0f - T) : 0.0f;
        if (im.out_alpha) im.out_alpha[pix] = 1.0f - T;
    }
}

template <int TS, bool SHORT>
__global__ __launch_bounds__(TS * TS) void k_raster_lidar(SceneDev s, ChunkDev c, RasterParams p)
{
    __shared__ std::conditional_t<SHORT, LidarShortLds<TS>, LidarLds<TS>> lds;
    int i;
    uint32_t t;
    tile_of_block(p, blockIdx.x, &i, &t);
    const ImageInfo im = c.img[i];
    const int tx = (int)(t % (uint32_t)im.tiles_x);
    const int ty = (int)(t / (uint32_t)im.tiles_x);
    if (im.kind == 2) lidar_tile<TS, true, SHORT>(s, c, i, im, tx, ty, t, lds);     // workgroup-uniform
    else lidar_tile<TS, false, SHORT>(s, c, i, im, tx, ty, t, lds);
}

template <int ST>
hipError_t project_lidar_st(const SceneDev& s, const ChunkDev& c, int ts, int ipt, hipStream_t st)
{
    const dim3 grid((unsigned)((s.n + 255) / 256), (unsigned)((c.n_img + ipt - 1) / ipt));
    hipLaunchKernelGGL((k_project_lidar<ST>), grid, dim3(256), 0, st, s, c, c.img, ts, ipt);
    return hipGetLastError();
}

template <int TS, bool SHORT>
hipError_t launch_lidar(const SceneDev& s, const ChunkDev& c, const RasterParams& p, hipStream_t stream)
{
    hipLaunchKernelGGL((k_raster_lidar<TS, SHORT>), dim3(p.n_blocks), dim3(TS * TS), 0, stream, s, c, p);
    return hipGetLastError();
}

}  // namespace

hipError_t launch_project_lidar(const SceneDev& s, const ChunkDev& c, int ts, int ipt, hipStream_t stream)
{
    if (s.n == 0 || c.n_img == 0) return hipSuccess;
    ipt = std::max(1, std::min(ipt, c.n_img / 32));     // small chunks: more threads, fewer images each
    if (s.storage == kF16) return project_lidar_st<kF16>(s, c, ts, ipt, stream);
    if (s.storage == kBF16) return project_lidar_st<kBF16>(s, c, ts, ipt, stream);
    return project_lidar_st<kF32>(s, c, ts, ipt, stream);
}

hipError_t launch_raster_lidar(const SceneDev& s, const ChunkDev& c, const RasterParams& p, hipStream_t stream)
{
    if (p.n_blocks == 0) return hipSuccess;
    const bool few = p.n_blocks > kOrderTilesMin && short_lists(p.entries, p.n_blocks) && p.longest <= kShortLongest;
    if (p.ts == 8) return few ? launch_lidar<8, true>(s, c, p, stream) : launch_lidar<8, false>(s, c, p, stream);
    if (p.ts == 16) return few ? launch_lidar<16, true>(s, c, p, stream) : launch_lidar<16, false>(s, c, p, stream);
    return hipErrorInvalidValue;                // 32 x 32 ray tiles exceed the workgroup size
}

}  // namespace gsr
