// Capture: rasterize every triangle into per-pixel (PPFL) or per-octant
// (POFL) fragment lists (Sec. 3.1 "Simple Layout" / "Octree Layout",
// Sec. 3.2 FHV_PPFL / FHV_POFL).
//
// Kernels, in stream order:
//   fills     head <- 0xFFFFFFFF, counter <- 0
//   k_setup   one thread per triangle: fixed-point vertices (PPFL: viewport
//             transform; POFL: grid snap, exact integer normal, octahedral
//             packing, tangent frame of the packed normal, projection),
//             orientation, sample bounding box, number of sample tiles of
//             64 samples (8x8, 16x4 or 32x2, a launch choice), edge
//             functions and attributes as linear forms of the sample
//   scan      inclusive prefix sum of tiles per triangle
//   k_raster  work items are (triangle, tile) pairs; a wave takes a
//             contiguous range of them and processes one tile at a time, one
//             lane per sample: integer edge functions with the top-left
//             rule, integer attribute interpolation, list append
//
// List append (Sec. 3.2): the waves count their ranges' covered samples and
// a workgroup reserves their slots with one atomic add on the global counter
// (instead of one increment per fragment; the slots are the same set). Each lane with
// a slot below the capacity swaps its index into the key's head and stores
// {w0, rgba, normal, previous head} plus the key sidecar. Without a head
// array (batches that only want arrays) the exchange is skipped and the
// link is 0xFFFFFFFF.
//
// The fp64 setup relies on IEEE-correct add, mul, div, sqrt and rint and on
// no contraction into fused multiply-adds (built with -ffp-contract=off):
// the tangent frame is then reproducible operation by operation.
#include <math.h>

#include <algorithm>

#include "fhv_common.h"

namespace fhv {

namespace {

__device__ __forceinline__ int32_t round_snorm(int64_t num, int64_t l1)
{
    const int64_t a = num < 0 ? -num : num;
    const int64_t q = (2 * 32767 * a + l1) / (2 * l1);
    return (int32_t)(num < 0 ? -q : q);
}

// Exact octahedral packing of an integer normal (Cigolle et al. 2014):
// n / |n|_1 folded when n_z < 0, components rounded to multiples of
// 1/32767 with halves away from zero; int16 x | int16 y << 16.
__device__ uint32_t oct_pack(int64_t nx, int64_t ny, int64_t nz)
{
    const int64_t ax = nx < 0 ? -nx : nx, ay = ny < 0 ? -ny : ny, az = nz < 0 ? -nz : nz;
    const int64_t l1 = ax + ay + az;
    if (l1 == 0) return 0;
    int32_t qx, qy;
    if (nz >= 0) {
        qx = round_snorm(nx, l1);
        qy = round_snorm(ny, l1);
    } else {
        qx = round_snorm(nx < 0 ? -(l1 - ay) : (l1 - ay), l1);
        qy = round_snorm(ny < 0 ? -(l1 - ax) : (l1 - ax), l1);
    }
    return (uint32_t)(uint16_t)(int16_t)qx | ((uint32_t)(uint16_t)(int16_t)qy << 16);
}

// Tangent (t) and bitangent (b) of the unit normal decoded from a packed
// normal; basis of Duff et al. (JCGT 2017), t x b = n.
__device__ void tangent_frame(uint32_t nrm, double t[3], double b[3])
{
    double px = (double)(int16_t)(nrm & 0xFFFFu) / 32767.0;
    double py = (double)(int16_t)(nrm >> 16) / 32767.0;
    double pz = 1.0 - fabs(px) - fabs(py);
    if (pz < 0.0) {
        const double tx = (1.0 - fabs(py)) * (px >= 0.0 ? 1.0 : -1.0);
        const double ty = (1.0 - fabs(px)) * (py >= 0.0 ? 1.0 : -1.0);
        px = tx;
        py = ty;
    }
    const double len = sqrt(px * px + py * py + pz * pz);
    const double nx = px / len, ny = py / len, nz = pz / len;
    const double s = copysign(1.0, nz);
    const double a = -1.0 / (s + nz);
    const double c = nx * ny * a;
    t[0] = 1.0 + s * nx * nx * a;
    t[1] = s * c;
    t[2] = -s * nx;
    b[0] = c;
    b[1] = s + ny * ny * a;
    b[2] = -ny;
}

template <class T>
__device__ __forceinline__ void swap2(T (&v)[3])
{
    const T t = v[1];
    v[1] = v[2];
    v[2] = t;
}

// Sample index range covered by [lo, hi] in 16.8 units: samples sit at
// 256 i + 128, so the first is ceil((lo - 128) / 256), the last
// floor((hi - 128) / 256) (arithmetic shifts round towards -inf).
__device__ __forceinline__ void sample_range(int64_t lo, int64_t hi, int32_t* i0, int32_t* i1)
{
    *i0 = (int32_t)((lo - 128 + 255) >> 8);
    *i1 = (int32_t)((hi - 128) >> 8);
}

// The linear forms of a narrow triangle. Twice the
// area of any triangle inside the box is at most W H <= 2^30, which bounds the
// edge functions at the samples of the box; at a covered sample they lie in
// [0, A] and sum to A, so with attribute values below 2^m the numerator's
// terms stay below 2^(31 + m), exact in a double for colours (m = 8) and grid
// positions (m <= 19). c carries half the area (rounding), the edges' missing
// ones and 1/2: the numerator then lies at least 1/2 from a multiple of A, so
// that the quotient estimated with the rounded 1 / A (off by less than
// 2^-52 of it) has the right floor while A times the quotient is below 2^50.
// Depths (m = 24) keep that bound for A < 2^26; above it the quotient is off
// by at most one and kTriDepth32 has the remainder's terms (below 2^31 in
// magnitude for A <= 2^30, hence right modulo 2^32). Returns the flags.
__device__ __forceinline__ uint32_t narrow_forms(TriRec& r, const int64_t X[3], const int64_t Y[3],
                                                 const int32_t a[3][3], const uint32_t col[3], int64_t A,
                                                 uint32_t mode)
{
    const int64_t px = 256 * (int64_t)r.h.lo_i + 128, py = 256 * (int64_t)r.h.lo_j + 128;
    int32_t miss[3];   // one where the edge does not own its samples
#pragma unroll
    for (int e = 0; e < 3; ++e) {
        const int p = e, q = (e + 1) % 3;
        const int64_t dx = X[q] - X[p], dy = Y[q] - Y[p];
        // top-left rule (CCW, y up): an edge owns its samples when it runs
        // downwards, or horizontally towards -x
        miss[e] = (dy < 0 || (dy == 0 && dx < 0)) ? 0 : 1;
        r.h.e0[e] = (int32_t)(dx * (py - Y[p]) - dy * (px - X[p])) - miss[e];
        if (e < 2) {
            r.h.ex[e] = (int32_t)-dy;
            r.h.ey[e] = (int32_t)dx;
        }
    }
    const double cA = (double)A, ch = (double)(A >> 1) + 0.5, m0 = (double)miss[1], m1 = (double)miss[2];
    auto form = [&](uint32_t a0, uint32_t a1, uint32_t a2) {
        TriAtt f;
        f.d0 = (double)a0 - (double)a2;
        f.d1 = (double)a1 - (double)a2;
        f.c = cA * (double)a2 + ch + m0 * f.d0 + m1 * f.d1;
        return f;
    };
#pragma unroll
    for (int ch8 = 0; ch8 < 4; ++ch8)
        r.n.att[ch8] = form((col[0] >> (8 * ch8)) & 0xFFu, (col[1] >> (8 * ch8)) & 0xFFu,
                            (col[2] >> (8 * ch8)) & 0xFFu);
    if (mode == FHV_PPFL) {
        const uint32_t z0 = (uint32_t)a[0][0], z1 = (uint32_t)a[1][0], z2 = (uint32_t)a[2][0];
        r.n.att[4] = form(z0, z1, z2);
        r.d.z[0] = z0;
        r.d.z[1] = z1;
        r.d.z[2] = z2;
        r.d.A = (uint32_t)A;
        r.d.half = (uint32_t)(A >> 1) + (uint32_t)miss[1] * z0 + (uint32_t)miss[2] * z1 + (uint32_t)miss[0] * z2;
        return kTriNarrow | (A >= (1 << 26) ? kTriDepth32 : 0u);
    }
#pragma unroll
    for (int c = 0; c < 3; ++c)
        r.n.att[4 + c] = form((uint32_t)a[0][c], (uint32_t)a[1][c], (uint32_t)a[2][c]);
    return kTriNarrow;
}

// Setup record `tr` of n_rec: triangle tr / copies. POFL projection: the
// tangent frame (FHV_PROJ_NORMAL), or an axis plane: `axis` (2: x-y, 0: y-z,
// 1: z-x), or with three copies per triangle the copy's own (tr mod 3).
__global__ void __launch_bounds__(kBlock)
k_setup(const float* __restrict__ pos, const uint32_t* __restrict__ rgba,
        const uint32_t* __restrict__ tri, const uint8_t* __restrict__ obj, uint32_t n_rec,
        uint32_t mode, uint32_t width, uint32_t height, uint32_t levels, uint32_t tile_shift,
        uint32_t proj, uint32_t axis, uint32_t copies,
        const uint32_t* __restrict__ scene_tri, uint32_t n_scenes,
        TriRec* __restrict__ recs, uint64_t* __restrict__ tiles)
{
    const uint32_t tr = blockIdx.x * kBlock + threadIdx.x;
    if (tr >= n_rec) return;
    const uint32_t t = tr / copies;
    if (copies == 3) axis = tr % 3;
    // scene of a batch: the last s in [0, n_scenes) with scene_tri[s] <= t
    // (only scene_tri[1 .. n_scenes-1] is read, so the result stays in range)
    uint32_t scene = 0;
    if (scene_tri) {
        uint32_t lo = 0, hi = n_scenes - 1;
        while (lo < hi) {
            const uint32_t mid = (lo + hi + 1) >> 1;
            if (scene_tri[mid] <= t)
                lo = mid;
            else
                hi = mid - 1;
        }
        scene = lo;
    }
    TriRec r;
    int64_t X[3], Y[3];
    int32_t a[3][3];
    uint32_t col[3];
    bool skip = false;
    uint32_t nrm;
    uint32_t vtx[3];
#pragma unroll
    for (int k = 0; k < 3; ++k) vtx[k] = tri[3 * (uint64_t)t + k];
#pragma unroll
    for (int k = 0; k < 3; ++k) col[k] = rgba[vtx[k]];
    // the loops over vertices are unrolled and leave nothing early, so that
    // the arrays stay in registers
    if (mode == FHV_PPFL) {
        int64_t q[3][3];
#pragma unroll
        for (int k = 0; k < 3; ++k) {
            const float* p = pos + 3 * (uint64_t)vtx[k];
            const double x = p[0], y = p[1], z = p[2];
            if (!(fabs(x) <= 64.0 && fabs(y) <= 64.0 && fabs(z) <= 64.0)) skip = true;
            X[k] = (int64_t)rint((x + 1.0) * ((double)width * 128.0));
            Y[k] = (int64_t)rint((y + 1.0) * ((double)height * 128.0));
            double zd = rint((z + 1.0) * 0.5 * 16777215.0);
            zd = zd < 0.0 ? 0.0 : (zd > 16777215.0 ? 16777215.0 : zd);
            a[k][0] = (int32_t)zd;
            a[k][1] = a[k][2] = 0;
            q[k][0] = (int64_t)rint(x * 1048576.0);
            q[k][1] = (int64_t)rint(y * 1048576.0);
            q[k][2] = (int64_t)rint(z * 1048576.0);
        }
        if (!skip) {
            const int64_t ux = q[1][0] - q[0][0], uy = q[1][1] - q[0][1], uz = q[1][2] - q[0][2];
            const int64_t vx = q[2][0] - q[0][0], vy = q[2][1] - q[0][1], vz = q[2][2] - q[0][2];
            nrm = oct_pack(uy * vz - uz * vy, uz * vx - ux * vz, ux * vy - uy * vx);
        }
    } else {
        const double G = (double)(1ll << (levels + 8));
#pragma unroll
        for (int k = 0; k < 3; ++k) {
            const float* p = pos + 3 * (uint64_t)vtx[k];
#pragma unroll
            for (int c = 0; c < 3; ++c) {
                const float f = p[c];
                if (!isfinite(f)) skip = true;
                double g = floor((double)f * G);
                g = g < 0.0 ? 0.0 : (g > G - 1.0 ? G - 1.0 : g);
                a[k][c] = (int32_t)g;
            }
        }
        if (!skip) {
            const int64_t ux = a[1][0] - a[0][0], uy = a[1][1] - a[0][1], uz = a[1][2] - a[0][2];
            const int64_t vx = a[2][0] - a[0][0], vy = a[2][1] - a[0][1], vz = a[2][2] - a[0][2];
            const int64_t nx = uy * vz - uz * vy, ny = uz * vx - ux * vz, nz = ux * vy - uy * vx;
            if (nx == 0 && ny == 0 && nz == 0) {
                skip = true;
            } else {
                nrm = oct_pack(nx, ny, nz);
                if (proj == FHV_PROJ_NORMAL) {
                    double tt[3], bb[3];
                    tangent_frame(nrm, tt, bb);
#pragma unroll
                    for (int k = 0; k < 3; ++k) {
                        const double px = (double)a[k][0], py = (double)a[k][1], pz = (double)a[k][2];
                        const double u = px * tt[0] + py * tt[1] + pz * tt[2];
                        const double v = px * bb[0] + py * bb[1] + pz * bb[2];
                        X[k] = (int64_t)rint(2.0 * u);
                        Y[k] = (int64_t)rint(2.0 * v);
                    }
                } else {
                    // axis plane: (u, v) = two grid coordinates in cyclic
                    // order after the axis, exact integers
#pragma unroll
                    for (int k = 0; k < 3; ++k) {
                        X[k] = 2 * (int64_t)(axis == 0 ? a[k][1] : axis == 1 ? a[k][2] : a[k][0]);
                        Y[k] = 2 * (int64_t)(axis == 0 ? a[k][2] : axis == 1 ? a[k][0] : a[k][1]);
                    }
                }
            }
        }
    }
    uint64_t n_tiles = 0;
    if (!skip) {
        int64_t A = (X[1] - X[0]) * (Y[2] - Y[0]) - (Y[1] - Y[0]) * (X[2] - X[0]);
        if (A != 0) {
            if (A < 0) {   // vertices 1 and 2 swapped (by value: indexing would put the arrays in memory)
                A = -A;
                swap2(X);
                swap2(Y);
                swap2(col);
#pragma unroll
                for (int c = 0; c < 3; ++c) {
                    const int32_t a1 = a[1][c];
                    a[1][c] = a[2][c];
                    a[2][c] = a1;
                }
            }
            int64_t xmin = X[0], xmax = X[0], ymin = Y[0], ymax = Y[0];
#pragma unroll
            for (int k = 1; k < 3; ++k) {
                xmin = X[k] < xmin ? X[k] : xmin;
                xmax = X[k] > xmax ? X[k] : xmax;
                ymin = Y[k] < ymin ? Y[k] : ymin;
                ymax = Y[k] > ymax ? Y[k] : ymax;
            }
            int32_t i0, i1, j0, j1;
            sample_range(xmin, xmax, &i0, &i1);
            sample_range(ymin, ymax, &j0, &j1);
            if (mode == FHV_PPFL) {
                i0 = i0 < 0 ? 0 : i0;
                j0 = j0 < 0 ? 0 : j0;
                i1 = i1 > (int32_t)width - 1 ? (int32_t)width - 1 : i1;
                j1 = j1 > (int32_t)height - 1 ? (int32_t)height - 1 : j1;
            }
            r.h.lo_i = i0;
            r.h.lo_j = j0;
            r.h.hi_i = i1;
            r.h.hi_j = j1;
            r.h.nrm = nrm;
            r.h.aux = obj ? (uint32_t)obj[t] << 24 : 0u;
            r.rA = 1.0 / (double)A;
            const int64_t bw = xmax - xmin, bh = ymax - ymin;
            uint32_t flags = 0;
            if (bw < (1 << 22) && bh < (1 << 22) && bw * bh <= (1 << 30)) {
                flags = narrow_forms(r, X, Y, a, col, A, mode);
            } else {
#pragma unroll
                for (int k = 0; k < 3; ++k) {
                    r.w.x[k] = (int32_t)X[k];
                    r.w.y[k] = (int32_t)Y[k];
                    r.w.rgba[k] = col[k];
                    for (int c = 0; c < 3; ++c) r.w.a[k][c] = a[k][c];
                }
                r.w.A = A;
            }
            r.h.flags = flags;
            r.h.scene = scene;
            if (i1 >= i0 && j1 >= j0) {
                // tiles of (1 << tile_shift) x (64 >> tile_shift) samples
                const uint32_t tx = ((uint32_t)(i1 - i0) >> tile_shift) + 1;
                const uint32_t ty = ((uint32_t)(j1 - j0) >> (6 - tile_shift)) + 1;
                r.h.tiles_x = tx;
                n_tiles = (uint64_t)tx * ty;
            } else {
                r.h.tiles_x = 0;
            }
            recs[tr] = r;
        }
    }
    tiles[tr] = n_tiles;
}

// floor((w0 a0 + w1 a1 + w2 a2 + floor(A/2)) / A) for non-negative weights
// and attributes: an fp64 estimate (within 1 of the quotient) corrected by
// the exact remainder, which is small and therefore exact in wrapped
// 64-bit arithmetic even when the numerator itself exceeds 64 bits.
__device__ __forceinline__ uint32_t interp(int64_t w0, int64_t w1, int64_t w2, int32_t a0,
                                           int32_t a1, int32_t a2, int64_t A, double rA)
{
    const int64_t half = A >> 1;
    const double est = ((double)w0 * (double)a0 + (double)w1 * (double)a1 + (double)w2 * (double)a2 +
                        (double)half) * rA;
    int64_t q = (int64_t)floor(est);
    const uint64_t num = (uint64_t)w0 * (uint64_t)(uint32_t)a0 + (uint64_t)w1 * (uint64_t)(uint32_t)a1 +
                         (uint64_t)w2 * (uint64_t)(uint32_t)a2 + (uint64_t)half;
    const int64_t rem = (int64_t)(num - (uint64_t)q * (uint64_t)A);
    if (rem < 0)
        q -= 1;
    else if (rem >= A)
        q += 1;
    return (uint32_t)q;
}

// Colours of a wide triangle: in doubles, as for narrow ones, while A times
// 2^8 is below 2^50.
__device__ __forceinline__ uint32_t interp_rgba(int64_t w0, int64_t w1, int64_t w2,
                                                const uint32_t c[3], int64_t A, double rA)
{
    uint32_t out = 0;
    if (A < (1ll << 42)) {
        const double d0 = (double)w0, d1 = (double)w1, d2 = (double)w2, h = (double)(A >> 1) + 0.5;
#pragma unroll
        for (int ch = 0; ch < 4; ++ch) {
            const double num = __builtin_fma(
                d0, (double)((c[0] >> (8 * ch)) & 0xFFu),
                __builtin_fma(d1, (double)((c[1] >> (8 * ch)) & 0xFFu),
                              __builtin_fma(d2, (double)((c[2] >> (8 * ch)) & 0xFFu), h)));
            out |= (uint32_t)(num * rA) << (8 * ch);
        }
        return out;
    }
#pragma unroll 1
    for (int ch = 0; ch < 4; ++ch) {
        const int32_t c0 = (c[0] >> (8 * ch)) & 0xFF, c1 = (c[1] >> (8 * ch)) & 0xFF,
                      c2 = (c[2] >> (8 * ch)) & 0xFF;
        out |= interp(w0, w1, w2, c0, c1, c2, A, rA) << (8 * ch);
    }
    return out;
}

// Record `t` (wave-uniform): the loads of the parts asked for are all issued
// before the first is waited for.
typedef uint32_t u32x16 __attribute__((ext_vector_type(16)));

__device__ __forceinline__ TriHead load_head(const TriRec* recs, uint32_t t)
{
    return __builtin_bit_cast(TriHead, *(const u32x16*)&recs[t].h);
}

struct TriBody {   // the 192 bytes after the head
    u32x16 v[3];
};

__device__ __forceinline__ TriBody load_body(const TriRec* recs, uint32_t t)
{
    const u32x16* p = (const u32x16*)(recs + t);
    TriBody b{{p[1], p[2], p[3]}};
    return b;
}

// Where a tile's samples start, from the record's first sample.
struct TileAt {
    int32_t ox, oy;
};

__device__ __forceinline__ TileAt tile_at(const TriHead& h, uint32_t tile, uint32_t ts)
{
    uint32_t tx = 0, ty = tile;   // most triangles are one tile wide
    if (h.tiles_x != 1) {
        ty = uniform32(tile / h.tiles_x);
        tx = tile - ty * h.tiles_x;
    }
    return TileAt{(int32_t)(tx << ts), (int32_t)(ty << (6 - ts))};
}

// A narrow triangle's edge functions (less one where the edge does not own
// its samples) at the sample (lx, ly) of a tile, right where the sample lies
// in the box, and whether the sample is covered.
struct Edges32 {
    int32_t e01, e12, e20;
    bool cov;
};

__device__ __forceinline__ Edges32 edges32(const TriHead& h, TileAt at, int lx, int ly)
{
    const int32_t ex[3] = {h.ex[0], h.ex[1], -h.ex[0] - h.ex[1]}, ey[3] = {h.ey[0], h.ey[1], -h.ey[0] - h.ey[1]};
    int32_t e[3];
#pragma unroll
    for (int k = 0; k < 3; ++k) {
        const uint32_t base = (uint32_t)h.e0[k] + 256u * ((uint32_t)at.ox * (uint32_t)ex[k] +
                                                          (uint32_t)at.oy * (uint32_t)ey[k]);
        // |ex|, |ey| < 2^22, lx, ly < 64: 24-bit products
        const uint32_t step = (uint32_t)__mul24(lx, ex[k]) + (uint32_t)__mul24(ly, ey[k]);
        e[k] = (int32_t)(base + (step << 8));
    }
    Edges32 o{e[0], e[1], e[2], false};
    o.cov = (e[0] | e[1] | e[2]) >= 0 && lx <= h.hi_i - h.lo_i - at.ox && ly <= h.hi_j - h.lo_j - at.oy;
    return o;
}

// A wide triangle's edge functions at sample (i, j) and its coverage.
struct Edges64 {
    int64_t e01, e12, e20;
    bool cov;
};

__device__ __forceinline__ Edges64 edges64(const TriHead& h, const TriWide& w, int32_t i, int32_t j)
{
    Edges64 s{0, 0, 0, false};
    s.cov = i <= h.hi_i && j <= h.hi_j;
    if (s.cov) {
        const int64_t px = 256 * (int64_t)i + 128, py = 256 * (int64_t)j + 128;
        const int64_t x0 = w.x[0], x1 = w.x[1], x2 = w.x[2];
        const int64_t y0 = w.y[0], y1 = w.y[1], y2 = w.y[2];
        s.e01 = (x1 - x0) * (py - y0) - (y1 - y0) * (px - x0);
        s.e12 = (x2 - x1) * (py - y1) - (y2 - y1) * (px - x1);
        s.e20 = (x0 - x2) * (py - y2) - (y0 - y2) * (px - x2);
        // top-left rule (CCW, y up): an edge owns its samples when it runs
        // downwards, or horizontally towards -x
        const bool o01 = (y1 < y0) || (y1 == y0 && x1 < x0);
        const bool o12 = (y2 < y1) || (y2 == y1 && x2 < x1);
        const bool o20 = (y0 < y2) || (y0 == y2 && x0 < x2);
        s.cov = (s.e01 > 0 || (s.e01 == 0 && o01)) && (s.e12 > 0 || (s.e12 == 0 && o12)) &&
                (s.e20 > 0 || (s.e20 == 0 && o20));
    }
    return s;
}

// Whether this lane's sample of tile `tile` of record t is covered.
__device__ __forceinline__ bool covered(const TriRec* recs, uint32_t t, uint32_t tile, int lx, int ly, uint32_t ts)
{
    const TriHead h = load_head(recs, t);
    const TileAt at = tile_at(h, tile, ts);
    if (h.flags & kTriNarrow) return edges32(h, at, lx, ly).cov;
    return edges64(h, recs[t].w, h.lo_i + at.ox + lx, h.lo_j + at.oy + ly).cov;
}

// A fragment: coverage, key, and the first three record words.
struct Frag {
    bool cov;
    uint64_t key;
    uint32_t w0, w1, w2;
};

template <int kMode>
__device__ __forceinline__ uint64_t frag_key(uint32_t scene, int32_t i, int32_t j, uint32_t width, uint32_t gx,
                                             uint32_t gy, uint32_t gz, uint32_t levels)
{
    if (kMode == FHV_PPFL) return (uint64_t)((uint32_t)j * width + (uint32_t)i);   // below 2^28
    // ten bits per axis in 32 bits, the eleventh (depth 11) above them
    const uint32_t kx = gx >> 8, ky = gy >> 8, kz = gz >> 8;
    uint64_t key = (spread3_10(kx & 1023u) << 2) | (spread3_10(ky & 1023u) << 1) | spread3_10(kz & 1023u);
    if (levels > 10) key |= (uint64_t)(((kx >> 10) << 2) | ((ky >> 10) << 1) | (kz >> 10)) << 30;
    return key | ((uint64_t)scene << (3 * levels));
}

// The fragment of this lane's sample (lx, ly) of tile `tile` of record t.
template <int kMode>
__device__ __forceinline__ Frag fragment(const TriRec* recs, uint32_t t, uint32_t tile, int lx, int ly, uint32_t ts,
                                         uint32_t width, uint32_t gmax, uint32_t levels)
{
    const TriHead h = load_head(recs, t);
    const TriBody b = load_body(recs, t);
    const TileAt at = tile_at(h, tile, ts);
    const int32_t i = h.lo_i + at.ox + lx, j = h.lo_j + at.oy + ly;
    Frag f{false, 0, 0, 0, h.nrm};
    uint32_t gx = 0, gy = 0, gz = 0;
    struct Rest {
        double rA;
        TriNarrow n;
        uint32_t pad[4];
    };
    const Rest rest = __builtin_bit_cast(Rest, b);
    const double rA = rest.rA;
    if (h.flags & kTriNarrow) {
        const Edges32 e = edges32(h, at, lx, ly);
        f.cov = e.cov;
        if (!e.cov) return f;
        const double e12 = (double)e.e12, e20 = (double)e.e20;
        auto eval = [&](int k) -> uint32_t {
            const TriAtt& a = rest.n.att[k];
            return (uint32_t)(__builtin_fma(e12, a.d0, __builtin_fma(e20, a.d1, a.c)) * rA);
        };
        f.w1 = eval(0) | (eval(1) << 8) | (eval(2) << 16) | (eval(3) << 24);
        if (kMode == FHV_PPFL) {
            uint32_t q = eval(4);
            if (h.flags & kTriDepth32) {
                const TriDepth& d = recs[t].d;
                const int32_t rem = (int32_t)((uint32_t)e.e12 * d.z[0] + (uint32_t)e.e20 * d.z[1] +
                                              (uint32_t)e.e01 * d.z[2] + d.half - q * d.A);
                q = rem < 0 ? q - 1 : (rem >= (int32_t)d.A ? q + 1 : q);
            }
            f.w0 = q | h.aux;
        } else {
            gx = eval(4);
            gy = eval(5);
            gz = eval(6);
        }
    } else {
        const TriWide& w = recs[t].w;
        const Edges64 e = edges64(h, w, i, j);
        f.cov = e.cov;
        if (!e.cov) return f;
        f.w1 = interp_rgba(e.e12, e.e20, e.e01, w.rgba, w.A, rA);
        if (kMode == FHV_PPFL) {
            f.w0 = interp(e.e12, e.e20, e.e01, w.a[0][0], w.a[1][0], w.a[2][0], w.A, rA) | h.aux;
        } else {
            gx = interp(e.e12, e.e20, e.e01, w.a[0][0], w.a[1][0], w.a[2][0], w.A, rA);
            gy = interp(e.e12, e.e20, e.e01, w.a[0][1], w.a[1][1], w.a[2][1], w.A, rA);
            gz = interp(e.e12, e.e20, e.e01, w.a[0][2], w.a[1][2], w.a[2][2], w.A, rA);
        }
    }
    if (kMode == FHV_POFL) {
        // interpolation stays within the vertices' range; the clamp only
        // keeps the key inside the head array
        gx = gx > gmax ? gmax : gx;
        gy = gy > gmax ? gmax : gy;
        gz = gz > gmax ? gmax : gz;
        f.w0 = (gx & 0xFFu) | ((gy & 0xFFu) << 8) | ((gz & 0xFFu) << 16) | h.aux;
    }
    f.key = frag_key<kMode>(h.scene, i, j, width, gx, gy, gz, levels);
    return f;
}

// Walks work items in ascending order (wave-uniform): 64 consecutive entries
// of the inclusive tile counts are held one per lane, so that an item's
// triangle is found with one ballot instead of a load per triangle.
struct ItemWalk {
    const uint64_t* incl;
    uint32_t n_tri;
    uint32_t t0;      // first triangle of the window
    uint64_t before;  // items before it
    uint64_t v;       // this lane's incl[t0 + lane] (all ones past the end)
    __device__ __forceinline__ void window(uint32_t t)
    {
        t0 = t;
        before = t ? uniform64(incl[t - 1]) : 0;
        const uint64_t k = (uint64_t)t + __lane_id();
        v = k < n_tri ? incl[k] : ~0ull;
    }
    // the window starts at the triangle of item w: 64 probes per step
    __device__ __forceinline__ void start(uint64_t w)
    {
        uint32_t lo = 0, n = n_tri;   // the first t with incl[t] > w lies in [lo, lo + n)
        while (n > kWave) {
            const uint32_t step = (n + kWave - 1) / kWave;
            const uint32_t off = ((uint32_t)__lane_id() + 1) * step;   // one past this lane's part
            const bool less = off <= n && incl[lo + off - 1] <= w;
            const uint32_t c = (uint32_t)__popcll(__ballot(less));
            lo += c * step;
            n = n - c * step < step ? n - c * step : step;
        }
        window(lo);
    }
    // triangle *t of item w (w not below the last one) and its first item
    __device__ __forceinline__ void find(uint64_t w, uint32_t* t, uint64_t* first)
    {
        uint32_t c;
        while ((c = (uint32_t)__popcll(__ballot(v <= w))) == kWave) window(t0 + kWave);
        *t = t0 + c;
        *first = c ? (uint64_t)(uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)v, c - 1) |
                         ((uint64_t)(uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)(v >> 32), c - 1) << 32)
                   : before;
    }
};

// Each wave owns a contiguous range of work items. It first counts the
// covered samples of the whole range; the workgroup then reserves its waves'
// pool slots with a single atomic add on the counter, and every wave walks
// its range again to emit the fragments into consecutive slots.
//
// What bounds it: with the edge functions and attributes in 64-bit integers
// the vector unit (about 3,500 cycles per tile, half of them 64-bit
// products); with the records' linear forms the scalar loads' latency and,
// with lists, the head exchanges at the memory side. Kernel times before and
// after the forms, the grouped counter, the 64-way search and the records'
// prefetch: 5.23 M fragments at depth 9 409 -> 208 us, 45 M at depth 10 2709
// -> 1767 us (27 M exchange requests, 15 G/s), 1.5 M pixel fragments 270 ->
// 86 us; without lists 307 -> 177 us (insert) and 234 -> 154 us (count); a
// batch of 32 M fragments 1353 -> 690 us.
//
// One add per workgroup of 8 waves: adds on one address run one after the
// other at the memory side, about 9 ns each, and with one per wave the time
// grew with the number of waves (1.47 M fragments at 1080p: 130 us with 4,096
// waves, 387 us with 32,768).
//
// kAct (two-pass capture into arrays, lists and pool unused): kActCount
// adds every fragment to its brick's histogram, kActInsert stores it in its
// brick's staging range with the key's low bits in w3.
// Captures without a counter take workgroups of 4 waves.
constexpr int raster_block(int act) { return act == kActList ? 512 : 256; }

template <int kMode, class KeyT, int kAct = kActList>
__global__ void __launch_bounds__(raster_block(kAct))
k_raster(const TriRec* __restrict__ recs, const uint64_t* __restrict__ incl, uint32_t n_tri,
         uint32_t width, uint32_t gmax, uint32_t levels, uint32_t ts, uint32_t* __restrict__ head,
         uint4* __restrict__ pool, KeyT* __restrict__ keys, uint64_t cap,
         unsigned long long* __restrict__ counter, BrickSink bs)
{
    constexpr int kRasterWaves = raster_block(kAct) / kWave;
    const uint64_t total = incl[n_tri - 1];
    const int lane = __lane_id();
    const uint64_t n_waves = (uint64_t)gridDim.x * kRasterWaves;
    const uint32_t wv = uniform32(threadIdx.x / kWave);
    const uint64_t wid = (uint64_t)blockIdx.x * kRasterWaves + wv;
    const uint64_t per = (total + n_waves - 1) / n_waves;
    const uint64_t w0 = wid * per;
    const uint64_t w1 = w0 + per < total ? w0 + per : total;
    if ((uint64_t)blockIdx.x * kRasterWaves * per >= total) return;   // whole workgroup
    if (kAct == kActInsert && *bs.skip) return;

    const int lx = lane & ((1 << ts) - 1), ly = lane >> ts;
    ItemWalk it{incl, n_tri, 0, 0, 0};
    if (w0 < w1) {
        it.start(w0);
        // one load per lane brings the first 64 lines of the wave's records
        // nearer: the scalar loads below follow one another, each waited for
        const uint64_t last = (uint64_t)n_tri * sizeof(TriRec) - 4;
        const uint64_t at = (uint64_t)it.t0 * sizeof(TriRec) + (uint64_t)lane * 64;
        const uint32_t x = *(const uint32_t*)((const char*)recs + (at < last ? at : last));
        asm volatile("" ::"v"(x));
    }
    constexpr int kBatch = 4;   // tiles per step; their memory operations overlap
    unsigned long long base = 0;
    if (kAct == kActList) {
        const ItemWalk it0 = it;
        uint64_t n_cov = 0;
        for (uint64_t w = w0; w < w1; ++w) {
            uint32_t t;
            uint64_t first;
            it.find(w, &t, &first);
            n_cov += (uint64_t)__popcll(__ballot(covered(recs, t, (uint32_t)(w - first), lx, ly, ts)));
        }
        __shared__ unsigned long long cnt[kRasterWaves], slots;
        if (lane == 0) cnt[wv] = n_cov;
        __syncthreads();
        unsigned long long sum = 0;
#pragma unroll
        for (int k = 0; k < kRasterWaves; ++k) {
            if (k == (int)wv) base = sum;
            sum += cnt[k];
        }
        if (threadIdx.x == 0) slots = sum ? atomicAdd(counter, sum) : 0;
        __syncthreads();
        base = uniform64(base + slots);
        if (n_cov == 0) return;
        it = it0;
    }

    uint32_t n_lane = 0;   // fragments counted by this lane
    for (uint64_t w = w0; w < w1; w += kBatch) {
        bool has[kBatch];
        uint64_t key[kBatch];
        uint32_t w0r[kBatch], w1r[kBatch], nrm[kBatch];
        uint64_t idx[kBatch];
#pragma unroll
        for (int g = 0; g < kBatch; ++g) {
            has[g] = false;
            key[g] = 0;
            idx[g] = 0;
            if (w + g >= w1) continue;   // wave-uniform
            uint32_t t;
            uint64_t first;
            it.find(w + g, &t, &first);
            const Frag f = fragment<kMode>(recs, t, (uint32_t)(w + g - first), lx, ly, ts, width, gmax, levels);
            if (kAct == kActList) {
                const uint64_t mask = __ballot(f.cov);
                idx[g] = base + (uint64_t)__popcll(mask & lanemask_lt());
                base += (uint64_t)__popcll(mask);
                has[g] = f.cov && idx[g] < cap;
            } else {
                has[g] = f.cov;
            }
            key[g] = f.key;
            nrm[g] = f.w2;
            w0r[g] = f.w0;
            w1r[g] = f.w1;
        }
        if (kAct != kActList) {
            // lanes of a tile with the same brick share one atomic; the
            // leaders' atomics of all the step's tiles are in flight at once
            uint64_t same[kBatch];
            uint32_t got[kBatch];
#pragma unroll
            for (int g = 0; g < kBatch; ++g) {
                const uint32_t b = (uint32_t)(key[g] >> kBrickShift);
                same[g] = w + g < w1 ? wave_same(b, has[g]) : 0ull;   // wave-uniform
                const bool leader = has[g] && (same[g] & lanemask_lt()) == 0;
                if (kAct == kActCount) {
                    n_lane += has[g] ? 1u : 0u;
                    if (leader) atomicAdd(bs.cnt + b, (uint32_t)__popcll(same[g]));
                } else {
                    got[g] = leader ? atomicAdd(bs.cur + b, (uint32_t)__popcll(same[g])) : 0u;
                }
            }
            if (kAct == kActInsert) {
#pragma unroll
                for (int g = 0; g < kBatch; ++g) {
                    if (w + g >= w1) continue;   // wave-uniform
                    const uint32_t slot =
                        (uint32_t)__shfl((int)got[g], __builtin_ctzll(same[g] | (1ull << 63)), kWave) +
                        lanes_below(same[g]);
                    if (has[g])
                        bs.stage[bs.off[key[g] >> kBrickShift] + slot] =
                            make_uint4(w0r[g], w1r[g], nrm[g], (uint32_t)key[g] & (kBrickKeys - 1));
                }
            }
            continue;
        }
        uint32_t prev[kBatch];
#pragma unroll
        for (int g = 0; g < kBatch; ++g) {
            prev[g] = kNil;
            if (head && has[g]) prev[g] = atomicExch(head + key[g], (uint32_t)idx[g]);
        }
#pragma unroll
        for (int g = 0; g < kBatch; ++g) {
            if (!has[g]) continue;
            pool[idx[g]] = make_uint4(w0r[g], w1r[g], nrm[g], prev[g]);
            keys[idx[g]] = (KeyT)key[g];
        }
    }
    if (kAct == kActCount && incl[n_tri - 1] >= kManyTiles) {
        unsigned long long n = n_lane;
#pragma unroll
        for (int d = kWave / 2; d >= 1; d >>= 1) n += __shfl_xor(n, d, kWave);
        if (lane == 0) atomicAdd(bs.total, n);
    }
}

}  // namespace

// Setup records per pass: three projected copies of every triangle for
// FHV_PROJ_AXES_1PASS, one otherwise.
static uint64_t records_of(const fhv_capture_desc* d, uint32_t n_tri)
{
    return d->mode == FHV_POFL && d->projection == FHV_PROJ_AXES_1PASS ? 3ull * n_tri : (uint64_t)n_tri;
}

size_t capture_ws_bytes(const fhv_capture_desc* d, uint32_t n_tri)
{
    const uint64_t n = records_of(d, n_tri);
    Carver c{nullptr, 0};
    c.take<TriRec>(n);
    c.take<uint64_t>(n);
    c.take<uint64_t>(n);
    c.take<uint64_t>(scan_partials(n));
    return c.off + 256;
}

// raster_wg counts workgroups of 4 waves per compute unit.
static unsigned raster_grid(const Device& dev, int act)
{
    return (unsigned)std::max(1u, (uint32_t)dev.cus * dev.tune.raster_wg * kBlock / (uint32_t)raster_block(act));
}

// Setup of pass `pass` (of one, or three for 3-Pass/1-Way) and the
// inclusive scan of its tiles per record.
static hipError_t setup_pass(const Device& dev, const fhv_mesh* m, const fhv_capture_desc* d, uint32_t pass,
                             const Scenes* sc, TriRec* recs, uint64_t* tiles, uint64_t* incl, uint64_t* part,
                             const char* setup_name, const char* scan_name, hipStream_t s)
{
    const uint64_t n_rec = records_of(d, m->n_tri);
    const uint32_t ts = dev.tune.tile_w == 32 ? 5u : (dev.tune.tile_w == 16 ? 4u : 3u);
    const uint32_t proj = d->mode == FHV_POFL ? d->projection : FHV_PROJ_NORMAL;
    const uint32_t copies = proj == FHV_PROJ_AXES_1PASS ? 3u : 1u;
    // the axis plane of the pass: y-z, z-x, x-y for 3-Pass/1-Way, x-y for
    // 1-Pass/View
    const uint32_t axis = proj == FHV_PROJ_AXES_3PASS ? pass : 2u;
    hipError_t e;
    {
        ProfScope ps(dev, setup_name, s);
        k_setup<<<dim3((unsigned)((n_rec + kBlock - 1) / kBlock)), dim3(kBlock), 0, s>>>(
            m->pos, m->rgba, m->tri, m->obj, (uint32_t)n_rec, d->mode, d->width, d->height, d->levels, ts, proj,
            axis, copies, sc ? sc->scene_tri : nullptr, sc ? sc->n_scenes : 1u, recs, tiles);
        e = hipGetLastError();
    }
    if (e != hipSuccess) return e;
    ProfScope ps(dev, scan_name, s);
    return scan_u64(tiles, incl, n_rec, true, part, nullptr, s);
}

hipError_t capture_bricks_launch(const Device& dev, const fhv_mesh* m, const fhv_capture_desc* d, void* ws,
                                 int act, const BrickSink& bs, bool again, hipStream_t s)
{
    const uint64_t n_rec = records_of(d, m->n_tri);
    Carver c{(char*)ws, 0};
    TriRec* recs = c.take<TriRec>(n_rec);
    uint64_t* tiles = c.take<uint64_t>(n_rec);
    uint64_t* incl = c.take<uint64_t>(n_rec);
    uint64_t* part = c.take<uint64_t>(scan_partials(n_rec));
    if (m->n_tri == 0) return hipSuccess;
    const uint32_t ts = dev.tune.tile_w == 32 ? 5u : (dev.tune.tile_w == 16 ? 4u : 3u);
    const uint32_t passes = d->projection == FHV_PROJ_AXES_3PASS ? 3u : 1u;
    const unsigned grid = raster_grid(dev, act);
    const uint32_t gmax = (1u << (d->levels + 8)) - 1u;
    const char* name = act == kActCount ? "arrays.count" : "arrays.insert";
    for (uint32_t pass = 0; pass < passes; ++pass) {
        hipError_t e = hipSuccess;
        if (!again || passes > 1)
            e = setup_pass(dev, m, d, pass, nullptr, recs, tiles, incl, part, "arrays.setup", "arrays.scan", s);
        if (e != hipSuccess) return e;
        ProfScope ps(dev, name, s);
        if (act == kActCount)
            k_raster<FHV_POFL, uint32_t, kActCount><<<dim3(grid), dim3(raster_block(act)), 0, s>>>(
                recs, incl, (uint32_t)n_rec, 0u, gmax, d->levels, ts, nullptr, nullptr, nullptr, 0, nullptr, bs);
        else
            k_raster<FHV_POFL, uint32_t, kActInsert><<<dim3(grid), dim3(raster_block(act)), 0, s>>>(
                recs, incl, (uint32_t)n_rec, 0u, gmax, d->levels, ts, nullptr, nullptr, nullptr, 0, nullptr, bs);
        e = hipGetLastError();
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}

hipError_t capture_launch(const Device& dev, const fhv_mesh* m, const fhv_capture_desc* d,
                          const fhv_lists* L, void* ws, hipStream_t s, const Scenes* sc)
{
    const uint64_t n_rec = records_of(d, m->n_tri);
    Carver c{(char*)ws, 0};
    TriRec* recs = c.take<TriRec>(n_rec);
    uint64_t* tiles = c.take<uint64_t>(n_rec);
    uint64_t* incl = c.take<uint64_t>(n_rec);
    uint64_t* part = c.take<uint64_t>(scan_partials(n_rec));
    const uint32_t ts = dev.tune.tile_w == 32 ? 5u : (dev.tune.tile_w == 16 ? 4u : 3u);
    hipError_t e;
    {
        ProfScope ps(dev, "capture.reset", s);
        e = fill_u32(L->head, L->head ? L->n_head : 0, kNil, s, L->counter);
    }
    if (e != hipSuccess || m->n_tri == 0) return e;
    // three passes for 3-Pass/1-Way, one otherwise
    const uint32_t passes = d->mode == FHV_POFL && d->projection == FHV_PROJ_AXES_3PASS ? 3u : 1u;
    const unsigned grid = raster_grid(dev, kActList);
    const uint32_t gmax = d->mode == FHV_POFL ? (1u << (d->levels + 8)) - 1u : 0u;
    const bool wide = L->n_head > (1ull << 32);
    for (uint32_t pass = 0; pass < passes; ++pass) {
        e = setup_pass(dev, m, d, pass, sc, recs, tiles, incl, part, "capture.setup", "capture.scan", s);
        if (e != hipSuccess) return e;
        ProfScope ps(dev, "capture.raster", s);
        if (d->mode == FHV_PPFL)
            k_raster<FHV_PPFL, uint32_t><<<dim3(grid), dim3(raster_block(kActList)), 0, s>>>(
                recs, incl, (uint32_t)n_rec, d->width, gmax, d->levels, ts, L->head, (uint4*)L->pool,
                (uint32_t*)L->keys, L->capacity, (unsigned long long*)L->counter, BrickSink{});
        else if (!wide)
            k_raster<FHV_POFL, uint32_t><<<dim3(grid), dim3(raster_block(kActList)), 0, s>>>(
                recs, incl, (uint32_t)n_rec, d->width, gmax, d->levels, ts, L->head, (uint4*)L->pool,
                (uint32_t*)L->keys, L->capacity, (unsigned long long*)L->counter, BrickSink{});
        else
            k_raster<FHV_POFL, uint64_t><<<dim3(grid), dim3(raster_block(kActList)), 0, s>>>(
                recs, incl, (uint32_t)n_rec, d->width, gmax, d->levels, ts, L->head, (uint4*)L->pool,
                (uint64_t*)L->keys, L->capacity, (unsigned long long*)L->counter, BrickSink{});
        e = hipGetLastError();
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}

}  // namespace fhv
