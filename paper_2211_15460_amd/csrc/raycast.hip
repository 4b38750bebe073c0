// Ray casting of per-octant arrays (Sec. 3.3, evaluation by ray casting).
//
// With an orthographic view the ray of a pixel meets a fragment when the
// fragment projects into that pixel (the one-pixel footprint of the splat),
// so the fragments that the rays of a screen tile meet are those that
// project into it. Two ways to find them:
//
// Tiles (first choice): bounding boxes over chunks of 64 consecutive
// fragments, over groups of 64 chunks and so on (16 bytes each, built per
// call), walked by one workgroup per 16 x 16 pixel tile down to the chunks
// that can reach the tile, whose fragments are projected one per lane.
// Nearest: a 64-bit minimum per pixel in LDS. Transparency: the hits are
// collected in LDS, grouped by pixel and ordered by (depth bits, index), and
// every lane composites its pixel front to back; a tile with more hits than
// LDS holds takes them in slabs of that order, nearest first, until every
// pixel is final.
//
//   k_ray_box     one workgroup per group: its chunks' boxes and its own
//   k_ray_node    boxes of the levels above, down to kTopNodes nodes
//   k_ray_tile    one workgroup per tile
//
// The workspace is sized by the octree depth alone, for the octree walk
// below; the boxes take 0.26 bytes per fragment of it. Where the arrays'
// capacity says that they fit, the tiles are the only way; where it does
// not, the fragment count decides on the device (each way's kernels return
// at once where the other one is taken). Both give the same image bit for
// bit. The walk's chain of dependent loads and its handing over of one hit at
// a time bound it (times of both at k_ray_tile).
//
// Octree walk. The occupancy of every octree level is rebuilt from the table of occupied
// leaves (Sec. 3.1: coarser levels hold only the occupancy of their
// children, for empty-space skipping). Then one wave per 8 x 8 pixel tile
// walks the octree from the root (every decision of the walk is uniform
// across the wave), descending only into occupied children whose box can
// project into the tile, down to bricks of 4^3 or 8^3 leaves; a brick's
// fragments are one contiguous range of the arrays, tested one per lane and
// handed to the lane owning the pixel they land in.
//
// Children are visited nearest first (one order per view). Each lane keeps
// the fragments met for its pixel in a list ordered by (depth bits, index)
// and composites them front to back as soon as no unvisited octant can hold
// a nearer one; a lane is final when its transmittance falls below the
// threshold, and the walk ends when every lane of the tile is final. An
// octant is skipped when its depth range lies behind every compositing
// lane's list, or in front of what earlier walks composited; when a list
// overflows, the walk is repeated for the fragments behind the last one
// composited.
//
//   k_occ_build   one thread per table row: the row's leaf bit and, where
//                 the row is the first of its parent octant, the bits of its
//                 ancestors (rows are in Morton order, so a parent's first
//                 row sets it once)
//   k_raycast     one wave per 8 x 8 pixel tile, one lane per pixel
//
// Workspace: level l (1 <= l <= L) has a bitmap of 8^l bits in Morton order
// (the 8 children of octant n of level l-1 are byte n of level l's bitmap);
// the leaf level has, per 64-bit word, the number of set bits before it,
// which turns a leaf's Morton code into its table row.
#include <algorithm>

#include "fhv_common.h"
#include "scan.h"

namespace fhv {

namespace {

constexpr int kCap = 16;   // fragments a lane keeps per walk

struct OccLayout {
    uint64_t word[kMaxRayLevels + 2];   // u32 offset of level l's bitmap, l = 1..L; [L+1] = end
    uint64_t n64;                       // 64-bit words of the leaf bitmap
};

OccLayout occ_layout(uint32_t L)
{
    OccLayout o{};
    uint64_t w = 0;
    for (uint32_t l = 1; l <= L; ++l) {
        o.word[l] = w;
        const uint64_t bits = 1ull << (3 * l);
        uint64_t words = (bits + 31) / 32;
        words = (words + 1) & ~1ull;   // 8-byte aligned levels
        w += words;
    }
    o.word[L + 1] = w;
    o.n64 = ((1ull << (3 * L)) + 63) / 64;
    return o;
}

// Fragments of the arrays' stored rows (contiguous, in row order).
struct Rows {
    const uint64_t* oct_key;
    const uint32_t *oct_off, *oct_cnt;
    const uint64_t* n_occ;
    uint64_t cap_occ, cap_frag;
    __device__ __forceinline__ uint64_t count() const { return *n_occ < cap_occ ? *n_occ : cap_occ; }
    __device__ __forceinline__ uint64_t frags() const
    {
        const uint64_t n = count();
        if (n == 0) return 0;
        const uint64_t f = (uint64_t)oct_off[n - 1] + oct_cnt[n - 1];
        return f < cap_frag ? f : cap_frag;
    }
};

// ------------------------------------------------------------------- tiles

constexpr uint32_t kFan = kWave;   // 2^6
constexpr uint32_t kTopNodes = 512;   // the walk starts from a level of at most this many nodes

// Levels of boxes over F fragments: 0 chunks, 1 groups of kFan chunks, and
// so on up to at most kTopNodes nodes (level 1 at least). Computed where
// they are needed: a table indexed by a variable would live in memory.
struct BoxLevels {
    uint64_t chunks;
    __host__ __device__ __forceinline__ explicit BoxLevels(uint64_t F) : chunks((F + kWave - 1) / kWave) {}
    __host__ __device__ __forceinline__ uint64_t n(uint32_t l) const
    {
        const uint32_t sh = 6 * l;
        return (chunks + ((uint64_t)1 << sh) - 1) >> sh;
    }
    __host__ __device__ __forceinline__ uint64_t off(uint32_t l) const   // boxes of the levels below l
    {
        uint64_t o = 0;
        for (uint32_t k = 0; k < l; ++k) o += n(k);
        return o;
    }
    __host__ __device__ __forceinline__ uint32_t top() const
    {
        uint32_t l = 1;
        while (n(l) > kTopNodes) ++l;
        return l;
    }
    __host__ __device__ __forceinline__ uint64_t total() const { return off(top() + 1); }
};

// Where the tiles' way keeps its data in the workspace; `room` boxes fit.
struct BoxArea {
    uint64_t* frags;   // fragments, 0 where the boxes do not fit
    uint4* box;
    uint64_t room;
};

// Grid position of a fragment (depth up to 10: 30-bit keys).
__device__ __forceinline__ void grid_pos(uint32_t w0, uint32_t key, uint32_t* x, uint32_t* y, uint32_t* z)
{
    *x = (compact3_10(key >> 2) << 8) | (w0 & 0xFFu);
    *y = (compact3_10(key >> 1) << 8) | ((w0 >> 8) & 0xFFu);
    *z = (compact3_10(key) << 8) | ((w0 >> 16) & 0xFFu);
}

// One workgroup per group of 64 chunks; boxes in units of 2^qs grid steps,
// which fit 16 bits. Reads every fragment's record (and
// its row's key) once: bound by those 16 bytes a fragment.
__global__ void __launch_bounds__(kBlock)
k_ray_box(const uint4* __restrict__ frag, Rows rows, BoxArea area, uint32_t qs)
{
    __shared__ BoxMin part[kBlock / kWave];
    const uint64_t F = rows.frags();
    const BoxLevels lv(F);
    const bool fits = lv.total() <= area.room;
    if (blockIdx.x == 0 && threadIdx.x == 0) *area.frags = fits ? F : 0;
    if (!fits) return;
    const uint64_t n_rows = rows.count();
    const int lane = __lane_id();
    const uint32_t wv = uniform32(threadIdx.x / kWave);
    constexpr uint32_t kPer = kFan / (kBlock / kWave);   // chunks per wave
    for (uint64_t g = blockIdx.x; g < lv.n(1); g += gridDim.x) {
        BoxMin all{{~0u, ~0u, ~0u}};
        for (uint32_t k0 = 0; k0 < kPer; k0 += 4) {
            const uint64_t ch = g * kFan + wv * kPer + k0;
            if (ch >= lv.chunks) break;   // wave-uniform
            uint4 r[4];
            uint32_t key[4];
            bool ok[4];
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                const uint64_t f = (ch + u) * kWave + lane;
                r[u] = frag[f < F ? f : F - 1];
                ok[u] = f < F && r[u].w < n_rows;
            }
#pragma unroll
            for (int u = 0; u < 4; ++u) key[u] = (uint32_t)rows.oct_key[ok[u] ? r[u].w : 0];
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                uint32_t x, y, z;
                grid_pos(r[u].x, key[u], &x, &y, &z);
                x >>= qs;
                y >>= qs;
                z >>= qs;
                const BoxMin m = wave_box(x, y, z, ok[u]);
                if (lane == 0 && ch + u < lv.chunks) area.box[ch + u] = box_store(m);
                all = box_join(all, m);
            }
        }
        if (lane == 0) part[wv] = all;
        __syncthreads();
        if (threadIdx.x == 0) {
            BoxMin m = part[0];
#pragma unroll
            for (int w = 1; w < kBlock / kWave; ++w) m = box_join(m, part[w]);
            area.box[lv.off(1) + g] = box_store(m);
        }
        __syncthreads();
    }
}

// Boxes of level l >= 2, one wave per node.
__global__ void __launch_bounds__(kBlock) k_ray_node(BoxArea area, uint32_t l)
{
    const BoxLevels lv(*area.frags);
    if (l > lv.top()) return;
    const int lane = __lane_id();
    const uint64_t n_waves = (uint64_t)gridDim.x * (kBlock / kWave);
    for (uint64_t node = uniform64((uint64_t)blockIdx.x * (kBlock / kWave) + threadIdx.x / kWave); node < lv.n(l);
         node += n_waves) {
        const uint64_t c = node * kFan + lane;
        BoxMin m{{~0u, ~0u, ~0u}};
        if (c < lv.n(l - 1)) m = box_load(area.box[lv.off(l - 1) + c]);
#pragma unroll
        for (int k = 0; k < 3; ++k) m.v[k] = wave_pk_min(m.v[k]);
        if (lane == 0) area.box[lv.off(l) + node] = box_store(m);
    }
}

struct RayTileArgs {
    float m[kMaxViews][12];
    const uint4* frag;
    Rows rows;
    BoxArea area;
    float4* out;           // [V][H][W]
    uint32_t width, height, tiles_x, qs;
    float grid;            // grid units per cube side
    float tau;
};

constexpr int kTile = 16;                   // tile side in pixels
constexpr int kPix = kTile * kTile;         // one pixel per thread of the first four waves
constexpr int kRayBlock = 512;
constexpr int kRayWaves = kRayBlock / kWave;
constexpr uint32_t kFront = 512;            // frontier capacity of the walk (node ids)
constexpr uint32_t kRoundGroups = 32;       // groups whose chunks are queued at a time
constexpr uint32_t kHits = 4000;            // hits held per slab
constexpr uint32_t kPerThread = (kHits + kRayBlock - 1) / kRayBlock;
constexpr uint32_t kMostPerPixel = 128;     // of one pixel: ordering a pixel's n hits takes n^2 comparisons
constexpr uint32_t kFinal = 1u << 31;       // in cnt: the pixel is final
constexpr uint64_t kPastKeys = 0x7F800001ull << 32;   // above the key of any hit

__device__ __forceinline__ float proj(const float* M, int row, float x, float y, float z)
{
    return ((M[4 * row + 0] * x + M[4 * row + 1] * y) + M[4 * row + 2] * z) + M[4 * row + 3];
}

// One workgroup of 8 waves per 16 x 16 pixel tile of one view, three tiles
// per compute unit (52 KB of LDS and 80 registers, which the blended form
// overruns: 61 values, 224 bytes a lane, go to scratch memory; four tiles with
// 64 registers and 3,328 hits spill more: 0.87 ms in place of 0.69; 16 waves a
// tile 1.49; 4 waves with 217 registers 0.96). The waves walk
// the boxes breadth first (64 per step, one per lane) to the groups that can
// reach the tile; each wave then takes groups in turn, tests their chunks and
// projects the fragments of those that can reach it, four chunks' loads in
// flight. A box is rejected only when every fragment inside it must miss the
// tile (or the slab): its fp32 extent is widened by 2^-20 of the sum of
// absolute terms, which covers the rounding of the extent and of any
// fragment's own projection.
//
// What bounds it is latency: 72 % of the tiles of a 1080p view are empty and
// take about 5 us each, one with 2,000 hits 40 us, half of it the loads of the
// chunks. Three 1080p views of 5.2 M fragments with random transparencies:
// 6.0 ms by the octree walk, 0.69 ms here; nearest fragment, one 720p view of
// 0.36 M fragments: 557 us, 27 us.
template <int kMode>
__global__ void __launch_bounds__(kRayBlock, 6) k_ray_tile(RayTileArgs a)
{
    __shared__ uint32_t front[2][kFront];
    __shared__ uint32_t queue[kRoundGroups * kFan];
    __shared__ uint32_t sh_n, sh_over;
    // nearest: the pixels' least keys. Transparency: the slab's hits, and per
    // pixel their number, where they start and a cursor
    __shared__ unsigned long long hit[kMode == 0 ? kPix : kHits];
    __shared__ uint8_t hit_px[kMode == 0 ? 1 : kHits];
    __shared__ uint32_t cnt[kMode == 0 ? 1 : kPix], off[kMode == 0 ? 1 : kPix + 1], cur[kMode == 0 ? 1 : kPix];
    __shared__ uint32_t sh_hits, sh_most[kRayWaves], sh_sum[kRayWaves];
    __shared__ unsigned long long sh_min, sh_max;
    __shared__ float unit[kMode == 0 ? 1 : 256];   // k / 255
    const uint64_t F = *a.area.frags;
    if (F == 0 && a.rows.frags() != 0) return;   // the boxes did not fit: the octree walk makes the image
    const int lane = __lane_id();
    const uint32_t t = threadIdx.x, wv = uniform32(t / kWave);
    const uint32_t v = blockIdx.y;
    const uint32_t x0 = (blockIdx.x % a.tiles_x) * kTile, y0 = (blockIdx.x / a.tiles_x) * kTile;
    const uint32_t px = x0 + t % kTile, py = y0 + t / kTile;
    const bool mine = t < (uint32_t)kPix && px < a.width && py < a.height;
    const float X0 = (float)x0, X1 = (float)(x0 + kTile), Y0 = (float)y0, Y1 = (float)(y0 + kTile);
    const float* const M = a.m[v];
    const BoxLevels lv(F);
    const uint32_t n_rows = (uint32_t)a.rows.count();
    // margins of the rows' extents
    float mg[3];
#pragma unroll
    for (int r = 0; r < 3; ++r)
        mg[r] = 0x1p-20f * ((fabsf(M[4 * r]) + fabsf(M[4 * r + 1]) + fabsf(M[4 * r + 2])) * a.grid + fabsf(M[4 * r + 3]) + 1.0f);
    const float q = (float)(1u << a.qs);
    // whether a fragment in the box can project into the tile with a depth in
    // [dlo, dhi] (written so that values that are not numbers reject nothing)
    auto reach = [&](const uint4& b, float dlo, float dhi) -> bool {
        const uint32_t lx = b.x & 0xFFFFu, ly = b.x >> 16, lz = b.y & 0xFFFFu, hx = b.y >> 16, hy = b.z & 0xFFFFu,
                       hz = b.z >> 16;
        // positions lie half a step from both ends of their units
        const float h = 0.5f * q;
        const float cx = (float)(lx + hx + 1) * h, cy = (float)(ly + hy + 1) * h, cz = (float)(lz + hz + 1) * h;
        const float ex = __builtin_fmaf((float)(hx - lx + 1), h, -0.5f), ey = __builtin_fmaf((float)(hy - ly + 1), h, -0.5f),
                    ez = __builtin_fmaf((float)(hz - lz + 1), h, -0.5f);
        float s[3], e[3];
#pragma unroll
        for (int r = 0; r < 3; ++r) {
            s[r] = __builtin_fmaf(M[4 * r], cx, __builtin_fmaf(M[4 * r + 1], cy, __builtin_fmaf(M[4 * r + 2], cz, M[4 * r + 3])));
            e[r] = __builtin_fmaf(fabsf(M[4 * r]), ex, __builtin_fmaf(fabsf(M[4 * r + 1]), ey,
                                                                      __builtin_fmaf(fabsf(M[4 * r + 2]), ez, mg[r])));
        }
        return lx <= hx && !(s[0] + e[0] < X0) && !(s[0] - e[0] >= X1) && !(s[1] + e[1] < Y0) &&
               !(s[1] - e[1] >= Y1) && !(s[2] + e[2] < dlo) && !(s[2] - e[2] > dhi);
    };
    // ---- the walk, to nodes of level `l` that can reach the tile
    uint32_t l = lv.top(), n_front = (uint32_t)lv.n(l), c = 0;
    if (t == 0) sh_n = 0;
    __syncthreads();
    const uint4* boxes = a.area.box + lv.off(l);
    for (uint32_t i0 = wv * kWave; i0 < n_front; i0 += kRayBlock) {
        const uint32_t i = i0 + lane;
        const bool ok = i < n_front && reach(boxes[i], 0.0f, INFINITY);
        const uint64_t m = __ballot(ok);
        uint32_t base = 0;
        if (lane == 0 && m) base = atomicAdd(&sh_n, (uint32_t)__popcll(m));
        base = uniform32(base);
        if (ok) front[0][base + lanes_below(m)] = i;
    }
    __syncthreads();
    n_front = sh_n;
    while (l > 1 && n_front > 0) {
        __syncthreads();
        if (t == 0) {
            sh_n = 0;
            sh_over = 0;
        }
        __syncthreads();
        boxes = a.area.box + lv.off(l - 1);
        const uint64_t n_child = lv.n(l - 1);
        for (uint32_t e = wv; e < n_front; e += kRayWaves) {
            const uint64_t child = (uint64_t)front[c][e] * kFan + lane;
            const bool ok = child < n_child && reach(boxes[child], 0.0f, INFINITY);
            const uint64_t m = __ballot(ok);
            uint32_t base = 0;
            if (lane == 0 && m) base = atomicAdd(&sh_n, (uint32_t)__popcll(m));
            base = uniform32(base) + lanes_below(m);
            if (ok) {
                if (base < kFront) front[c ^ 1][base] = (uint32_t)child;
                else sh_over = 1;
            }
        }
        __syncthreads();
        if (sh_over) break;   // keep the frontier of this level; its groups are all tested below
        n_front = sh_n;
        c ^= 1;
        --l;
    }
    const uint32_t* const nodes = front[c];
    const uint32_t down = 6 * (l - 1);   // log2 of the groups below a frontier node
    const uint64_t n_group = (uint64_t)n_front << down;
    // Every fragment with a depth in the slab that lands in the tile, kU
    // chunks at a time: fn(hits, keys, tile pixels) by all lanes. In rounds:
    // the waves test the chunks of kRoundGroups groups and queue those that
    // can reach the tile, then all draw the queue; the records are loaded two
    // steps ahead and their rows' keys one (a wave drawing the chunks of its
    // own groups, each step waiting for both, took 33 us where a tile has
    // 2,000 hits).
    constexpr int kU = 2;
    auto draw = [&](float dlo, float dhi, auto&& fn) {
        for (uint64_t e0 = 0; e0 < n_group; e0 += kRoundGroups) {
            __syncthreads();
            if (t == 0) sh_n = 0;
            __syncthreads();
            const uint64_t e1 = e0 + kRoundGroups < n_group ? e0 + kRoundGroups : n_group;
            for (uint64_t e = e0 + wv; e < e1; e += kRayWaves) {
                const uint64_t g = ((uint64_t)nodes[e >> down] << down) | (e & ((1ull << down) - 1ull));
                const uint64_t ch = g * kFan + lane;
                const bool ok = ch < lv.chunks && reach(a.area.box[ch < lv.chunks ? ch : 0], dlo, dhi);
                const uint64_t m = __ballot(ok);
                if (m == 0) continue;   // wave-uniform
                uint32_t base = 0;
                if (lane == 0) base = atomicAdd(&sh_n, (uint32_t)__popcll(m));
                base = uniform32(base);
                if (ok) queue[base + lanes_below(m)] = (uint32_t)ch;   // fewer than 2^26 chunks
            }
            __syncthreads();
            const uint32_t nq = sh_n;
            struct Step {
                uint32_t f[kU], x[kU], row[kU], key[kU];
            };
            auto load = [&](uint32_t i, Step& q) {
#pragma unroll
                for (int u = 0; u < kU; ++u) {
                    const uint32_t j = i + (uint32_t)(u * kRayWaves);
                    q.f[u] = (j < nq ? queue[j] : 0u) * kWave + (uint32_t)lane;
                    const bool ok = j < nq && q.f[u] < F;
                    const uint4 r = a.frag[ok ? q.f[u] : 0u];
                    q.x[u] = r.x;
                    q.row[u] = ok ? r.w : kNil;
                }
            };
            auto keys = [&](Step& q) {
#pragma unroll
                for (int u = 0; u < kU; ++u) q.key[u] = (uint32_t)a.rows.oct_key[q.row[u] < n_rows ? q.row[u] : 0u];
            };
            Step s0, s1, s2;
            constexpr uint32_t kStep = kU * kRayWaves;
            load(wv, s0);
            keys(s0);
            load(wv + kStep, s1);
            for (uint32_t i = wv; i < nq; i += kStep) {
                load(i + 2 * kStep, s2);
                keys(s1);
                bool in[kU];
                uint64_t k64[kU];
                uint32_t pix[kU];
#pragma unroll
                for (int u = 0; u < kU; ++u) {
                    uint32_t gx, gy, gz;
                    grid_pos(s0.x[u], s0.key[u], &gx, &gy, &gz);
                    const float x = (float)gx + 0.5f, y = (float)gy + 0.5f, z = (float)gz + 0.5f;
                    const float d = proj(M, 2, x, y, z);
                    const float fx = floorf(proj(M, 0, x, y, z)), fy = floorf(proj(M, 1, x, y, z));
                    in[u] = s0.row[u] < n_rows && d > 0.0f && fx >= X0 && fx < X1 && fy >= Y0 && fy < Y1;
                    k64[u] = ((uint64_t)__float_as_uint(d) << 32) | s0.f[u];
                    pix[u] = in[u] ? ((uint32_t)fy - y0) * kTile + ((uint32_t)fx - x0) : 0u;
                }
                fn(in, k64, pix);
                s0 = s1;
                s1 = s2;
            }
        }
    };
    const size_t o = ((size_t)v * a.height + py) * a.width + px;
    if (n_group == 0) {   // the whole workgroup
        if (mine) a.out[o] = make_float4(0.f, 0.f, 0.f, 0.f);
        return;
    }
    if (kMode == 0) {
        if (t < (uint32_t)kPix) hit[t] = ~0ull;
        __syncthreads();
        draw(0.0f, INFINITY, [&](const bool (&in)[kU], const uint64_t (&key)[kU], const uint32_t (&p)[kU]) {
#pragma unroll
            for (int u = 0; u < kU; ++u)
                if (in[u]) atomicMin(hit + p[u], (unsigned long long)key[u]);
        });
        __syncthreads();
        if (!mine) return;
        const uint64_t key = hit[t];
        float4 col = make_float4(0.f, 0.f, 0.f, 0.f);
        if (key != ~0ull) {
            const uint32_t rgba = a.frag[(uint32_t)key].y;
            col = make_float4((float)(rgba & 0xFFu) / 255.0f, (float)((rgba >> 8) & 0xFFu) / 255.0f,
                              (float)((rgba >> 16) & 0xFFu) / 255.0f, 1.0f);
        }
        a.out[o] = col;
        return;
    }
    if (t < 256) unit[t] = (float)t / 255.0f;
    float C0 = 0.0f, C1 = 0.0f, C2 = 0.0f, T = 1.0f;
    bool fin = !mine;
    // slabs [klo, khi) of keys, nearest first; `left`: hits at or beyond klo
    // once a slab up to the end has counted them, else 0
    uint64_t klo = 0, khi = ~0ull, left = 0;
    for (;;) {
        __syncthreads();
        if (t < (uint32_t)kPix) cnt[t] = fin ? kFinal : 0u;
        if (t == 0) {
            sh_hits = 0;
            sh_min = ~0ull;
            sh_max = 0;
        }
        __syncthreads();
        uint64_t kmin = ~0ull, kmax = 0;
        draw(__uint_as_float((uint32_t)(klo >> 32)), __uint_as_float((uint32_t)(khi >> 32)),
             [&](const bool (&in)[kU], const uint64_t (&key)[kU], const uint32_t (&p)[kU]) {
                 // pixels that are final take no more hits
                 uint64_t m[kU];
                 bool ok[kU];
                 uint32_t total = 0;
#pragma unroll
                 for (int u = 0; u < kU; ++u) {
                     ok[u] = in[u] && key[u] >= klo && key[u] < khi && cnt[p[u]] < kFinal;
                     m[u] = __ballot(ok[u]);
                     total += (uint32_t)__popcll(m[u]);
                 }
                 if (total == 0) return;   // wave-uniform
                 uint32_t base = 0;
                 if (lane == 0) base = atomicAdd(&sh_hits, total);
                 base = uniform32(base);
#pragma unroll
                 for (int u = 0; u < kU; ++u) {
                     const uint32_t at = base + lanes_below(m[u]);
                     base += (uint32_t)__popcll(m[u]);
                     if (!ok[u]) continue;
                     kmin = key[u] < kmin ? key[u] : kmin;
                     kmax = key[u] > kmax ? key[u] : kmax;
                     atomicAdd(cnt + p[u], 1u);
                     if (at < kHits) {
                         hit[at] = key[u];
                         hit_px[at] = (uint8_t)p[u];
                     }
                 }
             });
        __syncthreads();
        const uint32_t n = sh_hits;
        // where each pixel's hits start, and the most of any pixel
        const uint32_t mine_n = fin ? 0u : cnt[t];   // fin in all threads without a pixel
        const uint32_t sum = wave_incl_sum(mine_n);
        uint32_t most = wave_all_max(mine_n);
        if (lane == kWave - 1) {
            sh_sum[wv] = sum;
            sh_most[wv] = most;
        }
        __syncthreads();
        uint32_t before = sum - mine_n;
        most = 0;
#pragma unroll
        for (uint32_t w = 0; w < (uint32_t)kRayWaves; ++w) {
            before += w < wv ? sh_sum[w] : 0u;
            most = sh_most[w] > most ? sh_most[w] : most;
        }
        if (khi == ~0ull) left = n;
        if (n > kHits || most > kMostPerPixel) {
            // too many: a slab of about three quarters of what fits, as if
            // the hits were spread evenly over their keys (it holds the
            // nearest one at least and fewer than all)
            if (kmin <= kmax) {
                atomicMin(&sh_min, (unsigned long long)kmin);
                atomicMax(&sh_max, (unsigned long long)kmax);
            }
            __syncthreads();
            const double share = fmin(0.75 * (double)kHits / (double)n, 0.75 * (double)kMostPerPixel / (double)most);
            klo = sh_min;
            khi = klo + 1 + (uint64_t)(share * (double)(sh_max - klo));
            continue;
        }
        if (t < (uint32_t)kPix) off[t] = cur[t] = before;
        if (t == 0) off[kPix] = n;
        __syncthreads();
        // grouped by pixel (through registers, in place)
        uint64_t key[kPerThread];
        uint32_t to[kPerThread];   // pixel << 16 | place
#pragma unroll
        for (uint32_t k = 0; k < kPerThread; ++k) {
            if (k * kRayBlock >= n) continue;   // workgroup-uniform
            const uint32_t i = k * kRayBlock + t;
            key[k] = i < n ? hit[i] : 0;
            to[k] = i < n ? hit_px[i] : 0u;
            if (i < n) to[k] = (to[k] << 16) | atomicAdd(cur + to[k], 1u);
        }
        __syncthreads();
#pragma unroll
        for (uint32_t k = 0; k < kPerThread; ++k) {
            if (k * kRayBlock >= n) continue;
            if (k * kRayBlock + t < n) {
                hit[to[k] & 0xFFFFu] = key[k];
                hit_px[to[k] & 0xFFFFu] = (uint8_t)(to[k] >> 16);
            }
        }
        __syncthreads();
        // ordered: each hit counts the nearer ones of its pixel, and its
        // index goes to that place
        uint32_t idx[kPerThread], place[kPerThread];
#pragma unroll
        for (uint32_t k = 0; k < kPerThread; ++k) {
            if (k * kRayBlock >= n) continue;
            const uint32_t i = k * kRayBlock + t;
            if (i >= n) continue;
            const uint64_t x = hit[i];
            const uint32_t p = hit_px[i], lo = off[p], hi = off[p + 1];
            uint32_t nearer = 0;
#pragma unroll 4
            for (uint32_t j = lo; j < hi; ++j) nearer += hit[j] < x ? 1u : 0u;
            idx[k] = (uint32_t)x;
            place[k] = lo + nearer;
            __builtin_amdgcn_sched_barrier(0);   // one hit after the other: all at once would spill
        }
        __syncthreads();
        uint32_t* const order = (uint32_t*)hit;
#pragma unroll
        for (uint32_t k = 0; k < kPerThread; ++k) {
            if (k * kRayBlock >= n) continue;
            if (k * kRayBlock + t < n) order[place[k]] = idx[k];
        }
        __syncthreads();
        // composite front to back, four colours in flight
        const uint32_t end = fin ? 0u : off[t + 1];
        for (uint32_t j = fin ? 0u : off[t]; !fin && j < end; j += 4) {
            uint32_t rgba[4];
#pragma unroll
            for (uint32_t u = 0; u < 4; ++u) rgba[u] = a.frag[order[j + u < end ? j + u : j]].y;
#pragma unroll
            for (uint32_t u = 0; u < 4; ++u) {
                if (fin || j + u >= end) continue;
                const float al = unit[rgba[u] >> 24];
                const float wgt = T * al;
                C0 = C0 + wgt * unit[rgba[u] & 0xFFu];
                C1 = C1 + wgt * unit[(rgba[u] >> 8) & 0xFFu];
                C2 = C2 + wgt * unit[(rgba[u] >> 16) & 0xFFu];
                T = T * (1.0f - al);
                fin = T < a.tau || T == 0.0f;
            }
        }
        if (khi == ~0ull) break;
        // any pixel still compositing?
        const uint64_t open = __ballot(!fin);
        if (lane == 0) sh_most[wv] = open != 0 ? 1u : 0u;
        __syncthreads();
        uint32_t any = 0;
#pragma unroll
        for (uint32_t w = 0; w < (uint32_t)kRayWaves; ++w) any |= sh_most[w];
        if (any == 0) break;
        // the next slab: the rest if it fits, else as wide as this one, or
        // eight times as wide where this one held little. After an empty
        // slab the rest is counted, which finds where the hits go on: keys
        // leave gaps (between planes that face the view, 2^32 times their
        // depths' distance) that no width found inside a plane would cross.
        left = left > n ? left - n : 0;
        const uint64_t width = khi - klo;
        klo = khi;
        khi = ~0ull;
        if (left > kHits && n > 0) {
            const uint64_t wide = n >= kHits / 8 || most >= kMostPerPixel / 8 ? width
                                  : width < kPastKeys / 8 ? 8 * width : kPastKeys;
            // past the largest key (a depth of +inf) comes only the end: a
            // bound whose upper half reads as a negative depth would reject
            // every box (klo and wide are at most kPastKeys, below 2^63)
            if (klo + wide < kPastKeys) khi = klo + wide;
        }
    }
    if (mine) a.out[o] = make_float4(C0, C1, C2, 1.0f - T);
}

// -------------------------------------------------------------- octree walk

// Whether the tiles made the image: they ran at all (there was room for a
// box) and the fragments' boxes fitted.
__device__ __forceinline__ bool tiles_taken(const Rows& rows, uint64_t room)
{
    return room > 0 && BoxLevels(rows.frags()).total() <= room;
}

// The bitmaps cleared (n16 16-byte words), like all of the walk's kernels only
// where the tiles were not taken: at depth 10 the clear writes 153 MB, and the
// rank scan reads 268 and writes 67.
__global__ void __launch_bounds__(kBlock) k_occ_clear(Rows rows, uint64_t room, uint4* __restrict__ occ, uint64_t n16)
{
    if (tiles_taken(rows, room)) return;
    const uint64_t stride = (uint64_t)gridDim.x * kBlock;
    for (uint64_t i = (uint64_t)blockIdx.x * kBlock + threadIdx.x; i < n16; i += stride) occ[i] = make_uint4(0, 0, 0, 0);
}

struct SkipRanks {
    Rows rows;
    uint64_t room;
    __device__ bool operator()() const { return tiles_taken(rows, room); }
};

__global__ void __launch_bounds__(kBlock)
k_occ_build(Rows rows, uint64_t room, uint32_t* __restrict__ occ, OccLayout lay, uint32_t L)
{
    if (tiles_taken(rows, room)) return;
    const uint64_t n = rows.count();
    const uint64_t* __restrict__ const oct_key = rows.oct_key;
    const uint64_t stride = (uint64_t)gridDim.x * kBlock;
    for (uint64_t r = (uint64_t)blockIdx.x * kBlock + threadIdx.x; r < n; r += stride) {
        const uint64_t key = oct_key[r];
        const uint64_t prev = r > 0 ? oct_key[r - 1] : ~0ull;
        for (uint32_t l = L; l >= 1; --l) {
            const uint32_t sh = 3 * (L - l);
            const uint64_t b = key >> sh;
            if (l < L && r > 0 && (prev >> sh) == b) break;   // set by an earlier row
            atomicOr(occ + lay.word[l] + (b >> 5), 1u << (b & 31));
        }
    }
}

struct LoadPopc {
    const uint64_t* bits;
    __device__ uint32_t operator()(uint64_t i) const { return (uint32_t)__popcll(bits[i]); }
};

struct RayArgs {
    float m[kMaxViews][12];
    const uint4* frag;
    const uint64_t* oct_key;
    const uint32_t* oct_off;
    const uint32_t* oct_cnt;
    const uint32_t* occ;
    const uint32_t* rank;   // set leaf bits before each 64-bit word
    OccLayout lay;
    float4* out;            // [V][H][W]
    uint32_t order[kMaxViews];   // per view: child octants nearest first, 4 bits each
    uint32_t L, width, height, tiles_x, n_tiles;
    float tau;
    Rows rows;
    uint64_t room;          // boxes that the tiles' way has room for
};

__device__ __forceinline__ float wave_max(float x)
{
#pragma unroll
    for (int d = kWave / 2; d >= 1; d >>= 1) x = fmaxf(x, __shfl_xor(x, d, kWave));
    return __uint_as_float(__builtin_amdgcn_readfirstlane(__float_as_uint(x)));
}

__device__ __forceinline__ float wave_min(float x)
{
#pragma unroll
    for (int d = kWave / 2; d >= 1; d >>= 1) x = fminf(x, __shfl_xor(x, d, kWave));
    return __uint_as_float(__builtin_amdgcn_readfirstlane(__float_as_uint(x)));
}

// One wave per 8 x 8 pixel tile: the wave walks the octree once for the
// tile (its window is the tile, so every decision of the walk is uniform),
// projects a leaf's fragments one per lane and hands each fragment that
// lands in the tile to the lane owning its pixel. Per lane: the pixel's
// kept fragments, compositing state and depth window; the walk skips an
// octant only when it is outside the window of every lane still compositing.
template <int kMode>
__global__ void __launch_bounds__(kBlock) k_raycast(RayArgs a)
{
    // per-lane fragment list, interleaved so that lanes hit distinct banks
    __shared__ uint64_t lst[(kMode == 0 ? 1 : kCap) * kBlock];
    const int lane = __lane_id(), wv = threadIdx.x / kWave;
    const uint32_t tile = blockIdx.x * (kBlock / kWave) + wv;
    if (tile >= a.n_tiles) return;   // whole wave
    if (tiles_taken(a.rows, a.room)) return;
    const uint32_t x0 = (tile % a.tiles_x) * 8, y0 = (tile / a.tiles_x) * 8;
    const uint32_t px = x0 + (lane & 7), py = y0 + (lane >> 3);
    const bool mine = px < a.width && py < a.height;
    const uint32_t v = blockIdx.y;
    const float* M = a.m[v];
    const uint32_t L = a.L;
    const float tcx = (float)x0 + 4.0f, tcy = (float)y0 + 4.0f;
    const float ax = fabsf(M[0]) + fabsf(M[1]) + fabsf(M[2]), ay = fabsf(M[4]) + fabsf(M[5]) + fabsf(M[6]);
    const float az = fabsf(M[8]) + fabsf(M[9]) + fabsf(M[10]);
    // an octant's extent is widened as a box's is in k_ray_tile (along x and y
    // half the tile comes on top), without limit where a sum may overflow
    const float grid = (float)(256u << L);
    auto margin = [&](float abs_row, float off) -> float {
        const float t = abs_row * grid + fabsf(off) + 1.0f;
        return t < 0x1p126f ? 0x1p-20f * t : INFINITY;
    };
    const float mx4 = margin(ax, M[3]) + 4.0f, my4 = margin(ay, M[7]) + 4.0f, mz = margin(az, M[11]);
    const uint8_t* const occ8 = (const uint8_t*)a.occ;
    const uint64_t* const leaf64 = (const uint64_t*)(a.occ + a.lay.word[L]);
    uint64_t* const my = lst + threadIdx.x;
    const uint32_t order = a.order[v];
    const uint32_t my_c = (order >> (4 * (lane & 7))) & 7u;   // lanes 0..7 test child rank `lane`
    // the walk stops at bricks of 8^kBrick leaves (level B), whose fragments
    // are one contiguous range of the arrays: larger bricks trade fragment
    // tests, done 64 at a time, for fewer dependent loads along the walk
    // (measured best: 512 leaves for the nearest fragment, 64 with
    // transparency, where the walk stops earlier)
    constexpr uint32_t kBrick = kMode == 0 ? 3u : 2u;
    const uint32_t B = L > kBrick ? L - kBrick : 1;
    const uint64_t n_leaf = 1ull << (3 * L);
    // table rows of the leaves before Morton code k (k <= 8^L)
    auto rank_of = [&](uint64_t k) -> uint32_t {
        if (k >= n_leaf) return a.rank[a.lay.n64 - 1] + (uint32_t)__popcll(leaf64[a.lay.n64 - 1]);
        return a.rank[k >> 6] + (uint32_t)__popcll(leaf64[k >> 6] & ((1ull << (k & 63)) - 1ull));
    };

    // children of octant n (level l, origin o in leaves) that are occupied and
    // whose box can project into the tile; bit i stands for the i-th nearest
    // child of the view's order
    auto expand = [&](uint32_t l, uint32_t n, uint32_t ox, uint32_t oy, uint32_t oz) -> uint32_t {
        const uint32_t m = occ8[a.lay.word[l + 1] * 4 + n];
        const uint32_t hc = 1u << (L - l - 1);            // child side in leaves
        const float hw = (float)hc * 128.0f;              // half side in grid units
        const float X = (float)((ox + ((my_c >> 2) & 1u) * hc) * 256u) + hw;
        const float Y = (float)((oy + ((my_c >> 1) & 1u) * hc) * 256u) + hw;
        const float Z = (float)((oz + (my_c & 1u) * hc) * 256u) + hw;
        const float sx = proj(M, 0, X, Y, Z), sy = proj(M, 1, X, Y, Z);
        const bool ok = lane < 8 && ((m >> my_c) & 1u) && !(fabsf(sx - tcx) > hw * ax + mx4) &&
                        !(fabsf(sy - tcy) > hw * ay + my4);
        return (uint32_t)__ballot(ok) & 0xFFu;
    };

    float C0 = 0.0f, C1 = 0.0f, C2 = 0.0f, T = 1.0f;
    uint64_t after = 0;     // keys at or below this were composited
    bool walked = false;    // this lane composited in an earlier walk
    bool fin = !mine;       // this lane's pixel is final
    // composite one fragment (front to back); true when the pixel is final
    auto blend = [&](uint64_t key) -> bool {
        const uint32_t rgba = a.frag[(uint32_t)key].y;
        const float al = kMode == 0 ? 1.0f : (float)(rgba >> 24) / 255.0f;
        const float wgt = T * al;
        C0 = C0 + wgt * ((float)(rgba & 0xFFu) / 255.0f);
        C1 = C1 + wgt * ((float)((rgba >> 8) & 0xFFu) / 255.0f);
        C2 = C2 + wgt * ((float)((rgba >> 16) & 0xFFu) / 255.0f);
        T = T * (1.0f - al);
        after = key;
        walked = true;
        return T < a.tau || T == 0.0f;
    };
    for (;;) {
        // the lane's kept fragments are my[h .. n_in), ascending and below
        // `cut`: once a fragment is left out of a walk (list full, or its
        // octant skipped), no key at or above it may be kept in that walk,
        // so that what is composited stays in order. Depths beyond `far`
        // cannot enter the list; depths before `near` were composited.
        uint32_t h = 0, n_in = 0;
        bool over = false;
        uint64_t cut = ~0ull;
        float far = INFINITY;
        const float near = walked ? __uint_as_float((uint32_t)(after >> 32)) : -INFINITY;
        float wfar = wave_max(fin ? -INFINITY : far);
        const float wnear = wave_min(fin ? INFINITY : near);
        constexpr uint32_t cap = kMode == 0 ? 1u : (uint32_t)kCap;
        auto set_far = [&]() {
            float f = cut == ~0ull ? INFINITY : __uint_as_float((uint32_t)(cut >> 32));
            if (n_in - h == cap) f = fminf(f, __uint_as_float((uint32_t)(my[(n_in - 1) * kBlock] >> 32)));
            far = f;
        };
        auto take = [&](uint64_t key) {
            if (walked && key <= after) return;
            if (key >= cut) {
                over = true;
                return;
            }
            if (n_in == cap && h > 0) {   // reclaim the composited front
                for (uint32_t j = h; j < n_in; ++j) my[(j - h) * kBlock] = my[j * kBlock];
                n_in -= h;
                h = 0;
            }
            if (n_in == cap) {
                over = true;
                const uint64_t last = my[(cap - 1) * kBlock];
                if (key > last) {
                    cut = key;
                    set_far();
                    return;
                }
                cut = last;   // the farthest kept fragment makes room
                n_in = cap - 1;
            }
            uint32_t j = n_in;
            while (j > h && my[(j - 1) * kBlock] > key) {
                my[j * kBlock] = my[(j - 1) * kBlock];
                --j;
            }
            my[j * kBlock] = key;
            ++n_in;
            set_far();
        };
        // composite the kept fragments nearer than `front` (nothing still
        // unvisited can come before them), or all of them: depths may be
        // infinite, and a walk that composited none of those would be
        // repeated for ever
        auto drain = [&](bool all, float front) {
            while (!fin && h < n_in) {
                const uint64_t key = my[h * kBlock];
                if (!all && !(__uint_as_float((uint32_t)(key >> 32)) < front)) break;
                ++h;
                if (blend(key)) fin = true;
            }
        };
        // depth-first walk without a stack: per level the children still to
        // visit (8 bits each, levels 0..7 and 8..15 in two words)
        uint64_t mlo = 0, mhi = 0;
        auto get_m = [&](uint32_t l) -> uint32_t {
            return (uint32_t)(((l < 8 ? mlo : mhi) >> ((l & 7) * 8)) & 0xFFu);
        };
        auto set_m = [&](uint32_t l, uint32_t m) {
            const uint32_t sh = (l & 7) * 8;
            if (l < 8)
                mlo = (mlo & ~(0xFFull << sh)) | ((uint64_t)m << sh);
            else
                mhi = (mhi & ~(0xFFull << sh)) | ((uint64_t)m << sh);
        };
        uint32_t l = 0, n = 0, ox = 0, oy = 0, oz = 0;
        // nearest depth any unvisited octant of the walk can hold: the
        // nearest pending child on every level of the current path
        auto frontier = [&]() -> float {
            float f = INFINITY;
            for (uint32_t k = 0; k <= l; ++k) {
                const uint32_t m = get_m(k);
                if (m == 0) continue;
                const uint32_t c = (order >> (4 * (__ffs(m) - 1))) & 7u;
                const uint32_t side = 1u << (L - k), hc = side >> 1;
                const float hw = (float)hc * 128.0f;
                const float dc = proj(M, 2, (float)(((ox & ~(side - 1)) + ((c >> 2) & 1u) * hc) * 256u) + hw,
                                      (float)(((oy & ~(side - 1)) + ((c >> 1) & 1u) * hc) * 256u) + hw,
                                      (float)(((oz & ~(side - 1)) + (c & 1u) * hc) * 256u) + hw);
                f = fminf(f, dc - hw * az);
            }
            return mz < INFINITY ? f - mz : -INFINITY;
        };
        set_m(0, expand(0, 0, 0, 0, 0));
        for (;;) {
            const uint32_t m = get_m(l);
            if (m == 0) {
                if (l == 0) break;
                --l;
                n >>= 3;
                const uint32_t side = 1u << (L - l);
                ox &= ~(side - 1);
                oy &= ~(side - 1);
                oz &= ~(side - 1);
                continue;
            }
            const uint32_t c = (order >> (4 * (__ffs(m) - 1))) & 7u;
            set_m(l, m & (m - 1));
            const uint32_t hc = 1u << (L - l - 1);
            const uint32_t cx = ox + ((c >> 2) & 1u) * hc, cy = oy + ((c >> 1) & 1u) * hc,
                           cz = oz + (c & 1u) * hc;
            const uint32_t cn = n * 8 + c;
            {
                // the child's depth range against the lanes' windows
                const float hw = (float)hc * 128.0f;
                const float dc = proj(M, 2, (float)(cx * 256u) + hw, (float)(cy * 256u) + hw, (float)(cz * 256u) + hw);
                if (dc - hw * az > wfar + mz) {
                    // behind every compositing lane's window: left out of
                    // this walk, with everything as deep or deeper
                    if (!fin) {
                        over = true;
                        const uint64_t c2 = (uint64_t)(__float_as_uint(wfar) + 1u) << 32;
                        if (c2 < cut) {
                            cut = c2;
                            set_far();
                        }
                    }
                    continue;
                }
                if (dc + hw * az < wnear - mz) continue;
            }
            if (l + 1 < B) {
                ++l;
                n = cn;
                ox = cx;
                oy = cy;
                oz = cz;
                set_m(l, expand(l, n, ox, oy, oz));
                continue;
            }
            // brick cn: its leaves are consecutive Morton codes, so their
            // table rows and their fragments are consecutive too
            const uint32_t bs = 3 * (L - B);
            const uint32_t row_lo = rank_of((uint64_t)cn << bs);
            const uint32_t row_hi = rank_of((uint64_t)(cn + 1) << bs);
            const uint32_t off = row_hi > row_lo ? a.oct_off[row_lo] : 0u;
            const uint32_t cnt = row_hi > row_lo ? a.oct_off[row_hi - 1] + a.oct_cnt[row_hi - 1] - off : 0u;
            for (uint32_t b = 0; b < cnt; b += kWave) {
                bool hit = false;
                uint32_t t = 0;
                uint64_t key = 0;
                if (b + (uint32_t)lane < cnt) {
                    const uint32_t i = off + b + (uint32_t)lane;
                    const uint4 r = a.frag[i];
                    const uint64_t lk = a.oct_key[r.w];   // the fragment's leaf
                    const uint32_t lx = compact3(lk >> 2), ly = compact3(lk >> 1), lz = compact3(lk);
                    const float x = (float)((lx << 8) | (r.x & 0xFFu)) + 0.5f;
                    const float y = (float)((ly << 8) | ((r.x >> 8) & 0xFFu)) + 0.5f;
                    const float z = (float)((lz << 8) | ((r.x >> 16) & 0xFFu)) + 0.5f;
                    const float d = proj(M, 2, x, y, z);
                    const float fx = floorf(proj(M, 0, x, y, z)), fy = floorf(proj(M, 1, x, y, z));
                    if (d > 0.0f && fx >= (float)x0 && fx < (float)(x0 + 8) && fy >= (float)y0 &&
                        fy < (float)(y0 + 8)) {
                        hit = true;
                        t = ((uint32_t)fy - y0) * 8 + ((uint32_t)fx - x0);
                        key = ((uint64_t)__float_as_uint(d) << 32) | i;
                    }
                }
                // hand every hit to the lane that owns its pixel
                for (uint64_t bal = __ballot(hit); bal; bal &= bal - 1) {
                    const int s = __ffsll((unsigned long long)bal) - 1;
                    const uint32_t ts = (uint32_t)__shfl((int)t, s, kWave);
                    const uint64_t ks = ((uint64_t)(uint32_t)__shfl((int)(uint32_t)(key >> 32), s, kWave) << 32) |
                                        (uint32_t)__shfl((int)(uint32_t)key, s, kWave);
                    if ((uint32_t)lane == ts && !fin) take(ks);
                }
            }
            drain(false, frontier());
            if (__ballot(!fin) == 0) break;   // every pixel of the tile is final
            wfar = wave_max(fin ? -INFINITY : far);
        }
        // the walk is complete: everything kept can be composited
        drain(true, 0.0f);
        if (!fin && !over) fin = true;   // nothing was left out
        if (__ballot(!fin) == 0) break;
    }
    if (mine) a.out[((size_t)v * a.height + py) * a.width + px] = make_float4(C0, C1, C2, 1.0f - T);
}

}  // namespace

size_t raycast_ws_bytes(uint32_t levels)
{
    if (levels < 1 || levels > kMaxRayLevels) return 0;
    const OccLayout o = occ_layout(levels);
    const size_t occ_b = (size_t)o.word[levels + 1] * 4;
    const size_t rank_b = ((size_t)o.n64 * 4 + 255) & ~(size_t)255;
    const size_t part_b = (scan_partials(o.n64) * 4 + 255) & ~(size_t)255;
    return ((occ_b + 255) & ~(size_t)255) + rank_b + part_b;
}

hipError_t raycast_launch(const Device& dev, const fhv_pofa* p, uint32_t levels, const RayViews& rv,
                          uint32_t mode, float tau, float* out, void* ws, size_t ws_bytes, hipStream_t s)
{
    const OccLayout lay = occ_layout(levels);
    const size_t occ_b = (((size_t)lay.word[levels + 1] * 4) + 255) & ~(size_t)255;
    const size_t rank_b = ((size_t)lay.n64 * 4 + 255) & ~(size_t)255;
    uint32_t* occ = (uint32_t*)ws;
    uint32_t* rank = (uint32_t*)((char*)ws + occ_b);
    uint32_t* part = (uint32_t*)((char*)ws + occ_b + rank_b);
    const Rows rows{p->oct_key, p->oct_off, p->oct_cnt, p->n_occ, p->cap_occ, p->cap_frag};
    if (p->cap_occ == 0 || p->cap_frag == 0) {
        // no stored row or no record: no ray meets anything
        ProfScope ps(dev, "ray.tiles", s);
        return fill_u32((uint32_t*)out, 4ull * rv.n_views * rv.width * rv.height, 0u, s);
    }
    // the tiles' boxes: a word for the fragment count, then 16 bytes each
    BoxArea area{nullptr, nullptr, 0};
    const uintptr_t base = ((uintptr_t)ws + 255) & ~(uintptr_t)255, end = (uintptr_t)ws + ws_bytes;
    if (end >= base + 256 + sizeof(uint4)) {
        area.frags = (uint64_t*)base;
        area.box = (uint4*)(base + 256);
        area.room = (end - base - 256) / sizeof(uint4);
    }
    const BoxLevels most(p->cap_frag);
    hipError_t e;
    if (area.room > 0) {
        const uint32_t bits = levels + 8, qs = bits > 16 ? bits - 16 : 0;
        // levels that may be built: no more boxes than there is room for
        const uint64_t nodes = std::min(most.total(), area.room);
        {
            ProfScope ps(dev, "ray.boxes", s);
            const uint64_t g = (std::min(most.chunks, nodes) + kFan - 1) / kFan, gmax = (uint64_t)dev.cus * 16;
            k_ray_box<<<dim3((unsigned)std::max<uint64_t>(1, std::min(g, gmax))), dim3(kBlock), 0, s>>>(
                (const uint4*)p->frag, rows, area, qs);
            if ((e = hipGetLastError()) != hipSuccess) return e;
            for (uint32_t l = 2; l <= most.top(); ++l) {
                const uint64_t gn = (most.n(l) + kBlock / kWave - 1) / (kBlock / kWave);
                k_ray_node<<<dim3((unsigned)std::min(gn, gmax)), dim3(kBlock), 0, s>>>(area, l);
                if ((e = hipGetLastError()) != hipSuccess) return e;
            }
        }
        RayTileArgs a;
        for (uint32_t v = 0; v < rv.n_views; ++v)
            for (int k = 0; k < 12; ++k) a.m[v][k] = rv.m[v][k];
        a.frag = (const uint4*)p->frag;
        a.rows = rows;
        a.area = area;
        a.out = (float4*)out;
        a.width = rv.width;
        a.height = rv.height;
        a.tiles_x = (rv.width + kTile - 1) / kTile;
        a.qs = qs;
        a.grid = (float)(1u << bits);
        a.tau = tau;
        const dim3 grid(a.tiles_x * ((rv.height + kTile - 1) / kTile), rv.n_views);
        ProfScope ps(dev, "ray.tiles", s);
        if (mode == FHV_RAY_NEAREST)
            k_ray_tile<0><<<grid, dim3(kRayBlock), 0, s>>>(a);
        else
            k_ray_tile<1><<<grid, dim3(kRayBlock), 0, s>>>(a);
        if ((e = hipGetLastError()) != hipSuccess) return e;
        if (most.total() <= area.room) return hipSuccess;   // any number of fragments fits
    }
    {
        ProfScope ps(dev, "ray.occupancy", s);
        const uint64_t n16 = occ_b / 16;   // up to the ranks
        const auto grid = [&](uint64_t n, uint64_t per_cu) {
            return dim3((unsigned)std::min((n + kBlock - 1) / kBlock, (uint64_t)dev.cus * per_cu));
        };
        k_occ_clear<<<grid(n16, 32), dim3(kBlock), 0, s>>>(rows, area.room, (uint4*)occ, n16);
        if ((e = hipGetLastError()) != hipSuccess) return e;
        k_occ_build<<<grid(p->cap_occ, 8), dim3(kBlock), 0, s>>>(rows, area.room, occ, lay, levels);
        if ((e = hipGetLastError()) != hipSuccess) return e;
        e = scan<uint32_t>(LoadPopc{(const uint64_t*)(occ + lay.word[levels])}, StoreExcl<uint32_t>{rank},
                           lay.n64, part, (uint32_t*)nullptr, s, SkipRanks{rows, area.room});
        if (e != hipSuccess) return e;
    }
    RayArgs a;
    for (uint32_t v = 0; v < rv.n_views; ++v) {
        for (int k = 0; k < 12; ++k) a.m[v][k] = rv.m[v][k];
        // children by the depth of their offset (x, y, z) in {0, 1}^3,
        // nearest first (Morton child index x << 2 | y << 1 | z)
        uint32_t idx[8];
        float dep[8];
        for (uint32_t c = 0; c < 8; ++c) {
            idx[c] = c;
            dep[c] = rv.m[v][8] * (float)((c >> 2) & 1u) + rv.m[v][9] * (float)((c >> 1) & 1u) +
                     rv.m[v][10] * (float)(c & 1u);
        }
        for (int i = 1; i < 8; ++i)
            for (int j = i; j > 0 && dep[idx[j]] < dep[idx[j - 1]]; --j) {
                const uint32_t t = idx[j];
                idx[j] = idx[j - 1];
                idx[j - 1] = t;
            }
        a.order[v] = 0;
        for (int i = 0; i < 8; ++i) a.order[v] |= idx[i] << (4 * i);
    }
    a.frag = (const uint4*)p->frag;
    a.oct_key = p->oct_key;
    a.oct_off = p->oct_off;
    a.oct_cnt = p->oct_cnt;
    a.occ = occ;
    a.rank = rank;
    a.lay = lay;
    a.out = (float4*)out;
    a.L = levels;
    a.width = rv.width;
    a.height = rv.height;
    a.tiles_x = (rv.width + 7) / 8;
    a.n_tiles = a.tiles_x * ((rv.height + 7) / 8);
    a.tau = tau;
    a.rows = rows;
    a.room = area.room;
    const dim3 grid((a.n_tiles + kBlock / kWave - 1) / (kBlock / kWave), rv.n_views);
    ProfScope ps(dev, "ray.cast", s);
    if (mode == FHV_RAY_NEAREST)
        k_raycast<0><<<grid, dim3(kBlock), 0, s>>>(a);
    else
        k_raycast<1><<<grid, dim3(kBlock), 0, s>>>(a);
    return hipGetLastError();
}

}  // namespace fhv
